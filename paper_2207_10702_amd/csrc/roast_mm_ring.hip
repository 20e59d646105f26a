// Forward Y = X*W and dX = dY*W^T (Algorithm 1 and Section 4.3 of arXiv 2207.10702) of mid-sized bf16 calls on gfx950: 64 x 64 blocks,
// for calls with a copy of M, tiles that are multiples of 32 and whole blocks of columns.
//
// What bounds them is the fill of a CU, and that by the lines of 128 bytes that a load touches: an XCD's L2 gives each of its 32 CUs 64 bytes a
// clock of whole lines, 32 where a load takes half of each.  So a wave loads 64 contraction indices at a time, whole lines of A and (where a tile is as
// wide as the block) a run of M, straight into LDS, 16 bytes per lane.  The 16 KiB are its own: it reads nothing that another wave
// has loaded, the loop has no barrier, and while it multiplies, the next 16 KiB are on their way, 128 KiB to a CU.
// 512 x 2048 x 2048 15.5 -> 10.7 us (half lines of 32 indices at a time, two in flight: 11.4).  A further load ahead, of a line's first dword, makes it 11.3.
// Few blocks and a long contraction take parts of it, with a workspace: 41 x 13440 x 1280 20.9 -> 13 us, 265 x 6272 x 768 22.0 -> 12.9, where 128 x 192 blocks spend most
// of their rows on nothing.
#include <algorithm>
#include <atomic>

#include "roast_internal.hpp"

namespace roast {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));

constexpr int kWaves = 8, kUnit = 32, kHalf = 8192, kOwn = 2 * kHalf;   // contraction indices of a unit, of which two are loaded at a time; bytes of an operand, of a wave
constexpr int kTable = 2048;             // tile-table entries (4 bytes each)

struct RingArgs {
  MMArgs a;
  TileHash th;
  const uint16_t* A;                     // FWD: X, DX: dY
  int64_t lda;
  const uint16_t* Mb;                    // the copy of M (see roast_mm_wide.hip)
  int64_t mb_stride;
  uint16_t* C;
  int64_t ldc;
  int nbx, nby;
  float* G;                              // partial outputs of a split contraction, [part][rows][columns], or null
  int parts;
};

__device__ inline uint32_t pack_bf16x2(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 r = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, r);
}

// 16 bytes per lane from (uniform base) + (lane's byte offset) to LDS: lane l lands at lds + 16 * l
__device__ __forceinline__ void load_to_lds(const uint16_t* base, uint32_t bytes, uint32_t lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)((const char*)base + bytes),
                                   (__attribute__((address_space(3))) void*)(uintptr_t)lds, 16, 0, 0);
}
constexpr int vmcnt_only(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0f70; }

// LDS reads with their wait: in assembly, because the compiler would make every LDS read wait for all direct-to-LDS loads in flight.
// Rows along the contraction, 128 bytes each: f[4 ks + i] is fragment i (16 rows, 2 KiB on) of the unit ks (at1 = at0 with its chunks moved on by four).
__device__ __forceinline__ void read_rows(uint4v* f, uint32_t at0, uint32_t at1) {
  asm volatile(
      "ds_read_b128 %0, %8\n\tds_read_b128 %1, %8 offset:2048\n\tds_read_b128 %2, %8 offset:4096\n\tds_read_b128 %3, %8 offset:6144\n\t"
      "ds_read_b128 %4, %9\n\tds_read_b128 %5, %9 offset:2048\n\tds_read_b128 %6, %9 offset:4096\n\tds_read_b128 %7, %9 offset:6144\n\ts_waitcnt lgkmcnt(0)"
      : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]), "=&v"(f[7])
      : "v"(at0), "v"(at1)
      : "memory");
}
// Rows across the contraction, [k][64 columns], by transposing reads: lanes 4r .. 4r+3 of a group of 16 give the addresses of
// row r (k = r resp. 4 + r), lane c receives the eight k-values of column c.
__device__ __forceinline__ void read_columns(uint4v* f, uint32_t at) {
  uint2v l[8], h[8];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %1, %16 offset:512\n\tds_read_b64_tr_b16 %2, %17\n\tds_read_b64_tr_b16 %3, %17 offset:512\n\t"
      "ds_read_b64_tr_b16 %4, %18\n\tds_read_b64_tr_b16 %5, %18 offset:512\n\tds_read_b64_tr_b16 %6, %19\n\tds_read_b64_tr_b16 %7, %19 offset:512\n\t"
      "ds_read_b64_tr_b16 %8, %16 offset:4096\n\tds_read_b64_tr_b16 %9, %16 offset:4608\n\tds_read_b64_tr_b16 %10, %17 offset:4096\n\tds_read_b64_tr_b16 %11, %17 offset:4608\n\t"
      "ds_read_b64_tr_b16 %12, %18 offset:4096\n\tds_read_b64_tr_b16 %13, %18 offset:4608\n\tds_read_b64_tr_b16 %14, %19 offset:4096\n\tds_read_b64_tr_b16 %15, %19 offset:4608\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(l[0]), "=&v"(h[0]), "=&v"(l[1]), "=&v"(h[1]), "=&v"(l[2]), "=&v"(h[2]), "=&v"(l[3]), "=&v"(h[3]), "=&v"(l[4]), "=&v"(h[4]), "=&v"(l[5]), "=&v"(h[5]),
        "=&v"(l[6]), "=&v"(h[6]), "=&v"(l[7]), "=&v"(h[7])
      : "v"(at), "v"(at ^ 32u), "v"(at ^ 64u), "v"(at ^ 96u)
      : "memory");
#pragma unroll
  for (int j = 0; j < 8; ++j) f[j] = uint4v{l[j][0], l[j][1], h[j][0], h[j][1]};
}
// tile-table entries
__device__ __forceinline__ void read_entries(uint32_t* e, const uint32_t* at) {
  asm volatile("ds_read_b32 %0, %5\n\tds_read_b32 %1, %6\n\tds_read_b32 %2, %7\n\tds_read_b32 %3, %8\n\tds_read_b32 %4, %9\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(e[0]), "=&v"(e[1]), "=&v"(e[2]), "=&v"(e[3]), "=&v"(e[4])
               : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4])
               : "memory");
}

// A region of LDS: 64 rows of 64 contraction indices, [row][64 k], or 64 contraction indices of 64 columns, [k][64 columns].  A wave loads
// one, eight rows of 128 bytes to an instruction; the 16-byte chunks of a row are permuted, on the source address (a direct load fills
// LDS linearly) and on the read, which meets no bank twice in a clock then: by row / 2, or in pairs by swz(k).
__device__ __forceinline__ int swz(int k) { return ((k >> 1) & 1) | (((k >> 3) & 1) << 1); }
__device__ __forceinline__ int row_chunk(int v) {
  const int lane = threadIdx.x & 63;
  return (lane & 7) ^ (((8 * v + (lane >> 3)) >> 1) & 7);
}
__device__ __forceinline__ int column_of(int v) {  // of the lane's chunk in k-row 8 v + lane / 8
  const int lane = threadIdx.x & 63;
  return 16 * (((lane & 7) >> 1) ^ swz(8 * v + (lane >> 3))) + 8 * (lane & 1);
}
// fragments: lane 16 g + r holds the contraction indices 8 g .. of row (column) r
__device__ __forceinline__ uint32_t rows_at(uint32_t region) {
  const uint32_t r = threadIdx.x & 15, g = (threadIdx.x & 63) >> 4;
  return region + r * 128 + ((g ^ (r >> 1)) << 4);
}
__device__ __forceinline__ uint32_t columns_at(uint32_t region) {
  const uint32_t l = threadIdx.x & 63, tk = 8 * (l >> 4) + ((l & 15) >> 2);
  return region + tk * 128 + ((uint32_t)swz((int)tk) << 5) + (l & 3) * 8;
}

// rows m0 .. of A; those beyond the last one repeat it, they are not stored
struct RowLoads {
  const uint16_t* base;
  uint32_t off[8];
  __device__ void init(const uint16_t* A, int64_t lda, int m0, int I) {
    base = A + (int64_t)m0 * lda;
#pragma unroll
    for (int v = 0; v < 8; ++v) off[v] = (uint32_t)min(8 * v + (int)((threadIdx.x & 63) >> 3), I - 1 - m0) * ((uint32_t)lda * 2u) + 16u * (uint32_t)row_chunk(v);
  }
  __device__ void load(int k, uint32_t region) const {
#pragma unroll
    for (int v = 0; v < 8; ++v) load_to_lds(base + k, off[v], region + 1024 * v);
  }
};

// where 64 contraction indices start in their hash tile, and its row in the table (bytes); the second 32 of them
struct Pos {
  int in, row;
};
__device__ __forceinline__ Pos next_unit(const Pos& s, int zk, int row_bytes) {
  return s.in + kUnit >= zk ? Pos{0, s.row + row_bytes} : Pos{s.in + kUnit, s.row};
}

// Weights of columns n0 .. n0 + 63 (DX: rows of W).  Table: row = tile along the contraction, column = tile along the block's columns, from c0 on.
// A lane's v-th load takes entry (v / 4, v & 1): FWD: k-rows 8 v .., whose columns depend on v & 1; DX: rows 8 v .. of W, along the contraction, whose chunk does.
template <bool DX>
struct WeightLoads {
  uint32_t tab[4], half[4], in[8];       // half: which 32 contraction indices an entry is for
  uint32_t sg_tab, sg_half;              // of the sign that the lane looks up: fragment lane & 3 of the first (second) 32
  __device__ void init(const MMArgs& a, uint32_t table, int n0, int c0) {
    const int lane = threadIdx.x & 63, lr = lane >> 3, zn = DX ? a.Z1 : a.Z2;
#pragma unroll
    for (int v = 0; v < 8; ++v) {
      const int e = 2 * (v >> 2) + (v & 1), ch = row_chunk(v), n = DX ? n0 + 8 * v : n0 + column_of(v);
      if ((v & 2) == 0) {
        tab[e] = table + 4u * (uint32_t)(n / zn - c0);
        half[e] = DX ? (uint32_t)ch >> 2 : (uint32_t)v >> 2;
      }
      in[v] = 2u * (uint32_t)(DX ? (n % zn + lr) * a.Z2 + 8 * (ch & 3) : ((8 * v + lr) & 31) * a.Z2 + n % zn);
    }
    sg_tab = table + 4u * (uint32_t)((n0 + 16 * (lane & 3)) / zn - c0);
    sg_half = (uint32_t)(lane >> 2) & 1u;
  }
  // table addresses for the 64 contraction indices from s, t = next_unit(s), and for the signs of those from s1, t1
  __device__ void entries(const Pos& s, const Pos& t, const Pos& s1, const Pos& t1, uint32_t* at) const {
#pragma unroll
    for (int e = 0; e < 4; ++e) at[e] = tab[e] + (uint32_t)(half[e] ? t.row : s.row);
    at[4] = sg_tab + (uint32_t)(sg_half ? t1.row : s1.row);
  }
  __device__ void load(const uint16_t* Mb, int Z2, const Pos& s, const Pos& t, const uint32_t* e, uint32_t region) const {
    const uint32_t i0 = 2u * (uint32_t)(DX ? s.in : s.in * Z2), i1 = 2u * (uint32_t)(DX ? t.in : t.in * Z2);
#pragma unroll
    for (int v = 0; v < 8; ++v) {
      const int q = 2 * (v >> 2) + (v & 1);
      load_to_lds(Mb, 2u * e[q] + in[v] + (half[q] ? i1 : i0), region + 1024 * v);     // (doubling an entry drops the sign)
    }
  }
};
// NEG: the copy of M holds -M too and the sign picks the half; else it is an XOR of the weight fragments, by the entries' bit 31.
template <bool NEG>
__device__ __forceinline__ void fill_table(uint32_t* s_tab, const MMArgs& a, const TileHash& th, int64_t mb_stride, bool dx, int rows, int k0, int TN, int c0) {
  for (int e = threadIdx.x; e < rows * TN; e += blockDim.x) {
    const int ek = k0 + e / TN, en = c0 + e % TN;
    bool neg;
    const int64_t off = tile_place(a.hash, th, a.layer, (uint32_t)(dx ? en : ek), (uint32_t)(dx ? ek : en), &neg);
    // an odd offset is read from the second copy, where it is dword-aligned (everything added to it is even)
    const uint32_t o32 = (uint32_t)((off & 1) ? mb_stride + off - 1 : off);
    s_tab[e] = NEG ? o32 + (neg ? 2u * (uint32_t)mb_stride : 0u) : o32 | (neg ? 0x80000000u : 0u);
  }
}
__device__ __forceinline__ void put_signs(uint4v* bf, uint32_t entry) {
  const uint32_t signs = (uint32_t)__builtin_amdgcn_ballot_w64((int)entry < 0);
#pragma unroll
  for (int j = 0; j < 8; ++j) bf[j] ^= (uint32_t)((int)(signs << (31 - j)) >> 31) & 0x80008000u;
}
// the products of 32 contraction indices; weight (dM: dY) fragment first: a lane then holds 4 consecutive output columns of one output row
__device__ __forceinline__ void products(floatx4 (*acc)[4], const uint4v* af, const uint4v* bf) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, bf[j]), __builtin_bit_cast(bf16x8, af[i]), acc[i][j], 0, 0, 0);
}

template <bool DX, bool NEG>
__global__ __launch_bounds__(64 * kWaves, 2) void k_mm_ring(RingArgs p) {
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  uint32_t* s_tab = reinterpret_cast<uint32_t*>(smem + kWaves * kOwn);
  const MMArgs& a = p.a;
  const int K = DX ? (int)a.O : (int)a.H, I = (int)a.I;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Workgroups go to the 8 XCDs round-robin: XCD j takes the j-th eighth of the blocks, rows fastest, so that few columns of weights pass through its L2.
  const int plane = p.nbx * p.nby, total = plane * p.parts, chunk = (total + 7) / 8, t = ((int)blockIdx.x & 7) * chunk + ((int)blockIdx.x >> 3);
  if (((int)blockIdx.x >> 3) >= chunk || t >= total) return;      // whole workgroup leaves before any barrier
  const int bz = t / plane, bx = (t - bz * plane) / p.nby, by = t - bz * plane - bx * p.nby, m0 = 64 * by, n0 = 64 * bx;
  // The shares of the contraction are those of the kernels without a copy of M, whose sums are the same; a pair of units that two waves
  // share is loaded by both.
  const int u0 = 2 * (K / 64 * bz / p.parts), units = 2 * (K / 64 * (bz + 1) / p.parts) - u0;
  const int first = u0 + units * wave / kWaves, end = u0 + units * (wave + 1) / kWaves;
  const int p0 = first >> 1, p1 = (end + 1) >> 1;  // pairs (an empty share: none, or one without products)
  const uint32_t lds = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem);
  const uint32_t own = lds + wave * kOwn, tab = lds + kWaves * kOwn;
  RowLoads rows;
  rows.init(p.A, p.lda, m0, I);
  if (p0 < p1) rows.load(2 * kUnit * p0, own);
  const int zk = DX ? a.Z2 : a.Z1, zn = DX ? a.Z1 : a.Z2, c0 = n0 / zn, TN = (n0 + 63) / zn - c0 + 1, row_bytes = 4 * TN;
  WeightLoads<DX> weights;
  weights.init(a, tab, n0, c0);
  const int k0 = u0 * kUnit / zk;        // first tile along the contraction
  fill_table<NEG>(s_tab, a, p.th, p.mb_stride, DX, ((u0 + units) * kUnit - 1) / zk + 1 - k0, k0, TN, c0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  Pos pos = {2 * kUnit * p0 % zk, (2 * kUnit * p0 / zk - k0) * row_bytes};
  uint32_t at[5], e[5];
  if (p0 < p1) {
    const Pos half = next_unit(pos, zk, row_bytes);
    weights.entries(pos, half, pos, half, at);
    read_entries(e, at);
    weights.load(p.Mb, a.Z2, pos, half, e, own + kHalf);
  }
  floatx4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const uint32_t a_rd = rows_at(own), b_rd = DX ? rows_at(own + kHalf) : columns_at(own + kHalf);
#pragma unroll 1
  for (int pair = p0; pair < p1; ++pair) {
    __builtin_amdgcn_s_waitcnt(vmcnt_only(0));
    uint4v af[8], bf[8];
    const bool more = pair + 1 < p1;
    const Pos half = next_unit(pos, zk, row_bytes), next = more ? next_unit(half, zk, row_bytes) : pos, next_half = next_unit(next, zk, row_bytes);
    weights.entries(next, more ? next_half : half, pos, half, at);
    read_entries(e, at);
    read_rows(af, a_rd, a_rd ^ 64u);
    if constexpr (DX) read_rows(bf, b_rd, b_rd ^ 64u);
    else read_columns(bf, b_rd);
    if (more) {
      rows.load(2 * kUnit * (pair + 1), own);
      weights.load(p.Mb, a.Z2, next, next_half, e, own + kHalf);
    }
    if constexpr (!NEG) put_signs(bf, e[4]);
    if (2 * pair >= first) products(acc, af, bf);
    if (2 * pair + 1 < end) products(acc, af + 4, bf + 4);
    pos = next;
  }
  // acc[i][j][e]: row 16 i + r, column 16 j + 4 g + e.  The sums of the waves meet in LDS, wave 0's first; the pieces of four columns of a row are permuted by the row.
  __syncthreads();
  float* part = reinterpret_cast<float*>(smem);
  const int r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) *reinterpret_cast<floatx4*>(part + wave * 4096 + (16 * i + r) * 64 + 4 * ((4 * j + g) ^ r)) = acc[i][j];
  __syncthreads();
  const int orow = tid >> 3, oc = tid & 7;        // a thread adds up eight columns
  if (m0 + orow >= I) return;
  floatx4 sum[2];
#pragma unroll
  for (int w = 0; w < kWaves; ++w)
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const floatx4 x = *reinterpret_cast<const floatx4*>(part + w * 4096 + orow * 64 + 4 * ((2 * oc + v) ^ (orow & 15)));
      sum[v] = w == 0 ? x : sum[v] + x;
    }
  if (p.G) {
    float* to = p.G + ((int64_t)bz * I + m0 + orow) * (DX ? a.H : a.O) + n0 + 8 * oc;
#pragma unroll
    for (int v = 0; v < 2; ++v) *reinterpret_cast<floatx4*>(to + 4 * v) = a.lambda * sum[v];
    return;
  }
  uint4v out;
#pragma unroll
  for (int d = 0; d < 4; ++d) out[d] = pack_bf16x2(a.lambda * sum[d / 2][2 * (d & 1)], a.lambda * sum[d / 2][2 * (d & 1) + 1]);
  *reinterpret_cast<uint4v*>(p.C + (int64_t)(m0 + orow) * p.ldc + n0 + 8 * oc) = out;
}

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

template <bool DX, bool NEG>
roast_status launch(const RingArgs& p, hipStream_t s) {
  const int64_t total = (int64_t)p.nbx * p.nby * p.parts;
  if (total > (1ll << 22)) return ROAST_ERR_UNSUPPORTED;
  constexpr int smem = kWaves * kOwn + kTable * 4;
  static_assert(smem <= 160 * 1024 && kOwn * kWaves >= kWaves * 64 * 64 * 4, "LDS budget");
  static std::atomic<bool> configured{false};   // per instantiation; a race between host threads only repeats the call
  if (!configured.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_mm_ring<DX, NEG>), hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess) return ROAST_ERR_HIP;
    configured.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((k_mm_ring<DX, NEG>), dim3((unsigned)(cdiv(total, 8) * 8)), dim3(64 * kWaves), smem, s, p);
  return hip_status(hipGetLastError());
}

}  // namespace

bool ring_ok(int which, const MMArgs& a) {
  const int64_t K = which ? a.O : a.H, zk = which ? a.Z2 : a.Z1, zn = which ? a.Z1 : a.Z2;
  return a.hash.use_sign != 2 && a.Z1 % 32 == 0 && a.Z2 % 32 == 0 && a.H % 64 == 0 && a.O % 64 == 0 && a.m_size < (1ll << 28) &&
         a.I <= 65535 * 64 && cdiv(K, zk) * (cdiv(64, zn) + 1) <= kTable;   // (parts need no more)
}

// A and C 16-byte aligned, leading dimensions multiples of 8
roast_status ring_mm(int which, int parts, const MMArgs& a, const void* A, int64_t lda, const void* M_bf16, void* C, int64_t ldc, float* G, hipStream_t s) {
  if (lda >= (1ll << 23)) return ROAST_ERR_UNSUPPORTED;        // (32-bit byte offsets of 64 rows)
  RingArgs p{};
  p.a = a; p.th = make_tile_hash(a.hash, a.layer, a.nTx, a.nTy);
  p.A = (const uint16_t*)A; p.lda = lda; p.Mb = (const uint16_t*)M_bf16; p.mb_stride = shadow_stride(a.m_size); p.C = (uint16_t*)C; p.ldc = ldc;
  p.nbx = (int)((which ? a.H : a.O) / 64); p.nby = (int)cdiv(a.I, 64); p.parts = parts; p.G = parts > 1 ? G : nullptr;
  const bool neg = shadow_copies(a.m_size) == 4;
  if (which) return neg ? launch<true, true>(p, s) : launch<true, false>(p, s);
  return neg ? launch<false, true>(p, s) : launch<false, false>(p, s);
}

}  // namespace roast
