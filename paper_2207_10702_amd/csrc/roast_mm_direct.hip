// ROAST-MM for small calls on gfx950: forward Y = X*W and dX = dY*W^T (Algorithm 1 and Section 4.3 of arXiv
// 2207.10702) in one launch, on the matrix instruction of the operands' type, from operands as they lie in memory.
//
// What bounds a small call is latency: the larger kernels take a launch for the products and one to add up the parts of the
// contraction (fp32: and one to split the activations), 4-12 us each, for a microsecond of arithmetic.  Here a workgroup
// has one small output block and its eight waves share out the contraction, each with its own loads straight into
// the registers that the matrix instruction reads: no barrier and no LDS in the loop, one sum of eight at the end.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "roast_internal.hpp"

namespace roast {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

__device__ inline uint32_t pack_bf16x2(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 r = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, r);
}

// N floats that are only 4-byte aligned in memory (tile bases are arbitrary offsets into M)
template <int N>
struct __attribute__((packed, aligned(4))) Floats {
  float v[N];
};

constexpr int kWaves = 8;
constexpr int kTable = 2048;             // tile-table entries (8 bytes each) in LDS
constexpr int64_t kMaxBlocks = 0xffffffffll / (64 * kWaves) / 8 * 8;   // of a launch, whose threads are counted in 32 bits

struct DirectArgs {
  MMArgs a;
  TileHash th;
  const void* A;                         // FWD: X, DX: dY
  int64_t lda;
  const float* M;
  const uint16_t* Mb;                    // bf16: the copy of M, or null
  int64_t mb_stride;
  void* C;
  int64_t ldc;
  uint32_t mu1, mu2;                     // 2^32 / Z1, 2^32 / Z2, rounded up
  int nbx, nby;                          // column, row blocks
  int parts;                             // of the contraction (bf16: of 64 x 64 blocks alone), whose partial outputs go to G, [part][rows][columns]
  float* G;
  bool eighths;                          // (bf16, 64 x 64 blocks, no copy of M) how the blocks go to the XCDs, see direct_mm
};

template <typename V, typename T>
__device__ __forceinline__ V at(const T* base, uint32_t bytes) {
  return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) + bytes);
}

// q = n / z for n < 65536, z <= 65536
__device__ inline int quot(int n, uint32_t mu) { return (int)__umulhi((uint32_t)n, mu); }

// A 16 MI x 16 NJ output block.  Lane l = 16 g + r of a wave holds, of the 16 (bf16: 32) contraction indices of a unit, the KL = four
// (eight) KL g ..: of MI rows r of A, one 16-byte load each, and of the weights of NJ columns -- FWD: columns
// NJ r .. NJ r + NJ - 1, one load per contraction index; DX: columns r, 16 + r, ..., 16-byte loads along the contraction.
// fp32: matrix instruction s of a unit takes the indices 4 g + s.  bf16: one instruction a unit; the weights come from the copy of M (SH), or
// from fp32 M and are rounded in registers, which gives the same values and so the same sums; FWD packs them along the contraction.
template <typename T, bool SH, bool DX, int MI, int NJ>
__global__ __launch_bounds__(64 * kWaves, MI * NJ > 8 ? 2 : 4) void k_mm_direct(DirectArgs p) {
  constexpr bool BF = sizeof(T) == 2;
  constexpr int BM = 16 * MI, BN = 16 * NJ, KL = BF ? 8 : 4, KU = 4 * KL;
  constexpr int ROUNDS = BM * BN > 2048 ? 2 : 1, RI = MI / ROUNDS;   // of the sum over the waves: row fragments at a time
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int64_t* s_tab = reinterpret_cast<int64_t*>(smem);      // offset into M (SH: the copy of M) | sign << 63
  float* s_part = reinterpret_cast<float*>(smem);         // [wave][16 RI][BN], once the table is not needed any more
  const MMArgs& a = p.a;
  const T* A = static_cast<const T*>(p.A);
  const int K = DX ? (int)a.O : (int)a.H, N = DX ? (int)a.H : (int)a.O, I = (int)a.I;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  int bx, by, bz;
  if (BF && !SH && MI * NJ == 16 && p.eighths) {
    const int plane = p.nbx * p.nby, total = plane * p.parts, chunk = (total + 7) / 8, t = ((int)blockIdx.x & 7) * chunk + ((int)blockIdx.x >> 3);
    if (((int)blockIdx.x >> 3) >= chunk || t >= total) return;    // whole workgroup leaves before any barrier
    bz = t / plane;
    bx = (t - bz * plane) / p.nby;
    by = t - bz * plane - bx * p.nby;
  } else {
    const int plane = (int)(blockIdx.x / (unsigned)p.nbx);
    bx = (int)blockIdx.x - plane * p.nbx;
    bz = p.parts > 1 ? plane / p.nby : 0;
    by = plane - bz * p.nby;
  }
  const int m0 = by * BM, n0 = bx * BN;
  // (parts: of a contraction whose length is a multiple of 64, in whole 64s)
  const int u0 = p.parts > 1 ? 64 / KU * (K / 64 * bz / p.parts) : 0;
  const int units = p.parts > 1 ? 64 / KU * (K / 64 * (bz + 1) / p.parts) - u0 : (K + KU - 1) / KU;
  // a wave's share of them is contiguous: rows of A whose length is a power of two lie in the same few channels of the L2, and
  // waves that read next to one another would all ask those
  const int first = u0 + units * wave / kWaves, end = u0 + units * (wave + 1) / kWaves;
  // Addresses are a uniform base and a 32-bit offset in bytes: with 64-bit ones per lane the address arithmetic took
  // longer than the products.  Rows and columns beyond the problem repeat the last ones, they are not stored.
  const T* a_base = A + (int64_t)m0 * p.lda;
  uint32_t a_off[MI];
#pragma unroll
  for (int i = 0; i < MI; ++i) a_off[i] = (uint32_t)min(16 * i + r, I - 1 - m0) * (uint32_t)p.lda * (uint32_t)sizeof(T);
  // table: row = tile along the contraction, column = tile along the block's columns
  const int zk = DX ? a.Z2 : a.Z1, zn = DX ? a.Z1 : a.Z2;
  const uint32_t muk = DX ? p.mu2 : p.mu1, mun = DX ? p.mu1 : p.mu2;
  const int t0 = quot(u0 * KU, muk);     // first tile along the contraction
  const int c0 = quot(n0, mun), TN = quot(min(n0 + BN, N) - 1, mun) - c0 + 1;
  constexpr int NC = DX ? NJ : 1;        // columns (FWD: groups of NJ) a lane looks up
  int tc[NC];                            // its table column,
  uint32_t in[NC];                       // its place in its tile
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    const int col = DX ? min(n0 + 16 * j + r, N - 1) : min(n0 + NJ * r, N - NJ), t = quot(col, mun);
    tc[j] = t - c0;
    in[j] = (uint32_t)(col - t * zn) * (DX ? (uint32_t)a.Z2 : 1u);
  }
  using AVec = typename std::conditional<BF, uint4v, Floats<4>>::type;
  // a load of weights: WV of them, in WD dwords; loads of a unit
  constexpr int WV = DX ? (SH ? 8 : 4) : NJ, WD = SH ? WV / 2 : WV, WN = DX ? NJ * KL / WV : KL;
  struct Unit {
    AVec x[MI];
    Floats<WD> w[WN];
    uint32_t flip[NC];
  };
  auto load_x = [&](Unit& u, int kk) {
    const int k = min(KU * kk + KL * g, K - KL);
#pragma unroll
    for (int i = 0; i < MI; ++i) u.x[i] = at<AVec>(a_base, a_off[i] + (uint32_t)k * (uint32_t)sizeof(T));
  };
  auto load_w = [&](Unit& u, int kk) {
    const int k = min(KU * kk + KL * g, K - KL), t = quot(k, muk), kin = k - t * zk;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int64_t e = s_tab[(t - t0) * TN + tc[j]];
      u.flip[j] = (uint32_t)(e >> 32) & 0x80000000u;
      using W = typename std::conditional<SH, uint16_t, float>::type;
      const W* base;
      if constexpr (SH) base = p.Mb;
      else base = p.M;
      const uint32_t off = ((uint32_t)e + in[j] + (uint32_t)kin * (DX ? 1u : (uint32_t)a.Z2)) * (uint32_t)sizeof(W);
#pragma unroll
      for (int q = 0; q < (DX ? KL / WV : KL); ++q)
        u.w[DX ? j * (KL / WV) + q : q] = at<Floats<WD>>(base + (DX ? WV * q : q * a.Z2), off);
    }
  };
  // weight of column fragment j, contraction index s of the lane's
  auto weight = [&](const Unit& u, int j, int s) { return DX ? u.w[j * (KL / 4) + s / 4].v[s % 4] : u.w[s].v[j % WV]; };
  // (bf16) the two of contraction indices 2 d and 2 d + 1
  auto weights = [&](const Unit& u, int j, int d) -> uint32_t {
    if constexpr (!SH) return pack_bf16x2(weight(u, j, 2 * d), weight(u, j, 2 * d + 1));
    else if constexpr (DX) return __float_as_uint(u.w[j].v[d]);
    else return __builtin_amdgcn_perm(__float_as_uint(u.w[2 * d + 1].v[j / 2]), __float_as_uint(u.w[2 * d].v[j / 2]), j % 2 ? 0x07060302u : 0x05040100u);
  };
  Unit nxt;
  if (first < end) load_x(nxt, first);
  const int rows_k = quot(min((u0 + units) * KU, K) - 1, muk) + 1 - t0;
  for (int e = tid; e < rows_k * TN; e += 64 * kWaves) {
    const int row = e / TN, ek = t0 + row, en = c0 + e - row * TN;
    bool neg;
    const int64_t off = tile_place(a.hash, p.th, a.layer, (uint32_t)(DX ? en : ek), (uint32_t)(DX ? ek : en), &neg);
    // (an odd offset is read from the second copy, where it is dword-aligned: everything added to it is even)
    s_tab[e] = (SH && (off & 1) ? p.mb_stride + off - 1 : off) | (neg ? INT64_MIN : 0);
  }
  __syncthreads();
  // fp32: sums of at most 64 contraction indices, and of those: a chain of single adds over all of the wave's share
  // would be further from the exact product than the three-plane kernels (4096 indices: 4.1e-7 against 3.3e-7)
  floatx4 acc[MI][NJ], all[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = all[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  if (first < end) load_w(nxt, first);
#pragma unroll 1
  for (int kk = first, n = 1; kk < end; ++kk, ++n) {
    Unit u = nxt;
    if (kk + 1 < end) {
      load_x(nxt, kk + 1);
      load_w(nxt, kk + 1);
    }
    // a unit that the contraction does not fill: zeros on both sides (what was loaded there may be an infinity)
    const bool ragged = KU * (kk + 1) > K, cut = KU * kk + KL * g >= K;
    if constexpr (BF) {
      if (ragged && cut) {
#pragma unroll
        for (int i = 0; i < MI; ++i) u.x[i] = uint4v{0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const uint32_t flip = u.flip[DX ? j : 0] | (u.flip[DX ? j : 0] >> 16);
        uint4v w;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          w[d] = weights(u, j, d) ^ flip;
        }
        if (ragged) w = cut ? uint4v{0u, 0u, 0u, 0u} : w;
#pragma unroll
        for (int i = 0; i < MI; ++i)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, u.x[i]), __builtin_bit_cast(bf16x8, w), acc[i][j], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        float w[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          w[j] = __uint_as_float(__float_as_uint(weight(u, j, s)) ^ u.flip[DX ? j : 0]);
          if (cut) w[j] = 0.f;
        }
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          const float x = cut ? 0.f : u.x[i].v[s];
#pragma unroll
          for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, w[j], acc[i][j], 0, 0, 0);
        }
      }
      if ((n & 3) == 0 || kk + 1 >= end) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            all[i][j] += acc[i][j];
            acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
          }
      }
    }
  }
  // results[i][j][e]: row 16 i + 4 g + e, column NJ r + j (FWD) or 16 j + r (DX)
#pragma unroll
  for (int round = 0; round < ROUNDS; ++round) {
    __syncthreads();                     // the table, the sums of the round before have been read
    float* part = s_part + wave * (16 * RI * BN);
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          part[(16 * i + 4 * g + e) * BN + (DX ? 16 * j + r : NJ * r + j)] = BF ? acc[round * RI + i][j][e] : all[round * RI + i][j][e];
    __syncthreads();
    constexpr int V = BF ? 8 : 4;        // columns a thread adds up
    for (int q = tid; q < 16 * RI * BN / V; q += 64 * kWaves) {
      const int row = q / (BN / V), c = V * (q % (BN / V)), out_row = m0 + 16 * RI * round + row;
      if (out_row >= I || n0 + c >= N) continue;
      floatx4 sum[V / 4];
#pragma unroll
      for (int v = 0; v < V / 4; ++v) sum[v] = *reinterpret_cast<const floatx4*>(s_part + row * BN + c + 4 * v);
      for (int w = 1; w < kWaves; ++w)
#pragma unroll
        for (int v = 0; v < V / 4; ++v) sum[v] += *reinterpret_cast<const floatx4*>(s_part + w * (16 * RI * BN) + row * BN + c + 4 * v);
      if constexpr (!BF || MI * NJ == 16) {
        if (p.parts > 1) {
          float* part_to = p.G + ((int64_t)bz * I + out_row) * N + n0 + c;
#pragma unroll
          for (int v = 0; v < V / 4; ++v) *reinterpret_cast<floatx4*>(part_to + 4 * v) = a.lambda * sum[v];
          continue;
        }
      }
      T* to = static_cast<T*>(p.C) + (int64_t)out_row * p.ldc + n0 + c;
      if constexpr (BF) {
        uint4v out;
#pragma unroll
        for (int d = 0; d < 4; ++d) out[d] = pack_bf16x2(a.lambda * sum[d / 2][2 * (d & 1)], a.lambda * sum[d / 2][2 * (d & 1) + 1]);
        *reinterpret_cast<uint4v*>(to) = out;
      } else {
        Floats<4> out;
#pragma unroll
        for (int e = 0; e < 4; ++e) out.v[e] = a.lambda * sum[0][e];
        *reinterpret_cast<Floats<4>*>(to) = out;
      }
    }
  }
}

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

bool direct_ok(const MMArgs& a, bool bf16, bool dx, int bn) {
  const int64_t K = dx ? a.O : a.H, N = dx ? a.H : a.O, zk = dx ? a.Z2 : a.Z1, zn = dx ? a.Z1 : a.Z2;
  const int kl = bf16 ? 8 : 4;
  return a.hash.use_sign != 2 && zk % kl == 0 && (dx || zn % 4 == 0) && a.H % kl == 0 && a.O % kl == 0 && a.H < 65536 && a.O < 65536 &&
         a.Z1 >= 2 && a.Z1 <= 65536 && a.Z2 <= 65536 &&
         a.I <= 65535 * 64 &&                // (the generic kernels' limit)
         a.m_size < (1ll << 28) &&           // (32-bit byte offsets)
         (!bf16 || a.Z2 % 2 == 0) && cdiv(K, zk) * (cdiv(std::min<int64_t>(bn, N), zn) + 1) <= kTable;
}

struct Variant {
  bool bf16;
  int mi, nj;
  double fixed;                          // microseconds: a launch, a workgroup's start and end
  double alone[2], busy[2];              // nanoseconds a contraction index (forward, dX; 0: not built): where every CU has one workgroup, where more
};
constexpr Variant kVariants[] = {{false, 1, 1, 2.8, {3.15, 3.45}, {2.7, 3.1}},
                                 {false, 1, 2, 3.4, {4.1, 4.95}, {4.3, 5.0}},
                                 {false, 1, 4, 3.8, {6.6, 8.6}, {6.7, 8.7}},
                                 {false, 2, 2, 4.0, {6.15, 6.6}, {6.4, 6.7}},
                                 {false, 2, 4, 4.4, {10.7, 0.0}, {10.2, 0.0}},   // (dX: its registers leave a CU one workgroup)
                                 {true, 1, 2, 5.0, {2.34, 2.28}, {1.7, 2.45}},
                                 {true, 1, 4, 5.0, {3.05, 4.2}, {2.65, 4.1}},
                                 {true, 2, 4, 5.0, {3.55, 4.85}, {3.5, 4.85}},
                                 {true, 4, 4, 5.0, {5.5, 6.8}, {5.55, 7.05}}};

template <typename T, bool SH, bool DX, int MI, int NJ>
roast_status launch_one(const DirectArgs& p, hipStream_t s) {
  const int64_t blocks = (int64_t)p.nby * p.nbx * p.parts;   // (direct_plan: at most kMaxBlocks)
  constexpr size_t lds = std::max<size_t>((size_t)kTable * 8, (size_t)kWaves * std::min(16 * MI * 16 * NJ, 2048) * 4);
  static_assert(lds <= 64 * 1024, "LDS without an attribute");
  hipLaunchKernelGGL((k_mm_direct<T, SH, DX, MI, NJ>), dim3((unsigned)(p.eighths ? cdiv(blocks, 8) * 8 : blocks)), dim3(64 * kWaves), lds, s, p);
  return hip_status(hipGetLastError());
}

template <typename T, bool DX, int MI, int NJ>
roast_status launch(const DirectArgs& p, hipStream_t s) {
  if constexpr (sizeof(T) == 2)
    if (p.Mb) return launch_one<T, true, DX, MI, NJ>(p, s);
  return launch_one<T, false, DX, MI, NJ>(p, s);
}

template <bool DX>
roast_status launch_variant(bool bf16, int mi, int nj, const DirectArgs& p, hipStream_t s) {
  const int v = 10 * mi + nj;
  if (bf16) {
    if (v == 12) return launch<uint16_t, DX, 1, 2>(p, s);
    if (v == 14) return launch<uint16_t, DX, 1, 4>(p, s);
    if (v == 24) return launch<uint16_t, DX, 2, 4>(p, s);
    if (v == 44) return launch<uint16_t, DX, 4, 4>(p, s);
    return ROAST_ERR_UNSUPPORTED;
  }
  if (v == 11) return launch<float, DX, 1, 1>(p, s);
  if (v == 12) return launch<float, DX, 1, 2>(p, s);
  if (v == 14) return launch<float, DX, 1, 4>(p, s);
  if (v == 22) return launch<float, DX, 2, 2>(p, s);
  if constexpr (!DX)
    if (v == 24) return launch<float, DX, 2, 4>(p, s);
  return ROAST_ERR_UNSUPPORTED;
}

// the launch that adds up `parts` fp32 outputs of I x N
double finish_us(int parts, int64_t I, int64_t N) { return 2.5 + 0.12 * parts + (double)parts * (double)I * (double)N * 4.0 / 1.95e6; }

}  // namespace

// The block with the smallest modelled time.  The fp32 constants are fitted to 300 timed launches (most within 8 %) of 16 .. 1024 rows: up to two
// workgroups to a CU both run to the end; beyond that a CU takes the next as one ends.  Where M is larger than an XCD's L2 (4 MiB: 1 Mi slots) its
// share beyond that comes from the memory-side cache, in pieces of a tile's row: 6.5 TB/s, 3.5 where those are 64 or 128 bytes.
// An fp32 call with a workspace comes here where that is 8 % less than what the three-plane kernels are modelled to take: up to 1 GFLOP mostly, 4 at the few rows
// or columns that leave those idle.  Of 300 calls of 16 .. 2048 rows the worst loses 3 % by it.  64 x 256 x 256 17.9 -> 11.0 us of which the GPU is busy half,
// 885 x 576 x 384 26.5 -> 11.4, 512 x 1024 x 1024 32 -> 17, 46 x 3136 x 1728 31.6 -> 20.9, 39 x 7648 x 2496 over 1 Mi slots 48 -> 34, but over 4 Mi it stays (49, here 52 to 60), as
// does 2048 x 1024 x 1024.  Without one, against the generic kernel: 300 x 1096 x 520 162 -> 12.9.
// bf16, by the same margin on what the wide blocks are modelled to take: 206 x 1664 x 1152 17.0 -> 10.5, 512 x 2048 x 2048 without a copy of M 23.8 -> 17.2 (two
// launches; with one see roast_mm_ring.hip); without a workspace 35 x 4352 x 5504 43.7 -> 19.6.  A 64 x 64 block of bf16 takes 167 ns a unit of 32, 20 bytes a clock and CU:
// neither more units in flight nor fewer address instructions, whole lines of A or other channels of the L2 change that.
DirectPlan direct_plan(int which, bool bf16, const MMArgs& a, size_t room) {
  DirectPlan best{0, 0, 1, 1e300};
  const int64_t K = which ? a.O : a.H, N = which ? a.H : a.O, l2 = 1 << 20;
  auto search = [&](int max_parts) {
    for (const Variant& v : kVariants) {
      if (v.bf16 != bf16 || v.alone[which] == 0.0 || !direct_ok(a, bf16, which == 1, 16 * v.nj)) continue;
      const int64_t blocks = cdiv(a.I, 16 * v.mi) * cdiv(N, 16 * v.nj);
      for (int parts = 1; parts <= max_parts && blocks * parts <= kMaxBlocks; ++parts) {
        if (parts > 1 && (K < 128 * parts || blocks * parts > 768 || (size_t)parts * (size_t)a.I * (size_t)N * 4 > room)) break;
        const double r = (double)(blocks * parts) / 256.0;
        double rounds = 0.5 * (r + std::ceil(r)), us;
        if (!bf16 && r <= 2.0) rounds = 2.0;        // (some CUs have two workgroups from the start)
        us = v.fixed + 1e-3 * (double)K / parts * (r <= 1.0 ? v.alone[which] : v.busy[which] * rounds) + (bf16 ? 0.0 : 0.6 * std::max(0.0, std::ceil(r) - 2.0));
        if (!bf16 && a.m_size > l2) {               // weights from beyond the L2, once for each row of blocks
          const double bytes = (double)cdiv(a.I, 16 * v.mi) * (double)K * (double)N * 4.0 * (1.0 - (double)l2 / (double)a.m_size);
          us = std::max(us, v.fixed + bytes / (which || v.nj == 4 || a.Z2 <= 16 * v.nj ? 6.5e6 : 3.5e6));
        }
        if (parts > 1) us += 0.8 + finish_us(parts, a.I, N);
        if (us < best.us) best = {v.mi, v.nj, parts, us};
      }
    }
  };
  search(1);
  // fp32 with a workspace (whose planes leave room for the outputs of parts): parts of the contraction, where one workgroup to a block leaves half of the CUs idle or a row of A is
  // far longer than one of the output.  26 x 448 x 14400 dX 50.9 -> 16.3 us, 20 x 10560 x 704 33.7 -> 15.1, 36 x 320 x 4160 dX 17.5 -> 10.5, none of 140 random products slower.
  if (room > 0 && best.mi && a.H % 64 == 0 && a.O % 64 == 0 && a.Z1 % 32 == 0 && a.Z2 % 32 == 0 &&
      (cdiv(a.I, 16 * best.mi) * cdiv(N, 16 * best.nj) <= 128 || K >= 16 * N))
    search(kWideParts);
  return best;
}

// bf16 64 x 64 blocks in `parts` of the contraction, in microseconds: with a copy of M (roast_mm_ring.hip), a launch; a round of up to 256
// workgroups, whose start and end take 4 and a contraction index 2 ns, 3 where every CU has one, a quarter of the 2 more where a tile is wider than
// the block (its rows are pieces of 128 bytes at any multiple of four: two lines each); weights of an M beyond an XCD's L2, at 6.5 TB/s; the launch that
// adds up the parts.  Fitted to 1100 launches of 16 to 2048 rows, most within 12 %.  Without a copy (the kernel above) an index takes 5.2 ns, in dX 9.7.
static double ring_us(int which, int parts, const MMArgs& a, bool copy) {
  const double K = (double)(which ? a.O : a.H), N = (double)(which ? a.H : a.O), part = K / parts;
  const int64_t wgs = cdiv(a.I, 64) * ((which ? a.H : a.O) / 64) * parts, rest = wgs % 256;
  const double finish = parts == 1 ? 0.0 : finish_us(parts, a.I, (int64_t)N);
  if (!copy) return 5.0 + (double)cdiv(wgs, 256) * part * (which ? 9.7e-3 : 5.2e-3) + finish;
  const double index = 2.0e-3 * (a.Z2 >= 128 ? 1.25 : 1.0);
  double us = 1.3 + (double)(wgs / 256) * (4.05 + part * (index + 1.0e-3));
  if (rest) us += 4.05 + part * (index + 1.0e-3 * (double)rest / 256.0);
  if (a.m_size > (1 << 20)) us = std::max(us, 5.35 + 2.0 * K * N / 6.5e6);
  return us + finish;
}

// The best number of parts of those blocks for a call that takes copy_us, or nocopy_us without a copy of M, on other kernels: where a call with a copy is 8 % faster
// for it and one without, which has to give the same sums, no more than 10 % slower by the model.  Two rounds at most: in a third (60 products of
// 8500 to 12000 indices and 513 to 620 workgroups) calls without a copy took 1.04 to 1.43 times as long as on other kernels, those with one 0.76 to 1.30 times.
// Elsewhere, in draws of 16 to 2048 rows that take these blocks: 690 without a copy 1.18 times faster in the geometric mean, seven of them 5 to 11 % slower; 370 with one 1.40, two 8 and 11 %
// slower.  (mi == 0: none.)
DirectPlan ring_plan(int which, const MMArgs& a, int max_parts, double copy_us, double nocopy_us) {
  DirectPlan best{0, 0, 1, copy_us / 1.08};
  if (a.I > 2048 || !ring_ok(which, a) || !direct_ok(a, true, which == 1, 64)) return best;
  const int64_t K = which ? a.O : a.H, blocks = cdiv(a.I, 64) * ((which ? a.H : a.O) / 64);
  for (int parts = 1; parts <= max_parts && blocks * parts <= 512 && (parts == 1 || K >= 128 * parts); ++parts) {
    const double us = ring_us(which, parts, a, true);
    if (us < best.us && ring_us(which, parts, a, false) <= 1.1 * nocopy_us) best = {4, 4, parts, us};
  }
  return best;
}

// which: 0 forward, 1 dX.  bf16: A and C 16-byte aligned, leading dimensions multiples of 8
roast_status direct_mm(int which, bool bf16, const DirectPlan& d, const MMArgs& a, const void* A, int64_t lda, const float* M, const void* M_bf16, void* C, int64_t ldc,
                       float* G, hipStream_t s) {
  if (lda >= (1ll << 23)) return ROAST_ERR_UNSUPPORTED;       // (32-bit byte offsets of 64 rows)
  if (bf16 && M_bf16 && d.mi == 4 && d.nj == 4 && ring_ok(which, a)) return ring_mm(which, d.parts, a, A, lda, M_bf16, C, ldc, G, s);
  DirectArgs p{};
  p.a = a; p.th = make_tile_hash(a.hash, a.layer, a.nTx, a.nTy);
  p.A = A; p.lda = lda; p.M = M; p.Mb = (const uint16_t*)M_bf16; p.mb_stride = shadow_stride(a.m_size); p.C = C; p.ldc = ldc;
  auto mu = [](int64_t z) { return (uint32_t)(((1ull << 32) + (uint64_t)z - 1) / (uint64_t)z); };
  p.mu1 = mu(a.Z1); p.mu2 = mu(a.Z2);
  p.nbx = (int)cdiv(which ? a.H : a.O, 16 * d.nj); p.nby = (int)cdiv(a.I, 16 * d.mi); p.parts = d.parts; p.G = G;
  // Workgroups go to the 8 XCDs round-robin.  Blocks by rows, columns fastest, read the fp32 weights of an M beyond an XCD's L2 from the memory-side cache once for each row of
  // blocks: there XCD j takes the j-th eighth of the blocks, rows fastest, and they pass through its L2 once (184 x 6336 x 9024 over 9.6 Mi slots 155 -> 92 us, 173 x 7296 x 10880
  // over 2.1 Mi 143 -> 112).  For a smaller M that gains nothing and the divisions cost 0.3 us (6.5 and 6.8).
  p.eighths = bf16 && !M_bf16 && d.mi == 4 && d.nj == 4 && p.nby > 1 && a.m_size > (1 << 20);
  return which ? launch_variant<true>(bf16, d.mi, d.nj, p, s) : launch_variant<false>(bf16, d.mi, d.nj, p, s);
}

}  // namespace roast
