// Wide bf16 matrix-core kernels for ROAST-MM on gfx950: forward Y = X*W, dX = dY*W^T (weights from the
// bf16 shadow of M) and the products of dM = scatter(X^T*dY) -- Algorithm 1 and the Section 4.3
// gradients of arXiv 2207.10702 -- for shapes whose output fills the chip with 256-row blocks.
//
// What bounds them: the matrix pipe under its power limit.  With operands of all zeros the same code
// runs at 1.85-1.95 PFLOP/s, with N(0,1) values at 1.4-1.5 (8192 cubed).  Hence
//   - v_mfma_f32_16x16x32_bf16 rather than 32x32x16: half the accumulator traffic per product,
//     12 % faster on random data, and bit for bit the same sums (the instruction adds its two
//     16-deep halves one after the other);
//   - every operand goes from memory straight into LDS (global_load_lds, no registers, no ds_write).
//     An operand whose memory rows run along the contraction (X and dY of forward / dX, the weight
//     rows of dX) is read back with ds_read_b128; one whose rows run across it (the weight tile of
//     forward, X and dY of dM) with the transposing ds_read_b64_tr_b16.  Both are conflict-free: the
//     16-byte chunks of a row are XOR-permuted by the row number, on the source address of the load
//     (a direct load fills LDS linearly) and on the read;
//   - the hash sign costs little: the shadow of a small M holds -M too, and the sign picks the copy (NEG).  A large M
//     (and the fp32 planes), whose second set of copies would cost an update of M more than it saves here, takes an
//     XOR of the weight fragments, in the second half of the product slot before the fragment's first
//     use: 3 % on a 256 x 256 block, 4-8 % on the smaller ones (at the start of the slot that uses them, 6-9 %).
// One workgroup: 8 waves, a 256 x BN block (BN = 256: 2 x 4 waves of 128 x 64; BN = 128: 4 x 2 waves of
// 64 x 64; 128 rows: 2 x 4 waves of 64 x 48 or 64 x 32), two LDS stages of one 64-deep contraction step each.  A step is four phases per wave --
// (upper, lower half of its rows) x (first, second 32 of the step) -- and a phase a memory slot and a
// product slot.  The two waves of a SIMD run half a phase apart (the second four waves pass one
// barrier more at the start): while one issues LDS reads and loads, the other's products have the
// matrix pipe.  Fragments are read one phase ahead; a quarter of the A tile is loaded again as soon
// as its last read is over, so loads are four or five phases ahead of their use.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>

#include "roast_internal.hpp"

namespace roast {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));

enum { MODE_FWD = 0, MODE_DX = 1, MODE_DM = 2 };
constexpr int BK = 64;
constexpr int kTableDM = 1024;           // entries (8 bytes each) of dM's

struct WideArgs {
  MMArgs a;
  TileHash th;
  const uint16_t* A;   // FWD: X, DX: dY, DM: X
  int64_t lda;
  const uint16_t* B;   // DM: dY
  int64_t ldb;
  const uint16_t* Mb;  // FWD / DX: shadow of M: a copy, one shifted by one element at +mb_stride; NEG: both of -M from +2*mb_stride
  int64_t mb_stride;
  // X3 (fp32 operands as three bfloat16 planes): distance between the planes
  int64_t a_plane, b_plane, mb_plane;
  uint16_t* C;         // bf16 output
  float* C32;          // fp32 output (X3)
  int64_t ldc;
  float* G;            // FWD / DX: partial outputs of a split contraction [part][rows][columns]; DM: raw products
  float* dM;           // DM, atomic mode
  int nbx, nby, nbz;   // workgroups: columns, rows, parts of the contraction
  int nblk;            // consecutive column blocks per workgroup (a strip)
  bool runs;           // DM: adds over runs of slots (see the epilogue)
  int rows_per_split;
  int split_begin[kWideParts + 1];   // parts of unequal length (split_begin[1] > 0)
};

constexpr int vmcnt_only(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0f70; }

__device__ inline uint32_t pack_bf16x2(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 r = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, r);
}

// LDS reads of the product loop.  In assembly, because the compiler would make every LDS read wait for
// all direct-to-LDS loads in flight; the waits are placed by hand (lgkmcnt counts below), and the
// values are tied to them with empty asm statements.
template <int OFF>
__device__ __forceinline__ void lds_read16(uint4v& d, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF));
}
// Transposing read of an 8(k) x 16 block: lanes 4r .. 4r+3 of a group of 16 give the addresses of row r
// (k = r resp. 4 + r), lane c receives the eight k-values of column c.
template <int OFF, int OFF4>
__device__ __forceinline__ void lds_read16_t(uint4v& d, uint32_t addr) {
  uint2v lo, hi;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(addr), "n"(OFF));
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(addr), "n"(OFF4));
  d = uint4v{lo[0], lo[1], hi[0], hi[1]};
}
// the value is only used after this point (an LDS read that the hand-placed wait before it covers)
template <typename T>
__device__ __forceinline__ void tie(T& v) {
  asm volatile("" : "+v"(v));
}
__device__ __forceinline__ uint32_t lds_read4(uint32_t addr) {
  uint32_t d;
  asm volatile("ds_read_b32 %0, %1" : "=v"(d) : "v"(addr));
  return d;
}
// 16 bytes per lane from (uniform base) + (lane's byte offset) to LDS: lane l lands at lds + 16 * l
__device__ __forceinline__ void load_to_lds(const uint16_t* base, uint32_t bytes, uint32_t lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)((const char*)base + bytes),
                                   (__attribute__((address_space(3))) void*)(uintptr_t)lds, 16, 0, 0);
}

// the lane number, formed where it is needed instead of kept in a register across the product loop
__device__ __forceinline__ int lane_id() { return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>)
template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Workgroups go to the 8 XCDs round-robin; XCD j takes the j-th eighth of the block order, and inside it
// blocks are numbered in bands of four row blocks, rows fastest, so that the 32 workgroups an XCD runs
// at a time share 4 row slabs and 8 column slabs of the operands in its L2.
__device__ inline bool block_coords(const WideArgs& p, int* bx, int* by, int* bz) {
  const int plane = p.nbx * p.nby, total = plane * p.nbz;
  const int chunk = (total + 7) / 8;
  const int w = blockIdx.x;
  const int t = (w & 7) * chunk + (w >> 3);
  if ((w >> 3) >= chunk || t >= total) return false;
  *bz = t / plane;
  const int u = t - *bz * plane;
  const int band = u / (4 * p.nbx), r = u - band * 4 * p.nbx;
  const int rows = min(4, p.nby - 4 * band);
  *by = 4 * band + r % rows;
  *bx = r / rows;
  return true;
}

constexpr int lds_stages(int bm, int bn) { return bm == 128 || bn == 128 ? 3 : 2; }
constexpr int lds_operands(int bm, int bn) { return lds_stages(bm, bn) * (bm + bn) * BK * 2; }
// tile-table entries (4 bytes each) a forward / dX workgroup has room for in LDS
constexpr int table_entries(int bm, int bn) { return (160 * 1024 - lds_operands(bm, bn)) / 4; }

template <int MODE, int BM, int BN, bool X3, bool NEG>
__global__ __launch_bounds__(512, 2) void k_roast_mfma_wide(WideArgs p) {
  constexpr int WM = (BM == 256 && BN == 128) ? 4 : 2, WN = 8 / WM;
  constexpr int WTM = BM / WM, WTN = BN / WN;     // rows, columns of a wave
  constexpr int PH = WTM == 128 ? 4 : 2;          // phases of a step: (row halves) x (two k halves), or the k halves alone
  constexpr int NS = lds_stages(BM, BN);          // (PH == 4: 2, else 3)
  constexpr int RH = PH / 2;
  constexpr int AQ = BM / 64;                     // 64-row quarters of the A tile: one direct-to-LDS instruction per wave each
  constexpr int BI = BN / 64;                     // direct-to-LDS instructions per wave for the B tile
  constexpr int RQ = 64 / WM, SUB = RQ / 16;      // rows of a wave in a quarter, 16-row fragments of them
  constexpr int MI = WTM / 16 / RH, NJ = WTN / 16;   // 16-row / 16-column fragments of a phase
  constexpr bool TA = MODE == MODE_DM, TB = MODE != MODE_DX;   // operand rows run across the contraction
  constexpr bool ROWS = BN % 128 == 0;            // TB: LDS holds [k][BN] rows, else groups of 64 columns, [group][k][64]
  constexpr bool HASHED = MODE != MODE_DM;
  constexpr bool XSIGN = HASHED && !NEG;          // signs by XOR
  constexpr bool STRIPS = HASHED && !X3 && BN == 192;  // (256 x 256 blocks and fp32 planes have steps enough, a third copy of the step would not fit the registers; strips of 128 columns lost to those of 192 on all of 300 000 shapes)
  constexpr int A_BYTES = BM * 128, STAGE = A_BYTES + BN * 128;

  extern __shared__ __attribute__((aligned(1024))) char smem[];
  uint32_t* s_tab = reinterpret_cast<uint32_t*>(smem + NS * STAGE);     // tile table: offset into the shadow | sign << 31
  int64_t* s_dm = reinterpret_cast<int64_t*>(smem + NS * STAGE);        // dM: offset into M | sign << 63

  const MMArgs& a = p.a;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  int bx, by, bz;
  if (!block_coords(p, &bx, &by, &bz)) return;    // whole workgroup leaves before any barrier
  const int NB = STRIPS ? max(p.nblk, 1) : 1;     // column blocks of this workgroup's strip
  const int m0 = by * BM, n0 = bx * BN * NB;      // n0: first column of the strip
  const int I = (int)a.I;
  const int Mdim = MODE == MODE_DM ? (int)a.H : I;
  const int Ndim = MODE == MODE_DX ? (int)a.H : (int)a.O;
  int k_begin = 0, k_end = MODE == MODE_FWD ? (int)a.H : (MODE == MODE_DX ? (int)a.O : I);
  if (p.nbz > 1) {
    if (p.split_begin[1] > 0) {
      k_begin = p.split_begin[bz];
      k_end = p.split_begin[bz + 1];
    } else {
      k_begin = bz * p.rows_per_split;
      k_end = min(k_end, k_begin + p.rows_per_split);
    }
  }
  const int KQ = max((k_end - k_begin + BK - 1) / BK, 0);
  // A strip runs its blocks back to back as one sequence of steps: the loads never drain between two blocks.
  const int KT = X3 ? 6 * KQ : NB * KQ;           // steps
  const uint32_t sbase = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem);
  // hash tiles of the block: TN along the columns (dM: set below), x0 / y0 the first ones
  int TN = 1, y0 = 0, x0 = 0;
  if constexpr (MODE == MODE_FWD) { y0 = n0 / a.Z2; TN = (min(n0 + BN * NB, (int)a.O) - 1) / a.Z2 - y0 + 1; x0 = k_begin / a.Z1; }
  if constexpr (MODE == MODE_DX) { x0 = n0 / a.Z1; TN = (min(n0 + BN * NB, (int)a.H) - 1) / a.Z1 - x0 + 1; y0 = k_begin / a.Z2; }
  const int kt0 = MODE == MODE_FWD ? x0 : y0;
  const int row_bytes = 4 * TN;
  // Where a step stands in the contraction: its first index k, the table row of its hash tile (in bytes) and
  // the place inside the tile.  Kept as running uniform values, one step after the other,
  // so that the product loop divides nothing.  X3: step 6*kq + pair multiplies plane asel of A by plane
  // bsel of B.
  const int zk = HASHED ? (MODE == MODE_FWD ? a.Z1 : a.Z2) : BK;   // tile extent along the contraction (hashed: a multiple of 32)
  struct Pos {
    int k, row, in, pair, col;                     // col: the block's shift in the table (bytes)
  };
  const int in0 = HASHED ? k_begin - (MODE == MODE_FWD ? x0 : y0) * zk : 0;
  const int col_bytes = HASHED ? 4 * (BN / (MODE == MODE_FWD ? a.Z2 : a.Z1)) : 0;   // (strips: whole tiles per block)
  auto advance = [&](Pos& s) {
    if constexpr (X3) {
      if (++s.pair < 6) return;
      s.pair = 0;
    }
    s.k += BK;
    s.in += BK;
    if (s.in >= zk) { s.in -= zk; s.row += row_bytes; }
    if (s.in >= zk) { s.in -= zk; s.row += row_bytes; }
    if (STRIPS && s.k >= k_end) {                  // on to the next block of the strip
      s.k = k_begin;
      s.in = in0;
      s.col += col_bytes;
      s.row = s.col;
    }
  };
  auto asel = [&](const Pos& s) -> int64_t { return X3 ? (int64_t)((0x120100 >> (4 * s.pair)) & 3) : 0; };
  auto bsel = [&](const Pos& s) -> int64_t { return X3 ? (int64_t)((0x102010 >> (4 * s.pair)) & 3) : 0; };

  // Addresses are a uniform base plus a 32-bit offset per lane.  What a load of the product loop needs is
  // formed in a product slot before (prep_*), in the shadow of the matrix instructions: every vector,
  // scalar or branch instruction in a memory slot lengthens it (with the address arithmetic and two
  // uniform branches there the 256 x 256 forward ran at 1170 TFLOP/s, without at 1350).
  // ---- A tile.  Quarter q = 64 output rows, 8 KiB of LDS, one instruction per wave: [row][64 k] with the
  // wave's 8 rows, or (TA) [k][64 rows] with the wave's 8 k-rows.  Lane: row (k-row) lane >> 3, chunk a_ch.
  const int lr = lane >> 3;
  // ... of rows along the contraction: one ds_read_b128 takes 16 rows by 4 chunks, 16 lanes a clock, of which
  // half are rows 0-3 and 12-15 at one chunk and half rows 4-11 at the next (or the other way round).  With
  // row ^ (row >> 3) each such clock met every bank twice: 4 clocks more per read, a third to a half of the
  // LDS's busy time (SQ_LDS_BANK_CONFLICT 12288 of 30388 clocks per CU, 8192x768x3072); with this, none.
  // (The products hide most of it: 512x2048x2048 18.77 -> 18.68 us, 16384x4096x16384 1674 -> 1667, 8192x768x3072 40.1 -> 40.2.)
  auto swzRow = [](int r) { return (r >> 1) & 7; };
  auto swz64 = [](int k) { return ((k >> 1) & 1) | (((k >> 3) & 1) << 1); };        // 32-byte chunk permutation of 128-byte k-rows
  auto swzBN = [](int k) { return (k & 3) | (((k >> 3) & 1) << 2); };               // ... of k-rows of 256 bytes and more
  const int a_ch = TA ? ((lane & 7) ^ (2 * swz64(8 * wave + lr))) : ((lane & 7) ^ swzRow(8 * wave + lr));
  // constant part of the lane's offset: !TA: its row (rows beyond the last one repeat it, they are not
  // stored); TA: its columns (clamped likewise)
  uint32_t a_fix[AQ];
  const uint16_t* a_base[AQ];
#pragma unroll
  for (int q = 0; q < AQ; ++q) {
    if constexpr (!TA) {
      const int rb = min(m0 + 64 * q + 8 * wave, I - 1);
      a_base[q] = p.A + (int64_t)rb * p.lda;
      a_fix[q] = (uint32_t)min(lr, I - 1 - rb) * ((uint32_t)p.lda * 2u);
    } else {
      a_base[q] = p.A;
      a_fix[q] = 2u * (uint32_t)min(m0 + 64 * q + 8 * a_ch, (int)a.H - 8);
    }
  }
  // of a step: the part of the offset that moves with it, and (TA) the first row of the step
  struct AStep {
    uint32_t off;
    int64_t base;
  };
  auto prep_a = [&](const Pos& s) {
    AStep r;
    const int64_t pl = X3 ? asel(s) * p.a_plane : 0;
    if constexpr (!TA) {
      // pieces beyond a ragged contraction length come from the start of the row (and are zeroed, see cut)
      const int kc = s.k + 8 * a_ch;
      r.off = kc < k_end ? 2u * (uint32_t)kc : 0u;
      r.base = pl;
    } else {
      r.off = __umul24((uint32_t)min(8 * wave + lr, I - 1 - s.k), (uint32_t)p.lda * 2u);
      r.base = pl + (int64_t)s.k * p.lda;
    }
    return r;
  };
  auto load_a = [&](const AStep& s, uint32_t stage, auto Q) {
    constexpr int q = decltype(Q)::value & (AQ - 1);
    load_to_lds(a_base[q] + s.base, a_fix[q] + s.off, sbase + stage + q * 8192 + wave * 1024);
  };

  // ---- B tile: BN * 128 bytes, BI instructions per wave
  //   DX            : [row h][64 k]: instruction u = rows 8*(wave*BI + u) ..; lane: row lane >> 3, chunk of the step
  //   FWD / DM, rows: [k][BN]: a wave's instructions cover k-rows 8*wave .. +7, RPI each; lane: k-row lane / CPR, chunk of the row
  //   FWD / DM, else: [group][k][64]: instruction u = group u, k-rows 8*wave .. +7; lane: k-row lane >> 3, chunk of the group
  constexpr int CPR = ROWS ? BN / 8 : 8, RPI = ROWS ? 512 / BN : 0;
  constexpr int BV = (TB && !ROWS) ? 1 : (BI < 2 ? BI : 2);     // the chunk permutation depends on the parity of u at most
  int b_n[BV];                                     // TB: first column of the lane's chunk (!ROWS: inside its group); DX: contraction index of it in the step
#pragma unroll
  for (int v = 0; v < BV; ++v) {
    if constexpr (TB && ROWS) b_n[v] = min(n0 + 8 * ((lane % CPR) ^ (2 * swzBN(8 * wave + v * RPI + lane / CPR))), Ndim - 8);
    else if constexpr (TB) b_n[v] = 8 * ((lane & 7) ^ (2 * swz64(8 * wave + lr)));
    else b_n[v] = 8 * ((lane & 7) ^ swzRow(8 * (wave * BI + v) + lr));
  }
  const uint32_t tab = sbase + NS * STAGE;
  // FWD: table column and offset inside the tile, in bytes, of the lane's chunk
  constexpr int BF = MODE == MODE_FWD ? (ROWS ? BV : BI) : 1;
  uint32_t b_tab[BF], b_in[BF];
  if constexpr (MODE == MODE_FWD) {
#pragma unroll
    for (int v = 0; v < BF; ++v) {
      const int n = ROWS ? b_n[v < BV ? v : 0] : min(n0 + 64 * v + b_n[0], Ndim - 8);
      b_tab[v] = tab + 4 * (n / a.Z2 - y0);
      b_in[v] = 2 * (n % a.Z2 + a.Z2 * (lane / CPR));
    }
  }
  // DX: a wave's rows (8 per instruction) are 16 or 32 aligned ones, in one hash tile, unless the block is 192 wide
  constexpr bool ONE_TILE = BI != 3;
  constexpr int BE = MODE == MODE_FWD ? BF : (MODE == MODE_DX ? (ONE_TILE ? BV : BI) : 1);   // table entries a lane needs per step
  // DX: first row of the wave's (ONE_TILE: beyond the problem, any row of the last tile will do; rows of a tile
  // beyond the problem are inside M), of instruction u else
  const int dx0 = n0 + 8 * wave * BI;
  const int dx_x = min(dx0, (int)a.H - 1) / a.Z1, dx_in = dx0 < (int)a.H ? dx0 - dx_x * a.Z1 : 0;
  auto dx_row = [&](int u) { return min(dx0 + 8 * u, (int)a.H - 8); };
  // the table entries of a step: their addresses (prepared), the reads
  struct EStep {
    uint32_t at[BE];
  };
  auto prep_entries = [&](const Pos& s) {
    EStep r;
    if constexpr (MODE == MODE_FWD) {
      const int n = s.in + min(8 * wave, k_end - 8 - s.k);       // the wave's 8 k-rows lie in one tile
      const uint32_t row = (uint32_t)(s.row + (n >= zk ? row_bytes : 0));
#pragma unroll
      for (int v = 0; v < BE; ++v) r.at[v] = b_tab[v] + row;
    } else if constexpr (MODE == MODE_DX) {
      const uint32_t row = tab + (uint32_t)s.row;
#pragma unroll
      for (int u = 0; u < BE; ++u) {
        const int n = s.in + min(b_n[BV > 1 ? u & 1 : 0], k_end - 8 - s.k);
        r.at[u] = (n >= zk ? row + (uint32_t)row_bytes : row) + 4u * (uint32_t)((ONE_TILE ? dx_x : dx_row(u) / a.Z1) - x0);
      }
    }
    return r;
  };
  auto read_entries = [&](const EStep& s, uint32_t* ent) {
    if constexpr (HASHED) {
#pragma unroll
      for (int u = 0; u < BE; ++u) ent[u] = lds_read4(s.at[u]);
    }
  };
  struct BStep {
    uint32_t off[BI];
    const uint16_t* base;
  };
  auto prep_b = [&](const Pos& s, const uint32_t* ent) {
    BStep r;
    r.base = MODE == MODE_DM ? p.B + (X3 ? bsel(s) * p.b_plane : 0) + (int64_t)s.k * p.ldb : p.Mb + (X3 ? bsel(s) * p.mb_plane : 0);
    if constexpr (MODE == MODE_FWD) {
      int n = s.in + min(8 * wave, k_end - 8 - s.k);
      n = n >= zk ? n - zk : n;
#pragma unroll
      for (int u = 0; u < BI; ++u) {
        const int f = ROWS ? (BV > 1 ? u & 1 : 0) : u;
        r.off[u] = 2u * ent[f] + b_in[f] + (uint32_t)(2 * a.Z2 * (n + u * RPI));
      }
    } else if constexpr (MODE == MODE_DX) {
#pragma unroll
      for (int u = 0; u < BI; ++u) {
        int n = s.in + min(b_n[BV > 1 ? u & 1 : 0], k_end - 8 - s.k);
        n = n >= zk ? n - zk : n;
        const int row = ONE_TILE ? dx_in + 8 * u : dx_row(u) % a.Z1;
        r.off[u] = 2u * (ent[ONE_TILE && BV > 1 ? u & 1 : ONE_TILE ? 0 : u] + (uint32_t)(n + a.Z2 * lr)) + (uint32_t)(2 * a.Z2 * row);
      }
    } else {
#pragma unroll
      for (int u = 0; u < BI; ++u) {
        const int n = ROWS ? b_n[BV > 1 ? u & 1 : 0] : min(n0 + 64 * u + b_n[0], Ndim - 8);
        r.off[u] = __umul24((uint32_t)min(8 * wave + u * RPI + lane / CPR, I - 1 - s.k), (uint32_t)p.ldb * 2u) + 2u * (uint32_t)n;
      }
    }
    return r;
  };
  auto load_b = [&](const BStep& s, uint32_t stage, auto U) {
    constexpr int u = decltype(U)::value;
    load_to_lds(s.base, s.off[u], sbase + stage + A_BYTES + ((TB && !ROWS) ? u * 8192 + wave * 1024 : (wave * BI + u) * 1024));
  };

  // ---- prologue: A tiles are on their way while the tile table is hashed
  Pos p0{k_begin, 0, in0, 0, 0}, p1 = p0, p2;   // of steps t, t + 1, t + 2
  if (KT > 1) advance(p1);
  p2 = p1;
  if (KT > 2) advance(p2);
  if (KT > 0) {
    const AStep s0 = prep_a(p0), s1 = prep_a(p1);
    static_for<AQ>([&](auto Q) { load_a(s0, 0, Q); });
    static_for<(PH == 4 ? 2 : AQ)>([&](auto Q) { load_a(s1, STAGE, Q); });
  }
  if constexpr (HASHED) {
    const int nk = (max(k_end, k_begin + 1) - 1) / zk - kt0 + 1;
    for (int e = tid; e < nk * TN; e += 512) {
      const int ek = e / TN, en = e - ek * TN;
      bool neg;
      const int64_t off = tile_place(a.hash, p.th, a.layer, (uint32_t)(MODE == MODE_FWD ? x0 + ek : x0 + en),
                                     (uint32_t)(MODE == MODE_FWD ? y0 + en : y0 + ek), &neg);
      // an odd base is read from the second copy, where it is dword-aligned (everything added to it is even)
      const uint32_t o32 = (uint32_t)((off & 1) ? p.mb_stride + off - 1 : off);
      // (XSIGN: doubling an entry, to a byte offset, drops the sign)
      s_tab[e] = XSIGN ? o32 | (neg ? 0x80000000u : 0u) : o32 + (neg ? 2u * (uint32_t)p.mb_stride : 0u);
    }
  }
  if constexpr (MODE == MODE_DM) {
    if (p.G == nullptr) {
      x0 = m0 / a.Z1;
      y0 = n0 / a.Z2;
      TN = (min(n0 + BN, (int)a.O) - 1) / a.Z2 - y0 + 1;
      const int cnt = ((min(m0 + BM, (int)a.H) - 1) / a.Z1 - x0 + 1) * TN;
      for (int e = tid; e < cnt; e += 512) {
        bool neg;
        const int64_t off = tile_place(a.hash, p.th, a.layer, (uint32_t)(x0 + e / TN), (uint32_t)(y0 + e % TN), &neg);
        s_dm[e] = off | (neg ? INT64_MIN : 0);
      }
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  if (KT > 0) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      uint32_t ent[BE];
      if constexpr (HASHED) {
        read_entries(prep_entries(s == 0 ? p0 : p1), ent);
        asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
        for (int u = 0; u < BE; ++u) tie(ent[u]);
      }
      const BStep bs = prep_b(s == 0 ? p0 : p1, ent);
      static_for<BI>([&](auto U) { load_b(bs, s * STAGE, U); });
    }
  }

  // ---- fragments
  floatx4 acc[RH * MI][NJ];
#pragma unroll
  for (int i = 0; i < RH * MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  // k-contiguous operand: lane reads 8 k of row lane & 15, chunk (lane >> 4) + 4*ks; transposed: see lds_read16_t
  const uint32_t l_row = (uint32_t)swzRow(lane);
  const int tk = 8 * (lane >> 4) + ((lane & 15) >> 2);
  constexpr int AR = TA ? SUB : 2, BR = TB ? NJ : 2;
  uint32_t a_rd[AR], b_rd[BR];                     // by sub-row fragment / column fragment, or by k half
  if constexpr (!TA) {
    a_rd[0] = sbase + (wm * RQ + (lane & 15)) * 128 + ((((lane >> 4) ^ l_row) & 7) << 4);
    a_rd[1] = a_rd[0] ^ 64u;
  } else {
#pragma unroll
    for (int i = 0; i < SUB; ++i) a_rd[i] = sbase + tk * 128 + (((wm * SUB + i) ^ swz64(tk)) << 5) + (lane & 3) * 8;
  }
  if constexpr (!TB) {
    b_rd[0] = sbase + A_BYTES + (wn * WTN + (lane & 15)) * 128 + ((((lane >> 4) ^ l_row) & 7) << 4);
    b_rd[1] = b_rd[0] ^ 64u;
  } else
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int c = wn * NJ + j;                   // 16-column fragment of the block
      b_rd[j] = sbase + A_BYTES + (lane & 3) * 8 +
                (ROWS ? tk * (BN * 2) + ((c ^ swzBN(tk)) << 5) : (c >> 2) * 8192 + tk * 128 + (((c & 3) ^ swz64(tk)) << 5));
    }
  constexpr int KROW = ROWS ? BN * 2 : 128;        // TB: bytes between k-rows
  uint4v af[2][MI], bf[2][NJ];                     // A: [phase & 1]; B: [ks]
  constexpr int LA = (TA ? 2 : 1) * MI, LB = (TB ? 2 : 1) * NJ;   // LDS instructions of a phase
  constexpr int LAB = LA + LB < 15 ? LA + LB : 15;
  // (the fragment addresses move on to another stage by addition)
  auto to_stage = [&](int delta) {
#pragma unroll
    for (int i = 0; i < AR; ++i) a_rd[i] += (uint32_t)delta;
#pragma unroll
    for (int j = 0; j < BR; ++j) b_rd[j] += (uint32_t)delta;
  };
  // A fragments of phase P: row half P >> 1 (PH == 4), k half P & 1
  auto read_a = [&](auto P) {
    constexpr int ph = decltype(P)::value, ks = ph & 1;
    static_for<MI>([&](auto N) {
      constexpr int f = (ph >> 1) * MI + decltype(N)::value, q = f / SUB, sub = f % SUB;
      if constexpr (!TA) lds_read16<q * 8192 + sub * 2048>(af[ph & 1][decltype(N)::value], a_rd[ks]);
      else lds_read16_t<q * 8192 + ks * 4096, q * 8192 + ks * 4096 + 512>(af[ph & 1][decltype(N)::value], a_rd[sub]);
    });
  };
  auto read_b = [&](auto KS) {
    constexpr int ks = decltype(KS)::value;
    static_for<NJ>([&](auto N) {
      constexpr int j = decltype(N)::value;
      if constexpr (!TB) lds_read16<j * 2048>(bf[ks][j], b_rd[ks]);
      else lds_read16_t<ks * 32 * KROW, (ks * 32 + 4) * KROW>(bf[ks][j], b_rd[j]);
    });
  };
  auto tie_a = [&](auto S) {
#pragma unroll
    for (int i = 0; i < MI; ++i) tie(af[decltype(S)::value][i]);
  };
  auto tie_b = [&](auto S) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) tie(bf[decltype(S)::value][j]);
  };
  // Signs of a step: one per k half and FR 16-column fragments of the wave (a 32 x 32 block of W lies in one
  // hash tile); lane 2*g + half looks up the tile of group g, and a comparison makes one bit of each.
  constexpr int FR = WTN % 32 == 0 ? 2 : 1, NG = NJ / FR;
  uint32_t sgn = 0u, sgn_ent = 0u;                 // bit 2*g + half
  const int sg_lane = min(lane, 2 * NG - 1);
  uint32_t sg_col = 0u;
  if constexpr (XSIGN) {
    const int c = min(n0 + wn * WTN + 16 * FR * (sg_lane >> 1), Ndim - 1);
    sg_col = tab + 4 * (MODE == MODE_FWD ? c / a.Z2 - y0 : c / a.Z1 - x0);
  }
  auto prep_signs = [&](const Pos& s) -> uint32_t {
    if constexpr (!XSIGN) return 0u;
    const int n = s.in + min(32 * (lane_id() & 1), k_end - 1 - s.k);
    return sg_col + (uint32_t)(s.row + (n >= zk ? row_bytes : 0));
  };
  auto read_signs = [&](uint32_t at) {
    if constexpr (XSIGN) sgn_ent = lds_read4(at);
  };
  auto take_signs = [&] {
    if constexpr (XSIGN) {
      tie(sgn_ent);
      sgn = (uint32_t)__builtin_amdgcn_ballot_w64((int)sgn_ent < 0);
    }
  };
  auto put_signs = [&](auto KS) {
    constexpr int ks = decltype(KS)::value;
    if constexpr (XSIGN) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const uint32_t mask = (uint32_t)((int)(sgn << (31 - (2 * (j / FR) + ks))) >> 31) & 0x80008000u;
        bf[ks][j] ^= mask;
      }
    }
  };
  // the last step of a contraction length that is not a multiple of 64: zeros, in the fragments of both operands, since
  // what was loaded there (the start of the row, the last token again) may be an infinity, which times a zero would
  // be a NaN that the sum does not have (fp32 planes: the weights' alone, an infinity makes a NaN in any case, of its
  // zero planes)
  constexpr bool CUT_A = MODE == MODE_DM || !X3;
  auto cut = [&](auto KIND, auto KS) {
    constexpr int ks = decltype(KS)::value;
    if constexpr (decltype(KIND)::value < 2) return;   // (LAST, TAIL)
    const int rem = k_end - p0.k;                  // contraction indices left from the start of this step
    if (rem < BK) {
      const int cnt = rem - (32 * ks + 8 * (lane_id() >> 4));
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const uint32_t keep = cnt >= 2 * d + 2 ? 0xffffffffu : (cnt == 2 * d + 1 ? 0x0000ffffu : 0u);
#pragma unroll
        for (int j = 0; j < NJ; ++j) bf[ks][j][d] &= keep;
        if constexpr (CUT_A) {
#pragma unroll
          for (int i = 0; i < MI; ++i) af[ks][i][d] &= keep;
        }
      }
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;
  // Products of a phase, and in the shadow of the matrix instructions (16 clocks each, of which issuing
  // takes 4) whatever `prep` forms for the memory slots to come and, in the second half, the signs of the weight fragments that
  // were read in the memory slot before and are used next: SIGN = 1: k half 1 of this step, 0: k half 0 of the next,
  // 2: none.
  auto products = [&](auto P, auto SIGN, auto&& prep) {
    constexpr int ph = decltype(P)::value, ks = ph & 1, sg = XSIGN ? decltype(SIGN)::value : 2;
    constexpr int SPLIT = sg == 2 ? MI * NJ : MI * NJ / 2;
    auto product = [&](auto N) {
      constexpr int i = decltype(N)::value / NJ, j = decltype(N)::value % NJ;
      // weight (dM: dY) fragment first: a lane then holds 4 consecutive output columns of one output row
      acc[(ph >> 1) * MI + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          __builtin_bit_cast(bf16x8, bf[ks][j]), __builtin_bit_cast(bf16x8, af[ph & 1][i]), acc[(ph >> 1) * MI + i][j], 0, 0, 0);
    };
    // one matrix instruction, up to three others, and so on
    auto interleave = [&](auto COUNT) {
      static_for<decltype(COUNT)::value>([&](auto) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x6, 3, 0);
      });
      __builtin_amdgcn_sched_barrier(0);
    };
    __builtin_amdgcn_sched_barrier(0);
    prep();
    static_for<SPLIT>(product);
    interleave(std::integral_constant<int, SPLIT>{});
    if constexpr (sg != 2) {
      asm volatile("s_waitcnt lgkmcnt(0)");
      tie_b(std::integral_constant<int, sg>{});
      if constexpr (sg == 0) take_signs();
      put_signs(std::integral_constant<int, sg>{});
      static_for<MI * NJ - SPLIT>([&](auto N) { product(std::integral_constant<int, SPLIT + decltype(N)::value>{}); });
      interleave(std::integral_constant<int, MI * NJ - SPLIT>{});
    }
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  uint32_t ent[BE];
  auto tie_entries = [&] {
    if constexpr (HASHED) {
#pragma unroll
      for (int u = 0; u < BE; ++u) tie(ent[u]);
    }
  };
  // ---- results.  acc[f][j][e]: row 64*(f / SUB) + RQ*wm + 16*(f % SUB) + (lane & 15), column
  // WTN*wn + 16*j + 4*(lane >> 4) + e.  bf16: two fragments next to one another (columns j, j+1, or, for the
  // last of an odd number, rows f, f+1) exchange 16-lane rows so that a lane holds 8 consecutive columns, and
  // leave the registers in 16-byte stores, no LDS and no barrier involved.
  auto frag_row = [&](int f) { return m0 + 64 * (f / SUB) + RQ * wm + 16 * (f % SUB); };
  constexpr int NST = RH * MI * NJ / 2;            // store instructions of a bf16 block
  auto store_bf16 = [&](int cb, auto STRIP) {      // cb: first column of the wave
    const int l = lane_id(), g = l >> 4;
    auto pair_out = [&](auto& x, auto& y, int f0, int c0, int f1, int c1) {
      // x, y: 4 columns per lane of fragments (f0, c0), (f1, c1); 16-lane rows 1 / 0 and 3 / 2 change places
      uint2v a0 = {pack_bf16x2(a.lambda * x[0], a.lambda * x[1]), pack_bf16x2(a.lambda * x[2], a.lambda * x[3])};
      uint2v a1 = {pack_bf16x2(a.lambda * y[0], a.lambda * y[1]), pack_bf16x2(a.lambda * y[2], a.lambda * y[3])};
      const auto r0 = __builtin_amdgcn_permlane16_swap(a0[0], a1[0], false, false);
      const auto r1 = __builtin_amdgcn_permlane16_swap(a0[1], a1[1], false, false);
      const uint4v v = {r0[0], r1[0], r0[1], r1[1]};
      const int row = ((g & 1) ? frag_row(f1) : frag_row(f0)) + (l & 15), col = cb + ((g & 1) ? c1 : c0) + 8 * (g >> 1);
      if constexpr (decltype(STRIP)::value) {
        // every wave has to issue every store, the waits of the next step count them.  Columns are whole; a
        // row beyond the last one holds what the last one does (its operand rows were the same).
        *reinterpret_cast<uint4v*>(p.C + (int64_t)min(row, Mdim - 1) * p.ldc + col) = v;
      } else {
        if (row < Mdim && col < Ndim) *reinterpret_cast<uint4v*>(p.C + (int64_t)row * p.ldc + col) = v;
      }
    };
#pragma unroll
    for (int f = 0; f < RH * MI; ++f) {
#pragma unroll
      for (int j = 0; j + 1 < NJ; j += 2) pair_out(acc[f][j], acc[f][j + 1], f, 16 * j, f, 16 * j + 16);
      if (NJ % 2 == 1 && f % 2 == 1) pair_out(acc[f - 1][NJ - 1], acc[f][NJ - 1], f - 1, 16 * (NJ - 1), f, 16 * (NJ - 1));
    }
  };
  // The kinds of step: FIRST after a block of a strip has been stored (its stores are younger than loads in
  // flight: the waits have to allow for them), LAST of all (nothing is read or loaded ahead, and it alone can be cut
  // short; X3: and the five pairs before it, TAIL), or none of these.
  enum { MID = 0, FIRST = 1, LAST = 2, TAIL = 3 };
  auto wait_loads = [&](auto KIND, auto N) {
    constexpr int n = decltype(N)::value + (decltype(KIND)::value == FIRST ? NST : 0);
    static_assert(n < 64, "vmcnt has six bits");
    __builtin_amdgcn_s_waitcnt(vmcnt_only(n));
  };
  AStep a1, a2;                                    // of the step whose A tile is being loaded
  BStep b2;
  EStep e2;
  uint32_t sg_at = 0u;
  // A step of four phases, two stages.  Order of the loads (per wave): A quarters 2, 3 of step t+1 in phases
  // 0, 1; A quarters 0, 1 and the B tile of step t+2 in phases 2, 3 -- each after the last read of what it
  // overwrites has completed in every wave (reads of a phase are waited for before the barrier that
  // ends the memory slot of the next).  The vmcnt values leave exactly the younger loads in flight.
  auto step4 = [&](int t, auto KIND) {
    constexpr bool MORE = decltype(KIND)::value != LAST;
    const uint32_t cur = (t & 1) ? STAGE : 0, nxt = STAGE - cur;
    // phase 0
    read_b(I1{});
    read_a(I1{});
    if constexpr (MORE) load_a(a1, nxt, I2{});
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(LAB));
    tie_a(I0{});
    tie_b(I0{});
    cut(KIND, I0{});
    wait_loads(KIND, std::integral_constant<int, (MORE ? 3 : 2) + BI>{});     // A quarters 2, 3 of this step have landed
    __builtin_amdgcn_s_barrier();
    products(I0{}, I1{}, [&] {
      if constexpr (MORE) e2 = prep_entries(p2);
    });
    // phase 1
    if constexpr (MORE) read_entries(e2, ent);
    read_a(I2{});
    if constexpr (MORE) load_a(a1, nxt, I3{});
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(LA));
    tie_a(I1{});
    tie_b(I1{});
    if constexpr (MORE) tie_entries();
    cut(KIND, I1{});
    __builtin_amdgcn_s_barrier();
    products(I1{}, I2{}, [&] {
      if constexpr (MORE) {
        a2 = prep_a(p2);
        b2 = prep_b(p2, ent);
      }
    });
    // phase 2
    read_a(I3{});
    if constexpr (MORE) {
      load_a(a2, cur, I0{});
      load_a(a2, cur, I1{});
      load_b(b2, cur, I0{});
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(LA));
    tie_a(I0{});
    if constexpr (CUT_A) cut(KIND, I0{});
    if constexpr (MORE) wait_loads(KIND, std::integral_constant<int, 5>{});          // B and A quarters 0, 1 of step t+1 have landed
    __builtin_amdgcn_s_barrier();
    products(I2{}, I2{}, [&] {
      if constexpr (MORE) {
        to_stage((t & 1) ? -STAGE : STAGE);
        sg_at = prep_signs(p1);
      }
    });
    // phase 3
    if constexpr (MORE) {
      read_signs(sg_at);
      read_b(I0{});
      read_a(I0{});
      static_for<BI - 1>([&](auto U) { load_b(b2, cur, std::integral_constant<int, decltype(U)::value + 1>{}); });
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(MORE ? LAB : 0));
    tie_a(I1{});
    if constexpr (CUT_A) cut(KIND, I1{});
    __builtin_amdgcn_s_barrier();
    products(I3{}, std::integral_constant<int, MORE ? 0 : 2>{}, [&] {
      if constexpr (MORE) {
        a1 = a2;
        p0 = p1;
        p1 = p2;
        if (t + 3 < KT) advance(p2);
      }
    });
  };
  // A step of two phases, three stages: the loads of step t+2 go into the stage of step t-1, all of them at
  // the start (they are in flight for a whole step).
  auto step2 = [&](int t, uint32_t cur, uint32_t nxt, uint32_t nn, auto KIND) {   // stages of steps t, t + 1, t + 2
    constexpr bool MORE = decltype(KIND)::value != LAST;
    // phase 0
    read_b(I1{});
    read_a(I1{});
    if constexpr (MORE) {
      static_for<AQ>([&](auto Q) { load_a(a2, nn, Q); });
      static_for<BI>([&](auto U) { load_b(b2, nn, U); });
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(LAB));
    tie_a(I0{});
    tie_b(I0{});
    cut(KIND, I0{});
    if constexpr (MORE) wait_loads(KIND, std::integral_constant<int, AQ + BI>{});    // step t+1 has landed
    __builtin_amdgcn_s_barrier();
    Pos p3 = p2;
    products(I0{}, I1{}, [&] {
      if constexpr (MORE) {
        if (t + 3 < KT) advance(p3);
        e2 = prep_entries(p3);
        to_stage((int)(nxt - cur));
        sg_at = prep_signs(p1);
      }
    });
    // phase 1
    if constexpr (MORE) {
      read_signs(sg_at);
      read_entries(e2, ent);
      read_b(I0{});
      read_a(I0{});
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(MORE ? LAB : 0));
    tie_a(I1{});
    tie_b(I1{});
    if constexpr (MORE) tie_entries();
    cut(KIND, I1{});
    __builtin_amdgcn_s_barrier();
    products(I1{}, std::integral_constant<int, MORE ? 0 : 2>{}, [&] {
      if constexpr (MORE) {
        p0 = p1;
        p1 = p2;
        p2 = p3;
        a2 = prep_a(p3);
        b2 = prep_b(p3, ent);
      }
    });
  };
  if (KT > 0) {
    __builtin_amdgcn_s_waitcnt(vmcnt_only(BI));            // step 0 has landed
    __builtin_amdgcn_s_barrier();
    read_signs(prep_signs(p0));
    if constexpr (PH == 2) {
      read_entries(prep_entries(p2), ent);
      a2 = prep_a(p2);
    } else {
      a1 = prep_a(p1);
    }
    read_b(I0{});
    read_a(I0{});
    asm volatile("s_waitcnt lgkmcnt(0)");
    if constexpr (XSIGN) {
      tie_b(I0{});
      take_signs();
      put_signs(I0{});
    }
    if constexpr (PH == 2) tie_entries();
    if constexpr (PH == 2) b2 = prep_b(p2, ent);
    if (wave >= 4) __builtin_amdgcn_s_barrier();           // half a phase behind from here on
    uint32_t s0 = 0, s1 = STAGE, s2 = 2 * STAGE;   // (PH == 2: the stages, taking turns)
    auto step = [&](int t, auto KIND) {
      if constexpr (PH == 4) {
        step4(t, KIND);
      } else {
        step2(t, s0, s1, s2, KIND);
        const uint32_t r = s0;
        s0 = s1; s1 = s2; s2 = r;
      }
    };
    int t = 0;
    for (int blk = 0;; ++blk) {
      const int end = X3 ? KT - 6 : STRIPS && blk < NB - 1 ? (blk + 1) * KQ : KT - 1;
      for (; t < end; ++t) step(t, std::integral_constant<int, MID>{});
      if constexpr (X3)
        for (; t < KT - 1; ++t) step(t, std::integral_constant<int, TAIL>{});
      if constexpr (!STRIPS) break;
      if (blk >= NB - 1) break;
      store_bf16(n0 + BN * blk + wn * WTN, std::true_type{});        // a block that another follows (a strip's blocks have two steps at least)
#pragma unroll
      for (int i = 0; i < RH * MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
      step(t, std::integral_constant<int, FIRST>{});
      ++t;
    }
    step(KT - 1, std::integral_constant<int, LAST>{});
    if (wave < 4) __builtin_amdgcn_s_barrier();
    // loads of a step that does not come may still be on their way to LDS: let them land
    __builtin_amdgcn_s_waitcnt(vmcnt_only(0));
    if (MODE == MODE_DM && p.G == nullptr) __builtin_amdgcn_s_barrier();   // the operand stages are about to be used for something else
  }

  // ---- epilogue
  const int cb = n0 + BN * (NB - 1) + wn * WTN;    // first column of the wave in the last (or only) block
  if constexpr (MODE != MODE_DM && !X3) {
    if (p.G == nullptr) {
      store_bf16(cb, std::false_type{});
      return;
    }
  }
  if (MODE != MODE_DM || p.G != nullptr) {
    // fp32 out: raw products or partial outputs, which another kernel reads, or (X3) the result
    const int l = lane_id();
    float* out = p.G ? p.G + (int64_t)bz * Mdim * Ndim : p.C32;
    const int64_t ldo = p.G ? (int64_t)Ndim : p.ldc;
    const float scale = MODE == MODE_DM ? 1.f : a.lambda;
#pragma unroll
    for (int f = 0; f < RH * MI; ++f)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int row = frag_row(f) + (l & 15), col = cb + 16 * j + 4 * (l >> 4);
        if (row < Mdim && col < Ndim) *reinterpret_cast<floatx4*>(out + (int64_t)row * ldo + col) = scale * acc[f][j];
      }
    return;
  }
  if constexpr (MODE == MODE_DM) {
    // A wave passes 16 rows at a time through its own part of the operand stages and adds them row by row
    // (LDS operations of one wave complete in order).
    const int elane = lane_id();
    constexpr int ES32 = WTN * 4 + 16;             // bytes per staged row
    char* ebuf = smem + wave * (16 * ES32);
    // Consecutive lanes take consecutive columns of a row: the chip serves atomic adds by the 64-byte
    // piece (18.7 G pieces/s), so the lanes of an instruction should share as few as possible.  64
    // lanes cover one row of 64 columns, or 4/3 rows of 48: a pattern of PAT instructions.
    constexpr int PAT = WTN == 48 ? 3 : 1, NIT = 16 * WTN / 64;
    static_assert(WTN == 64 || WTN == 48, "rows of 64 or 48 columns");
    // Tiles as wide as the wave's columns or a half, a quarter of them: their 16 rows are one run of slots, and lanes run over it
    // from a multiple of 64 bytes on, 64 slots at a time -- 65 pieces for 16 x 64 where rows from any offset
    // on make 79 (two runs of 33 against 94 with tiles 32 wide).  8192 x 768 x 3072 63.8 -> 61.3 us, 512 x 4096 x 4096 77 -> 67,
    // 635 x 2816 x 6144 with tiles 16 wide 143 -> 110.
    const bool runs = WTN == 64 && p.runs && a.Z2 >= 16 && 64 % a.Z2 == 0 && cb + 64 <= (int)a.O;
    int er[PAT], eo[PAT], ey[PAT];
#pragma unroll
    for (int v = 0; v < PAT; ++v) {
      er[v] = (64 * v + elane) / WTN;
      const int o = cb + (64 * v + elane) % WTN;
      const int oc = min(o, (int)a.O - 1);
      ey[v] = oc / a.Z2 - y0;
      eo[v] = o < (int)a.O ? oc % a.Z2 : -1;
    }
#pragma unroll
    for (int f = 0; f < RH * MI; ++f) {
      const int h0 = frag_row(f);                  // 16 rows of one row of hash tiles (Z1 % 16 == 0)
      if (h0 >= (int)a.H) continue;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        *reinterpret_cast<floatx4*>(ebuf + (elane & 15) * ES32 + (16 * j + 4 * (elane >> 4)) * 4) = acc[f][j];
      const int x = h0 / a.Z1;
      if (runs && h0 + 16 <= (int)a.H) {
        const int len = 16 * a.Z2, zl = 31 - __builtin_clz(a.Z2);
        for (int t = 0; t < 64 >> zl; ++t) {
          const int64_t e = s_dm[(x - x0) * TN + ((cb >> zl) + t - y0)];
          float* to = p.dM + (e & INT64_MAX) + (int64_t)a.Z2 * (h0 - x * a.Z1);
          const float sc = e < 0 ? -a.lambda : a.lambda;
          const int shift = (int)(((uintptr_t)to >> 2) & 15);
          constexpr int B = 9;                     // reads of the staged rows at a time (a run of 32-wide tiles, half of one of 64)
          for (int i0 = elane - shift; i0 - elane < len; i0 += 64 * B) {
            float val[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
              const int i = min(max(i0 + 64 * u, 0), len - 1);
              val[u] = *reinterpret_cast<const float*>(ebuf + (i >> zl) * ES32 + ((t << zl) + (i & (a.Z2 - 1))) * 4);
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
              const int i = i0 + 64 * u;
              if (i >= 0 && i < len) unsafeAtomicAdd(to + i, sc * val[u]);
            }
          }
        }
        continue;
      }
      float* d[PAT];
      float sc[PAT];
#pragma unroll
      for (int v = 0; v < PAT; ++v) {
        const int64_t e = s_dm[(x - x0) * TN + ey[v]];
        d[v] = p.dM + (e & INT64_MAX) + (int64_t)a.Z2 * (h0 - x * a.Z1 + er[v]) + eo[v];
        sc[v] = e < 0 ? -a.lambda : a.lambda;
      }
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int v = it % PAT, r = (it / PAT) * (64 * PAT / WTN);
        const float val = *reinterpret_cast<const float*>(ebuf + (r + er[v]) * ES32 + ((64 * v + elane) % WTN) * 4);
        if (eo[v] >= 0 && h0 + r + er[v] < (int)a.H) unsafeAtomicAdd(d[v] + (int64_t)a.Z2 * r, sc[v] * val);
      }
    }
  }
}

template <int MODE, int BM, int BN, bool X3, bool NEG>
roast_status launch(const WideArgs& p, hipStream_t s) {
  const int64_t total = (int64_t)p.nbx * p.nby * p.nbz;
  if (total > (1ll << 30)) return ROAST_ERR_UNSUPPORTED;
  constexpr int smem = MODE == MODE_DM ? lds_operands(BM, BN) + kTableDM * 8 : 160 * 1024;
  static_assert(smem <= 160 * 1024 && 8 * 16 * (64 * 4 + 16) <= lds_operands(BM, BN), "LDS budget");
  static std::atomic<bool> configured{false};   // per instantiation; a race between host threads only repeats the call
  if (!configured.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_roast_mfma_wide<MODE, BM, BN, X3, NEG>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, smem) != hipSuccess)
      return ROAST_ERR_HIP;
    configured.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((k_roast_mfma_wide<MODE, BM, BN, X3, NEG>), dim3((unsigned)((total + 7) / 8 * 8)), dim3(512), smem, s, p);
  return hip_status(hipGetLastError());
}

template <int MODE, bool X3, bool NEG>
roast_status launch_block(const WideArgs& p, int bm, int bn, hipStream_t s) {
  if (bm == 256 && bn == 256) return launch<MODE, 256, 256, X3, NEG>(p, s);
  if (bm == 256 && bn == 192) return launch<MODE, 256, 192, X3, NEG>(p, s);
  if (bm == 256 && bn == 128) return launch<MODE, 256, 128, X3, NEG>(p, s);
  if (bm == 128 && bn == 192) return launch<MODE, 128, 192, X3, NEG>(p, s);
  return ROAST_ERR_UNSUPPORTED;
}

template <int MODE>
roast_status launch_hashed(const WideArgs& p, int bm, int bn, bool x3, hipStream_t s) {
  if (x3) return launch_block<MODE, true, false>(p, bm, bn, s);
  if (bm == 128 && bn == 128) return shadow_copies(p.a.m_size) == 4 ? launch<MODE, 128, 128, false, true>(p, s) : launch<MODE, 128, 128, false, false>(p, s);
  return shadow_copies(p.a.m_size) == 4 ? launch_block<MODE, false, true>(p, bm, bn, s) : launch_block<MODE, false, false>(p, bm, bn, s);
}

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

bool hashed_ok(const MMArgs& a) {
  return a.hash.use_sign != 2 && a.Z1 % 32 == 0 && a.Z2 % 32 == 0 && a.H % 8 == 0 && a.O % 8 == 0 && a.m_size < (1ll << 28);   // byte offsets into the shadow in 32 bits
}

// ---- which block, how many blocks to a strip, how many parts of the contraction: the smallest
// modelled time.  The constants (microseconds) are fitted to timed launches (not kept) of 160 layer shapes with
// 16 .. 16384 rows and 256 .. 16384 columns.
struct Block {
  int bm, bn;
  double step, busy;     // forward / dX: a 64-deep step; added to it when all CUs are busy (clocks and memory)
  double fixed, more;    // a workgroup's start and end; a further block of a strip
  double dm_step, dm_fixed, dm_adds;   // dM: the same; atomic adds per microsecond, whole chip, as if nothing overlapped them (0.36e6: 28 G 64-byte pieces/s, where the chip serves 18.7)
};
constexpr Block kBlocks[] = {{256, 256, 1.0, 0.33, 5.9, 0.0, 1.11, 8.7, 0.36e6},
                             {256, 192, 0.88, 0.25, 5.2, 4.6, 1.03, 7.7, 0.29e6},    // (48-column rows of a wave: more pieces)
                             {256, 128, 0.67, 0.18, 4.0, 0.0, 0.78, 4.9, 0.36e6},
                             {128, 192, 0.57, 0.14, 4.2, 1.9, 0.635, 4.8, 0.29e6}};

double rounds_of(double wgs) {                     // of 256 workgroups; a last partial round costs less than a full one
  const double r = wgs / 256.0;
  return r <= 1.0 ? 1.0 : 0.63 * std::ceil(r) + 0.37 * r;
}

// A call without a copy of M runs on the 256 x 128 kernel, in as many parts (both give the same sums).  Where the number
// that is best here costs that kernel over a tenth more than its own best, the one with the least
// time of both together, among those close to the best here: within 7 %, or, if the best is no split at all, 8 % less
// 1.2 microseconds (a first split is a launch more, which the model sees too small on short calls: with a copy 168 x 392 x 552
// would go from 11.2 to 13.3 us, 26 x 600 x 4392 from 12.1 to 14.6).  With a copy and without, by the best here and by this rule:
// 64 x 4096 x 4096 17.9 and 27.4 -> 17.4 and 19.7 us, 126 x 5480 x 4264 22.2 and 43.6 -> 22.4 and 29.3,
// 1024 x 2048 x 2048 25.1 and 34.9 -> 25.4 and 28.6.
int parts_for_both(int64_t I, int64_t N, int64_t K, const double* cost_of, int best) {
  const int64_t tiles = cdiv(N, 128) * cdiv(I, 256);
  double narrow[kWideParts + 1], least = 1e300;
  for (int parts = 1; parts <= kWideParts; ++parts) {
    narrow[parts] = (double)cdiv(tiles * parts, 256) * (0.95 * (double)cdiv(cdiv(K, parts), BK) + 4.0) +
                    (parts > 1 ? 4.0 + (double)parts * (double)I * (double)N * 4.0 / 3.0e6 : 0.0);
    least = std::min(least, narrow[parts]);
  }
  if (narrow[best] <= 1.1 * least) return best;
  const double limit = best == 1 ? 1.08 * cost_of[1] - 1.2 : 1.07 * cost_of[best];
  for (int parts = 1; parts <= kWideParts; ++parts)
    if (cost_of[parts] <= limit && cost_of[parts] + narrow[parts] < cost_of[best] + narrow[best]) best = parts;
  return best;
}

// which: MODE_FWD / MODE_DX; max_parts == 1: no workspace for a split
WidePlan plan_hashed(int which, const MMArgs& a, int max_parts, bool x3) {
  if (!hashed_ok(a)) return {};
  const int64_t N = which == MODE_FWD ? a.O : a.H, K = which == MODE_FWD ? a.H : a.O;
  const int64_t zn = which == MODE_FWD ? a.Z2 : a.Z1, zk = which == MODE_FWD ? a.Z1 : a.Z2;
  const int pairs = x3 ? 6 : 1;
  WidePlan of[kWideParts + 1];                     // the fastest launch with each number of parts
  double cost_of[kWideParts + 1];
  std::fill(cost_of, cost_of + kWideParts + 1, 1e300);
  for (const Block& b : kBlocks) {
    for (int64_t t = 1; t <= 4; ++t) {
      // a strip: whole blocks of whole tiles, no ragged step, two steps to a block at least
      if (t > 1 && (x3 || b.bn != 192 || K % BK != 0 || K < 2 * BK || N % (b.bn * t) != 0 || b.bn % zn != 0)) continue;
      const int64_t tn = t > 1 ? b.bn * t / zn : cdiv(b.bn, zn) + 1;
      const double blocks = (double)cdiv(a.I, b.bm) * (double)cdiv(N, b.bn * t);
      // (a split of what fills the chip anyway only adds work)
      for (int parts = 1; parts <= max_parts && (parts == 1 || (t == 1 && blocks < 256.0 && blocks * parts <= 512.0)); ++parts) {
        const int64_t steps = cdiv(cdiv(K, parts), BK);
        if (parts > 1 && (steps * pairs < 2 || cdiv(K, steps * BK) != parts)) continue;
        if ((cdiv(steps * BK, zk) + 1) * tn > table_entries(b.bm, b.bn)) continue;
        const double wgs = blocks * parts;
        const double step = b.step + b.busy * std::min(wgs / 256.0, 1.0);
        double cost = rounds_of(wgs) * ((double)(steps * t * pairs) * step + b.fixed + b.more * (double)(t - 1));
        if (parts > 1) cost += 3.8 + (double)parts * (double)a.I * (double)N * 4.0 / 3.0e6;   // the pass over the partial outputs
        if (cost < cost_of[parts]) {
          cost_of[parts] = cost;
          of[parts] = {b.bm, b.bn, (int)t, parts, (int)(steps * BK), cost};
        }
      }
    }
  }
  int best = (int)(std::min_element(cost_of + 1, cost_of + max_parts + 1) - cost_of);
  if (cost_of[best] == 1e300) return {};
  if (!x3 && max_parts > 1) best = parts_for_both(a.I, N, K, cost_of, best);
  return of[best];
}

// The same launch in 128 x 128 blocks, where all of them run at a time and that is modelled to be faster: more CUs for a product that leaves a third of them or more
// without a block.  In microseconds with blocks of 128 x 192 or 256 x 128 and with these, by their number: 1659 x 2432 x 896 247, 16.8 and 14.5;
// 3823 x 448 x 896 120, 15.0 and 12.4; 3549 x 896 x 3008 196, 35.9 and 29.2; 1198 x 2752 x 1792 220, 25.4 and 20.7; 1290 x 1344 x 320 121, 9.2 and 7.8.
// In two rounds they are slower than what there is (264 of them 23.7 and 33.9), and so they are for fp32 planes (252 over 1280 indices 83.0 and 87.8).  The
// parts stay as they are: a call without a copy of M gives the same sums.  Tiles that a block holds whole, and 16 blocks at least (below, no call is long).
WidePlan plan_square(int which, const MMArgs& a, const WidePlan& w) {
  const int64_t N = which == MODE_FWD ? a.O : a.H, zn = which == MODE_FWD ? a.Z2 : a.Z1, zk = which == MODE_FWD ? a.Z1 : a.Z2;
  const int64_t wgs = cdiv(a.I, 128) * cdiv(N, 128) * w.parts, K = which == MODE_FWD ? a.H : a.O;
  const int64_t rows = w.parts > 1 ? w.rows : cdiv(K, BK) * BK;
  if (w.nblk != 1 || wgs > 256 || wgs < 16 || 128 % zn != 0 || (cdiv(rows, zk) + 1) * (128 / zn + 1) > table_entries(128, 128)) return w;
  const double finish = w.parts > 1 ? 3.8 + (double)w.parts * (double)a.I * (double)N * 4.0 / 3.0e6 : 0.0;
  const double us = (double)(rows / BK) * (0.45 + 0.07 * (double)wgs / 256.0) + 3.9 + finish;
  return us < w.us ? WidePlan{128, 128, 1, w.parts, w.rows, us} : w;
}

// parts > 0: the number of parts is given (and the products go to a workspace)
WidePlan plan_dm(const MMArgs& a, int parts, bool x3) {
  WidePlan best{};
  if (a.H % 8 != 0 || a.O % 8 != 0 || (parts == 0 && (a.hash.use_sign == 2 || a.Z1 % 16 != 0))) return best;
  const int pairs = x3 ? 6 : 1;
  double best_cost = 1e300;
  for (const Block& b : kBlocks) {
    if (parts == 0 && (cdiv(b.bm, a.Z1) + 1) * (cdiv(b.bn, a.Z2) + 1) > kTableDM) continue;
    const int64_t tiles = cdiv(a.H, b.bm) * cdiv(a.O, b.bn);
    for (int q = parts > 0 ? parts : 1; q <= (parts > 0 ? parts : kWideParts); ++q) {
      const int64_t steps = cdiv(cdiv(a.I, q), BK);
      if (parts == 0 && q > 1 && (steps * pairs < 2 || cdiv(a.I, steps * BK) != q)) continue;
      double cost = rounds_of((double)(tiles * q)) * ((double)(steps * pairs) * b.dm_step + b.dm_fixed);
      // rows of tiles narrower than a wave's 64 columns break the adds into more pieces; adds to one address
      // (|M| far smaller than the layer) complete 25 ns apart
      if (parts == 0)
        cost += (double)q * (double)a.H * (double)a.O * ((a.Z2 < 64 ? 1.2 : 1.0) / b.dm_adds + 0.025 / (double)a.m_size);
      if (cost < best_cost) {
        best_cost = cost;
        best = {b.bm, b.bn, 1, q, (int)(steps * BK), cost};
      }
    }
  }
  return best;
}

}  // namespace

WidePlan wide_fwd_plan(const MMArgs& a, int max_parts, bool x3) {
  return remembered<WidePlan>(a, 4 * max_parts + MODE_FWD, x3, [&] { return plan_hashed(MODE_FWD, a, max_parts, x3); });
}
WidePlan wide_dx_plan(const MMArgs& a, int max_parts, bool x3) {
  return remembered<WidePlan>(a, 4 * max_parts + MODE_DX, x3, [&] { return plan_hashed(MODE_DX, a, max_parts, x3); });
}
WidePlan wide_square_plan(int which, const MMArgs& a, const WidePlan& plan) { return plan_square(which, a, plan); }
WidePlan wide_dm_plan(const MMArgs& a, int parts, bool x3) {
  return remembered<WidePlan>(a, 4 * parts + MODE_DM, x3, [&] { return plan_dm(a, parts, x3); });
}

// plan.parts > 1: ws holds the partial outputs
roast_status wide_mm(int which, const MMArgs& a, const WidePlan& plan, const uint16_t* A, int64_t lda, int64_t a_plane,
                     const uint16_t* Mb, bool x3, uint16_t* C, float* C32, int64_t ldc, float* ws, hipStream_t s) {
  if (lda >= (1ll << 24)) return ROAST_ERR_UNSUPPORTED;     // 8 rows' byte offsets in 32 bits
  WideArgs p{};
  p.a = a; p.th = make_tile_hash(a.hash, a.layer, a.nTx, a.nTy);
  p.A = A; p.lda = lda; p.a_plane = a_plane; p.Mb = Mb; p.mb_stride = shadow_stride(a.m_size);
  p.mb_plane = 2 * p.mb_stride; p.C = C; p.C32 = C32; p.ldc = ldc;
  const int64_t n = which == MODE_FWD ? a.O : a.H;
  p.nblk = plan.nblk;
  p.nbx = (int)cdiv(n, (int64_t)plan.bn * plan.nblk); p.nby = (int)cdiv(a.I, plan.bm); p.nbz = plan.parts;
  if (plan.parts > 1) { p.G = ws; p.rows_per_split = plan.rows; }
  return which == MODE_FWD ? launch_hashed<MODE_FWD>(p, plan.bm, plan.bn, x3, s) : launch_hashed<MODE_DX>(p, plan.bm, plan.bn, x3, s);
}

roast_status wide_mm_dM(const MMArgs& a, const WidePlan& plan, const uint16_t* X, int64_t ldx, int64_t a_plane, const uint16_t* dY,
                        int64_t ldy, int64_t b_plane, bool x3, float* dM, float* G, const int* split_begin, hipStream_t s) {
  if (ldx >= (1ll << 23) || ldy >= (1ll << 23)) return ROAST_ERR_UNSUPPORTED;   // 24-bit products with row numbers
  WideArgs p{};
  p.a = a; p.th = make_tile_hash(a.hash, a.layer, a.nTx, a.nTy);
  p.A = X; p.lda = ldx; p.a_plane = a_plane; p.B = dY; p.ldb = ldy; p.b_plane = b_plane; p.dM = dM; p.G = G;
  p.nbx = (int)cdiv(a.O, plan.bn); p.nby = (int)cdiv(a.H, plan.bm); p.nbz = plan.parts;
  p.rows_per_split = plan.rows;
  // A launch with few adds waits for the steps of its epilogue one after the other, of which runs have more: 64 x 448 x 1024 (0.5 M adds) 10.4 -> 12.1 us,
  // 67 x 1728 x 768 (1.3 M) 16.1 -> 18.2, but 48 x 3072 x 640 (2 M) 29.4 -> 22.4.
  p.runs = (double)plan.parts * (double)a.H * (double)a.O >= 1.6e6;
  if (split_begin)
    for (int i = 0; i <= plan.parts; ++i) p.split_begin[i] = split_begin[i];
  return x3 ? launch_block<MODE_DM, true, false>(p, plan.bm, plan.bn, s) : launch_block<MODE_DM, false, false>(p, plan.bm, plan.bn, s);
}

}  // namespace roast
