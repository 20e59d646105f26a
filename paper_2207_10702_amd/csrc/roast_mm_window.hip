// Gradient of M, dM = scatter(X^T*dY) (Section 4.3 of arXiv 2207.10702), of few tokens and an M smaller than the layer, on gfx950.
//
// What bounds the blocks of the wide kernels there is their atomic adds, one for each virtual weight whatever the number of tokens: 0.3 T/s, 57 us for
// 1640 x 12608 and 61 tokens.  Here a workgroup owns a window of consecutive slots of M, as fp64 sums in LDS, and takes the products of all tiles (of
// its share of them) that reach into it: a slot is added to dM once per workgroup of its window, not once per tile that holds it.  The price is
// that operands are read once for each tile, not once for a block of many; few tokens keep them in the L2.
#include <algorithm>
#include <atomic>
#include <cmath>

#include "roast_internal.hpp"

namespace roast {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));

constexpr int kStep = 32;                // tokens of a step
constexpr int kGuard = 64;               // slots beside a window
constexpr int kList = 2048;              // tiles of the window at hand

struct WindowArgs {
  MMArgs a;
  TileHash th;
  const uint16_t* X;
  int64_t ldx;
  const uint16_t* dY;
  int64_t ldy;
  float* dM;
  int window;                            // slots of a window (a power of two)
  int shares;                            // workgroups of a window, which share out the tiles
};

// Rows of U columns; their chunks of 32 bytes are permuted by k, which meets no bank twice in a clock.
template <int U>
__device__ __forceinline__ int swz(int k) {
  return U == 64 ? ((k >> 1) & 1) | (((k >> 3) & 1) << 1) : (k >> 3) & 1;
}
// The fragments of 16 columns of [k][U columns] by transposing reads: lanes 4r .. 4r+3 of a group of 16 give the addresses
// of row r (k = r resp. 4 + r), lane c receives the eight k-values of column c.
template <int U>
__device__ __forceinline__ void read_columns(uint4v* f, char* at) {
  typedef short short4 __attribute__((ext_vector_type(4)));
  const int lane = threadIdx.x & 63, tk = 8 * (lane >> 4) + ((lane & 15) >> 2);
  const uint32_t off = (uint32_t)(tk * 2 * U + (swz<U>(tk) << 5) + (lane & 3) * 8);
  auto read = [&](uint32_t o) {
    return __builtin_bit_cast(uint2v, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4*)(at + o)));
  };
#pragma unroll
  for (int j = 0; j < U / 16; ++j) {
    const uint2v l = read(off ^ (32u * j)), h = read((off ^ (32u * j)) + 8u * U);
    f[j] = uint4v{l[0], l[1], h[0], h[1]};
  }
}

// bytes of a wave's stage: kStep rows of U1 columns of X, and of U2 of dY
constexpr int stage_bytes(int u1, int u2) { return kStep * 2 * (u1 + u2); }

// U1, U2: a wave's unit of work, 64 x 64 or (sides that are no multiple of 64) 32 wide, inside one tile.
template <int U1, int U2, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES / 4) void k_dm_window(WindowArgs p) {
  constexpr int NI = U1 / 16, NJ = U2 / 16, LX = U1 / 8, LY = U2 / 8, NX = kStep * LX / 64, NY = kStep * LY / 64;   // lanes of a row, loads of a step
  constexpr int kStage = stage_bytes(U1, U2), kStageY = kStep * 2 * U1;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const MMArgs& a = p.a;
  double* image = reinterpret_cast<double*>(smem + WAVES * kStage) + kGuard;
  uint2v* list = reinterpret_cast<uint2v*>(image + p.window + kGuard);            // offset | sign << 31; tile x | y << 16
  int* count = reinterpret_cast<int*>(list + kList);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4;
  const int share = (int)blockIdx.x % p.shares, w0 = (int)blockIdx.x / p.shares * p.window;
  const int I = (int)a.I, H = (int)a.H, O = (int)a.O, Z2 = a.Z2, area = a.Z1 * a.Z2;
  char* stage = smem + wave * kStage;
  for (int i = tid; i < p.window / 2; i += 64 * WAVES) reinterpret_cast<floatx4*>(image)[i] = floatx4{0.f, 0.f, 0.f, 0.f};
  // Operands come through registers (a step of each wave on its way) and the wave's own stage.
  const uint32_t ldx2 = (uint32_t)p.ldx * 2u, ldy2 = (uint32_t)p.ldy * 2u;
  const int tiles = (int)(a.nTx * a.nTy), nTy = (int)a.nTy;
  const int sub2 = a.Z2 / U2, sub = a.Z1 / U1 * sub2;                    // units of a tile, of its row

  // What a wave does next: a step of a unit.  n: unit number in the list (tile * sub + unit of it)
  struct Work {
    int n, k, h0, o0, off;               // tokens from k on; the unit's first row and column; slot of its first weight less w0
    uint32_t flip;
  };
  int have = 0;                          // tiles in the list
  auto seek = [&](Work& w) {             // the first unit from w.n on, in steps of the waves, that has weights in the window
    for (; w.n < have * sub; w.n += WAVES) {
      const int e = w.n / sub, s = w.n - e * sub, sx = s / sub2;
      const uint2v t = list[e];
      const uint32_t place = __builtin_amdgcn_readfirstlane(t[0]), xy = __builtin_amdgcn_readfirstlane(t[1]);
      const int x = (int)(xy & 0xffffu), y = (int)(xy >> 16), i1 = sx * U1, i2 = (s - sx * sub2) * U2;
      w.h0 = x * a.Z1 + i1;
      w.o0 = y * a.Z2 + i2;
      if (w.h0 >= H || w.o0 >= O) continue;
      w.off = (int)(place & 0x7fffffffu) - w0 + i1 * Z2 + i2;
      if (w.off >= p.window || w.off + (U1 - 1) * Z2 + U2 <= 0) continue;
      w.flip = place & 0x80000000u;
      w.k = 0;
      return;
    }
    w.n = -1;
  };
  struct Buf {
    uint4v x[NX], y[NY];
  };
  auto load = [&](Buf& q, const Work& w) {
    // columns beyond the last ones, and tokens, repeat those: they are not added, resp. cut
    const char* x = reinterpret_cast<const char*>(p.X + (int64_t)w.k * p.ldx);
    const char* y = reinterpret_cast<const char*>(p.dY + (int64_t)w.k * p.ldy);
    const uint32_t cx = 2u * (uint32_t)min(w.h0 + 8 * (lane % LX), H - 8), cy = 2u * (uint32_t)min(w.o0 + 8 * (lane % LY), O - 8);
#pragma unroll
    for (int v = 0; v < NX; ++v) q.x[v] = *reinterpret_cast<const uint4v*>(x + (__umul24((uint32_t)min(64 / LX * v + lane / LX, I - 1 - w.k), ldx2) + cx));
#pragma unroll
    for (int v = 0; v < NY; ++v) q.y[v] = *reinterpret_cast<const uint4v*>(y + (__umul24((uint32_t)min(64 / LY * v + lane / LY, I - 1 - w.k), ldy2) + cy));
  };
  auto put = [&](const Buf& q) {
#pragma unroll
    for (int v = 0; v < NX; ++v) {
      const int row = 64 / LX * v + lane / LX, c = lane % LX;
      *reinterpret_cast<uint4v*>(stage + row * 2 * U1 + (((c >> 1) ^ swz<U1>(row)) << 5) + (c & 1) * 16) = q.x[v];
    }
#pragma unroll
    for (int v = 0; v < NY; ++v) {
      const int row = 64 / LY * v + lane / LY, c = lane % LY;
      *reinterpret_cast<uint4v*>(stage + kStageY + row * 2 * U2 + (((c >> 1) ^ swz<U2>(row)) << 5) + (c & 1) * 16) = q.y[v];
    }
  };
  for (int base = share; base < tiles;) {
    // ---- the tiles that reach into the window, until the list may be full
    __syncthreads();                     // the list before has been worked off (and the image is zero)
    if (tid == 0) *count = 0;
    __syncthreads();
    do {
      const int64_t t = base + (int64_t)tid * p.shares;
      if (t < tiles) {
        const int x = (int)t / nTy, y = (int)t - x * nTy;
        bool neg;
        const int64_t off = tile_place(a.hash, p.th, a.layer, (uint32_t)x, (uint32_t)y, &neg);
        if (off < (int64_t)w0 + p.window && off + area > w0)
          list[atomicAdd(count, 1)] = uint2v{(uint32_t)off | (neg ? 0x80000000u : 0u), (uint32_t)x | (uint32_t)y << 16};
      }
      base = (int)std::min<int64_t>(base + (int64_t)64 * WAVES * p.shares, tiles);
      __syncthreads();
      have = *count;
      __syncthreads();
    } while (base < tiles && have <= kList - 64 * WAVES);
    have = __builtin_amdgcn_readfirstlane(have);
    // ---- their products; waves go their own ways
    Work w{wave, 0, 0, 0, 0, 0u};
    seek(w);
    Buf buf;
    if (w.n >= 0) load(buf, w);
    floatx4 acc[NI][NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    while (w.n >= 0) {
      put(buf);
      Work next = w;
      next.k += kStep;
      if (next.k >= I) {
        next.n += WAVES;
        seek(next);
      }
      if (next.n >= 0) load(buf, next);
      uint4v af[NI], bf[NJ];
      read_columns<U1>(af, stage);
      read_columns<U2>(bf, stage + kStageY);
      const int rem = I - w.k;
      if (rem < kStep) {                 // zeros in both operands: what was loaded there may be an infinity
        const int cnt = rem - 8 * g;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const uint32_t keep = cnt >= 2 * d + 2 ? 0xffffffffu : (cnt == 2 * d + 1 ? 0x0000ffffu : 0u);
#pragma unroll
          for (int i = 0; i < NI; ++i) af[i][d] &= keep;
#pragma unroll
          for (int j = 0; j < NJ; ++j) bf[j][d] &= keep;
        }
      }
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          // acc[i][j][e]: row 16 i + 4 g + e, column 16 j + r
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, af[i]), __builtin_bit_cast(bf16x8, bf[j]), acc[i][j], 0, 0, 0);
      if (w.k + kStep >= I) {
        // A row of the unit is U2 consecutive slots; one that is partly in the window has the others in the guards beside it.
        const int rows = min(U1, H - w.h0);
        const bool whole = w.off >= 0 && w.off + (U1 - 1) * Z2 + U2 <= p.window && rows == U1;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const int at = w.off + 16 * i * Z2;
          if (at < p.window && at + 15 * Z2 + U2 > 0) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int row = 16 * i + 4 * g + e, slot = w.off + row * Z2;
              float v[NJ];
#pragma unroll
              for (int j = 0; j < NJ; ++j) v[j] = __uint_as_float(__float_as_uint(acc[i][j][e]) ^ w.flip);
              double* to = image + slot + r;
              if (w.o0 + U2 > O) {       // (a ragged last unit)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                  if (slot > -U2 && slot < p.window && row < rows && w.o0 + 16 * j + r < O) unsafeAtomicAdd(to + 16 * j, (double)v[j]);
              } else if (whole || (slot > -U2 && slot < p.window && row < rows)) {
#pragma unroll
                for (int j = 0; j < NJ; ++j) unsafeAtomicAdd(to + 16 * j, (double)v[j]);
              }
            }
          }
        }
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
      w = next;
    }
  }
  __syncthreads();
  for (int i = tid; i < p.window && w0 + i < (int)a.m_size; i += 64 * WAVES) {
    const double v = image[i];
    if (v != 0.0) unsafeAtomicAdd(p.dM + w0 + i, (float)((double)a.lambda * v));
  }
}

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

template <int U1, int U2, int WAVES>
roast_status launch(const WindowArgs& p, int64_t wgs, hipStream_t s) {
  const int smem = WAVES * stage_bytes(U1, U2) + 8 * (p.window + 2 * kGuard) + 8 * kList + 16;
  static std::atomic<bool> configured{false};   // per instantiation; a race between host threads only repeats the call
  if (!configured.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_dm_window<U1, U2, WAVES>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess) return ROAST_ERR_HIP;
    configured.store(true, std::memory_order_release);
  }
  hipLaunchKernelGGL((k_dm_window<U1, U2, WAVES>), dim3((unsigned)wgs), dim3(64 * WAVES), (size_t)smem, s, p);
  return hip_status(hipGetLastError());
}

bool window_ok(const MMArgs& a) {
  return a.hash.use_sign != 2 && a.Z1 % 32 == 0 && a.Z2 % 32 == 0 && a.H % 8 == 0 && a.O % 8 == 0 && a.H < 65536 && a.O < 65536 &&
         a.nTx < 65536 && a.nTy < 65536 && a.m_size < (1ll << 28) && (int64_t)a.Z1 * a.Z2 < (1ll << 20) && a.I <= 384;
}

}  // namespace

// As many workgroups to a window as make 256 of all, one to a CU.  Time in microseconds, by the unit's side (64 or 32 wide): a launch; for each unit of a wave, of which
// windows at both ends of a tile's span take copies, a start and its adds and then the steps; the search through the tiles; the adds to dM.  Fitted to
// 320 launches of 16 to 700 tokens, most within 18 %.  Taken where that is a tenth (a sixth) below what the blocks of the wide kernels (wide_us) are
// modelled to take, and up to 384 tokens: with more the operands, read once for each tile, cost what the adds save.  61 x 1640 x 12608 over 64 Ki slots 82 -> 40 us, 16 x 9944 x 15512 over 3.2 Mi
// 496 -> 234, 246 x 1984 x 1024 over 4096 25 -> 13, 91 x 2432 x 3584 over 118 Ki 43 -> 20; 284 x 2880 x 2496 over 219 Ki 32.5 and 31, 237 x 8128 x 2752 over 9.5 Mi stays, 85 and 109.
// Over 130 random sizes 1.21 times faster in the geometric mean, none slower by more than the runs differ.
WindowPlan window_plan(const MMArgs& a, double wide_us) {
  if (!window_ok(a)) return {};
  const bool u64 = a.Z1 % 64 == 0 && a.Z2 % 64 == 0;
  const int window = a.m_size > 4096 ? 8192 : 4096;
  const int64_t windows = cdiv(a.m_size, window), tiles = a.nTx * a.nTy;
  const int shares = (int)std::min<int64_t>(std::max<int64_t>(256 / windows, 1), tiles);
  const double side = u64 ? 64.0 : 32.0, waves = u64 ? 8.0 : 16.0, wgs = (double)(windows * shares);
  const double span = (side - 1.0) * a.Z2 + side, copies = a.m_size > window ? (span + window) / window : 1.0;
  const double units = (double)cdiv(a.H, (int64_t)side) * (double)cdiv(a.O, (int64_t)side) * copies / wgs;
  const double start = u64 ? (a.Z2 >= 128 ? 3.4 : 2.25) : 2.2, step = u64 ? 0.715 : 0.6;
  const double us = 4.4 + std::max(wgs / 256.0, 1.0) * (((units + (u64 ? 1.1 : 0.25) * std::sqrt(units)) / waves + 0.5) * (start + step * (double)cdiv(a.I, kStep)) +
                                                      1.1 * (double)tiles / shares / (64.0 * waves)) +
                    (u64 ? 1.2e-6 : 1.8e-6) * wgs * (double)std::min<int64_t>(window, a.m_size);
  return (u64 ? 1.1 : 1.2) * us < wide_us ? WindowPlan{window, shares} : WindowPlan{};
}

// X and dY 16-byte aligned, leading dimensions multiples of 8
roast_status window_dM(const MMArgs& a, const WindowPlan& w, const void* X, int64_t ldx, const void* dY, int64_t ldy, float* dM, hipStream_t s) {
  if (ldx >= (1ll << 23) || ldy >= (1ll << 23)) return ROAST_ERR_UNSUPPORTED;   // (24-bit products with row numbers)
  WindowArgs p{};
  p.a = a; p.th = make_tile_hash(a.hash, a.layer, a.nTx, a.nTy);
  p.X = (const uint16_t*)X; p.ldx = ldx; p.dY = (const uint16_t*)dY; p.ldy = ldy; p.dM = dM;
  p.window = w.window; p.shares = w.shares;
  const int64_t wgs = cdiv(a.m_size, w.window) * w.shares;
  if (a.Z2 % 64 == 0) return a.Z1 % 64 == 0 ? launch<64, 64, 8>(p, wgs, s) : launch<32, 64, 8>(p, wgs, s);
  return launch<32, 32, 16>(p, wgs, s);
}

}  // namespace roast
