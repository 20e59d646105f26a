// Deterministic reduction of the ROAST-MM gradient into M (gradient equation of Section 4.3 of
// arXiv 2207.10702: every slot of M receives the lambda-scaled sum of the gradients of all
// virtual weights hashed to it).
//
// Steps: (1) the tile table (offset, sign) is computed on the device and the tiles are ranked by
// (offset, tile id); (2) the per-tile products G = X^T dY are written, unscaled, to the workspace,
// one copy per I-split; (3) a workgroup of consecutive slots of M walks the tiles whose interval
// [offset, offset + Z1*Z2) reaches into them -- a contiguous run of the ranked table because all tiles have
// the same length -- and adds their contributions in a fixed order, splits in index order.  No
// atomics, so the result is bit-identical from run to run.
#include <type_traits>

#include "roast_internal.hpp"

namespace roast {
namespace {

constexpr int64_t kMaxTilesDet = 1 << 17;  // the ranking pass is quadratic in the number of tiles

struct DetLayout {
  size_t g_off, key_off, soff_off, order_off, sgn_off, total;
};

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

inline DetLayout det_layout(const MMArgs& a, int splits) {
  const size_t nT = (size_t)(a.nTx * a.nTy);
  DetLayout l;
  l.g_off = 0;
  l.key_off = align_up((size_t)splits * (size_t)a.H * (size_t)a.O * sizeof(float), 256);
  l.soff_off = l.key_off + align_up(nT * sizeof(int64_t), 256);
  l.order_off = l.soff_off + align_up(nT * sizeof(int64_t), 256);
  l.sgn_off = l.order_off + align_up(nT * sizeof(uint32_t), 256);
  l.total = l.sgn_off + align_up(nT * sizeof(int8_t), 256);
  return l;
}

// rank of tile t among all tiles by (offset, id); writes the sorted offsets and the permutation.
// Sixteen lanes share TILES tiles; each counts the smaller keys among every sixteenth key of the staged
// block, and the counts are added up across the lanes (integers: any order).  Bound: a comparison for each pair of tiles.  Offset and
// id in one key make it one, and several tiles to a lane use a key that was read (11 880 tiles 84 -> 35 us, 65 536 1250 -> 347, beside one tile to a lane, offset and id by themselves).
constexpr int kRankLanes = 16, kRankBlock = 1024;
template <int TILES>
__global__ __launch_bounds__(256) void k_rank_tiles(int64_t nT, const int64_t* __restrict__ off,
                                                    int64_t* __restrict__ sorted_off, uint32_t* __restrict__ order) {
  static_assert(kMaxTilesDet <= 1 << 17, "the id's bits of a key");
  __shared__ int64_t buf[kRankBlock];
  const int64_t t0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kRankLanes * TILES;
  const int sub = threadIdx.x % kRankLanes;
  int64_t mine[TILES];
  int rank[TILES];
#pragma unroll
  for (int i = 0; i < TILES; ++i) {
    mine[i] = t0 + i < nT ? off[t0 + i] << 17 | (t0 + i) : 0;    // (fewer than 2^46 slots: 2^48 bytes)
    rank[i] = 0;
  }
  for (int64_t base = 0; base < nT; base += kRankBlock) {
    __syncthreads();
#pragma unroll
    for (int v = 0; v < kRankBlock / 256; ++v) {
      const int64_t u = base + 256 * v + threadIdx.x;
      buf[256 * v + threadIdx.x] = u < nT ? off[u] << 17 | u : INT64_MAX;
    }
    __syncthreads();
    const int lim = (int)min((int64_t)kRankBlock, nT - base);
#pragma unroll 4
    for (int q = sub; q < lim; q += kRankLanes) {
      const int64_t key = buf[q];
#pragma unroll
      for (int i = 0; i < TILES; ++i) rank[i] += key < mine[i] ? 1 : 0;
    }
  }
#pragma unroll
  for (int i = 0; i < TILES; ++i) {
#pragma unroll
    for (int d = kRankLanes / 2; d >= 1; d >>= 1) rank[i] += __shfl_xor(rank[i], d, 64);
    if (t0 + i < nT && sub == 0) {
      sorted_off[rank[i]] = mine[i] >> 17;
      order[rank[i]] = (uint32_t)(t0 + i);
    }
  }
}

// Number of sorted offsets below x, by all 64 lanes of a wave: 64 places at a time.
__device__ inline int count_below(const int64_t* __restrict__ sorted_off, int n, int64_t x) {
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = n;
  while (lo < hi) {
    const int step = (hi - lo + 63) / 64, at = lo + (lane + 1) * step - 1;
    const bool below = at < hi && sorted_off[min(at, n - 1)] < x;
    lo += __builtin_popcountll(__builtin_amdgcn_ballot_w64(below)) * step;
    hi = min(hi, lo + step - 1);
  }
  return lo;
}

// dM[j] += sum over every virtual weight that lands on slot j, in a fixed order: a workgroup has 64 * V consecutive slots, each wave takes every
// WAVES-th of the tiles that reach into them, in rank order, and the waves' fp64 sums are added in theirs.  Bound: the products, read once; the lanes of
// a wave read consecutive ones of a tile.  (One slot to eight lanes, each with tiles of its own, read them in pieces of 32 bytes, searched for every slot and
// divided 64-bit numbers: 41 tokens of 6336 x 7680 over 5.6 Mi slots 641 us.)
template <int V, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_dm_gather(MMArgs a, int splits, const float* __restrict__ G,
                                                          const int64_t* __restrict__ sorted_off,
                                                          const uint32_t* __restrict__ order, const int8_t* __restrict__ sgn,
                                                          float* __restrict__ dM) {
  __shared__ double s_sum[WAVES][64 * V];
  __shared__ uint32_t s_any[WAVES][64];          // bit v: slot 64 * v + lane has a weight
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t w0 = (int64_t)blockIdx.x * (64 * V), L = (int64_t)a.Z1 * a.Z2, plane = a.H * a.O;
  const int nT = (int)(a.nTx * a.nTy);
  const int first = count_below(sorted_off, nT, w0 - L + 1), end = count_below(sorted_off, nT, w0 + 64 * V);
  double total[V];
  uint32_t any = 0u;
#pragma unroll
  for (int v = 0; v < V; ++v) total[v] = 0.0;
  for (int q = first + wave; q < end; q += WAVES) {
    const uint32_t t = order[q];
    const int64_t p0 = w0 - sorted_off[q];
    const int64_t h0 = (int64_t)(t / (uint32_t)a.nTy) * a.Z1, c0 = (int64_t)(t % (uint32_t)a.nTy) * a.Z2;
    const double sign = (double)sgn[t];
    const float* from[V];
    bool have[V];
    float es[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int64_t p = p0 + 64 * v + lane;
      have[v] = p >= 0 && p < L;
      int64_t h, c;
      if (L < (1ll << 31)) {
        const uint32_t n = have[v] ? (uint32_t)p : 0u, r = n / (uint32_t)a.Z2;
        h = h0 + r;
        c = c0 + (n - r * (uint32_t)a.Z2);
      } else {
        const int64_t n = have[v] ? p : 0, r = n / a.Z2;
        h = h0 + r;
        c = c0 + (n - r * a.Z2);
      }
      have[v] = have[v] && h < a.H && c < a.O;
      from[v] = G + (have[v] ? h * a.O + c : 0);
      es[v] = a.hash.use_sign == 2 ? (float)elem_sign(a.hash, a.layer, (uint64_t)h, (uint64_t)c) : 1.f;
      any |= have[v] ? 1u << v : 0u;
    }
    double sum[V];
#pragma unroll
    for (int v = 0; v < V; ++v) sum[v] = 0.0;
#pragma unroll 4
    for (int s = 0; s < splits; ++s)
#pragma unroll
      for (int v = 0; v < V; ++v) sum[v] += (double)from[v][s * plane];
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (have[v]) total[v] += sign * (double)es[v] * sum[v];
  }
#pragma unroll
  for (int v = 0; v < V; ++v) s_sum[wave][64 * v + lane] = total[v];
  s_any[wave][lane] = any;
  __syncthreads();
  for (int i = threadIdx.x; i < 64 * V; i += 64 * WAVES) {
    double sum = 0.0;
    uint32_t some = 0u;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      sum += s_sum[w][i];
      some |= s_any[w][i & 63] >> (i >> 6);
    }
    if (w0 + i < a.m_size && (some & 1u)) dM[w0 + i] += (float)((double)a.lambda * sum);
  }
}

// Sum the per-split products and scatter them: one workgroup per (tile, block of rows of the tile).
// dM[offset + Z2*o1 + o2] += lambda * sign * sum_s G[s][x*Z1 + o1][y*Z2 + o2].
// One atomic per virtual weight instead of one per weight and split.  Needs Z2 % 4 == 0, O % 4 == 0.
__global__ __launch_bounds__(256) void k_dm_scatter(MMArgs a, int splits, int rows_per_wg,
                                                    const float* __restrict__ G, float* __restrict__ dM) {
  __shared__ int64_t s_off;
  __shared__ float s_scale;
  const int chunks = (a.Z1 + rows_per_wg - 1) / rows_per_wg;
  const int64_t tile = blockIdx.x / chunks;
  const int r_begin = (blockIdx.x % chunks) * rows_per_wg;
  const int x = (int)(tile / a.nTy), y = (int)(tile % a.nTy);
  if (threadIdx.x == 0) {
    s_off = block_offset(a.hash, a.layer, (uint64_t)x, (uint64_t)y);
    s_scale = a.lambda * (float)block_sign(a.hash, a.layer, (uint64_t)x, (uint64_t)y);
  }
  __syncthreads();
  const int64_t off = s_off;
  const float scale = s_scale;
  const int n = min(rows_per_wg, a.Z1 - r_begin) * a.Z2;
  const int64_t plane = a.H * a.O;
  // Consecutive lanes take consecutive weights: the loads coalesce and each wave's atomics fall in
  // as few cache lines as possible.  The workspace is read once: non-temporal loads, the splits of
  // one element in flight together.
  for (int e = threadIdx.x; e < n; e += 256) {
    const int r = r_begin + e / a.Z2, c = e % a.Z2;
    const int64_t h = (int64_t)x * a.Z1 + r, o = (int64_t)y * a.Z2 + c;
    if (h >= a.H || o >= a.O) continue;
    const float* g = G + h * a.O + o;
    auto ld = [&](int s) { return __builtin_nontemporal_load(g + (int64_t)s * plane); };
    float acc = 0.f;
    int s = 0;
    for (; s + 8 <= splits; s += 8) {
      const float v0 = ld(s), v1 = ld(s + 1), v2 = ld(s + 2), v3 = ld(s + 3);
      const float v4 = ld(s + 4), v5 = ld(s + 5), v6 = ld(s + 6), v7 = ld(s + 7);
      acc += ((v0 + v1) + (v2 + v3)) + ((v4 + v5) + (v6 + v7));
    }
    for (; s < splits; ++s) acc += ld(s);
    unsafeAtomicAdd(dM + off + (int64_t)a.Z2 * r + c, scale * acc);
  }
}

}  // namespace

// ---- split products through the workspace, then one scatter (the fast path of the ATOMIC mode when
// the caller provides a workspace): S*H*O floats.
int dm_ws_splits(const MMArgs& a) {
  if (a.hash.use_sign == 2) return 0;   // the scatter pass applies one sign per tile
  const int s = dm_pick_splits(((a.H + 255) / 256) * ((a.O + 127) / 128), a.I, 0);   // one atomic per weight whatever s
  return s > 1 ? s : 0;               // a single split gains nothing over direct atomics
}

size_t dm_ws_workspace_bytes(const MMArgs& a) {
  const int s = dm_ws_splits(a);
  return s ? (size_t)s * (size_t)a.H * (size_t)a.O * sizeof(float) : 0;
}

roast_status dm_ws_run(const MMArgs& a, const void* X, int64_t ldx, const void* dY, int64_t ldy, float* dM, void* ws,
                       hipStream_t s) {
  const int splits = dm_ws_splits(a);
  if (!splits) return ROAST_ERR_UNSUPPORTED;
  float* G = (float*)ws;
  roast_status st = mfma_mm_bwd_dM(a, X, ldx, dY, ldy, nullptr, G, splits, s);
  if (st != ROAST_OK) return st;      // UNSUPPORTED: the caller falls back to direct atomics
  const int rows_per_wg = a.Z2 >= 1024 ? 1 : 1024 / a.Z2;    // four weights per thread
  const int chunks = (a.Z1 + rows_per_wg - 1) / rows_per_wg;
  const int64_t blocks = a.nTx * a.nTy * chunks;
  if (blocks > 0x7fffffffll) return ROAST_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(k_dm_scatter, dim3((unsigned)blocks), dim3(256), 0, s, a, splits, rows_per_wg, G, dM);
  return hip_status(hipGetLastError());
}

int dm_det_splits(const MMArgs& a) {
  // A fixed function of the shape only, so that the summation order never depends on the machine.
  const int64_t tiles = ((a.O + 255) / 256) * ((a.H + 255) / 256);
  int64_t s = (512 + tiles - 1) / tiles;
  const int64_t max_s = (a.I + 511) / 512;
  if (s > max_s) s = max_s;
  if (s > 64) s = 64;
  if (s < 1) s = 1;
  return (int)s;
}

size_t dm_det_workspace_bytes(const MMArgs& a) {
  if (a.nTx * a.nTy > kMaxTilesDet) return 0;
  return det_layout(a, dm_det_splits(a)).total;
}

roast_status dm_det_run(const MMArgs& a, roast_dtype dt, const void* X, int64_t ldx, const void* dY, int64_t ldy,
                        float* dM, void* ws, hipStream_t s) {
  const int splits = dm_det_splits(a);
  const DetLayout l = det_layout(a, splits);
  char* base = (char*)ws;
  float* G = (float*)(base + l.g_off);
  int64_t* keys = (int64_t*)(base + l.key_off);
  int64_t* soff = (int64_t*)(base + l.soff_off);
  uint32_t* order = (uint32_t*)(base + l.order_off);
  int8_t* sgn = (int8_t*)(base + l.sgn_off);
  const int64_t nT = a.nTx * a.nTy;

  roast_status st = tile_index_launch(a, keys, sgn, s);
  if (st != ROAST_OK) return st;
  // (few tiles: one to sixteen lanes, for more waves)
  auto rank = [&](auto TILES) {
    constexpr int per_wg = 256 / kRankLanes * decltype(TILES)::value;
    hipLaunchKernelGGL((k_rank_tiles<decltype(TILES)::value>), dim3((unsigned)((nT + per_wg - 1) / per_wg)), dim3(256), 0, s, nT, keys, soff, order);
  };
  if (nT <= 4096) rank(std::integral_constant<int, 1>{});
  else if (nT <= 16384) rank(std::integral_constant<int, 2>{});
  else rank(std::integral_constant<int, 4>{});
  st = hip_status(hipGetLastError());
  if (st != ROAST_OK) return st;

  st = ROAST_ERR_UNSUPPORTED;
  if (dt == ROAST_BF16) st = mfma_mm_bwd_dM(a, X, ldx, dY, ldy, nullptr, G, splits, s);
  if (st == ROAST_ERR_UNSUPPORTED) st = generic_dm_launch(a, dt, X, ldx, dY, ldy, nullptr, G, splits, s);
  if (st != ROAST_OK) return st;

  // A small M is few workgroups: one value to a lane, and where a slot has many of them 16 waves to share its tiles (300 tokens of 512 x 1024 over 50000 slots,
  // 10 products to a slot, 16 waves 10.8 us; 8192 of 768 x 3072 over 47185, 750 to a slot, 39 where eight lanes to a slot took 57).
  auto gather = [&](auto V, auto WAVES) {
    constexpr int v = decltype(V)::value, w = decltype(WAVES)::value;
    hipLaunchKernelGGL((k_dm_gather<v, w>), dim3((unsigned)((a.m_size + 64 * v - 1) / (64 * v))), dim3(64 * w), 0, s, a, splits, G, soff, order, sgn, dM);
  };
  using std::integral_constant;
  if (a.m_size >= (256ll << 10)) gather(integral_constant<int, 4>{}, integral_constant<int, 4>{});
  else if ((double)a.H * (double)a.O * splits < 32.0 * (double)a.m_size) gather(integral_constant<int, 1>{}, integral_constant<int, 4>{});
  else gather(integral_constant<int, 1>{}, integral_constant<int, 16>{});
  return hip_status(hipGetLastError());
}

}  // namespace roast
