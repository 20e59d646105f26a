// ROAST lookup kernels: out[n, c*Z + o] = lambda * sign * M[offset(table, row, c) + o]
// (lookup equation of Section 4.1 of arXiv 2207.10702) and its scatter-add gradient (Section 4.3).
//
// HBM-bound streaming kernels.  Work item = one chunk of one lookup, numbered g = n*C + c, so that
// consecutive items are consecutive in `out`.  The integer work is done per lookup, not per chunk:
// the part of the hash that depends on (table, row) is computed once and the chunk index is walked
// incrementally.  With Z = 32 and VEC = 4, eight lanes serve a chunk and one step of a wave moves
// 1 KiB of contiguous output.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "roast_internal.hpp"

namespace roast {
namespace {

// 4 floats that are only 4-byte aligned in memory (chunk bases are arbitrary offsets into M).
struct __attribute__((packed, aligned(4))) f4u {
  float v[4];
};
typedef float vfloat4 __attribute__((ext_vector_type(4)));

// All chunk keys of one lookup: the row part of the hash once, then one cheap step per chunk.
// `walk` says whether the incremental walk is valid (chunks per row <= P); otherwise every chunk is
// hashed from scratch.  f(c, offset, sign) is called for c = 0 .. C-1.
template <typename F>
__device__ inline void for_each_chunk(const EmbedArgs& a, bool walk, uint64_t table, uint64_t row, F&& f) {
  if (walk) {
    const RowHash rh = row_hash(a.hash, table, row);
    ChunkWalk w;
    for (int64_t c = 0; c < a.C; ++c) {
      int64_t off; int sgn;
      w.get(a.hash, rh, &off, &sgn);
      f(c, off, sgn);
      w.next(a.hash);
    }
  } else {
    for (int64_t c = 0; c < a.C; ++c)
      f(c, block_offset(a.hash, table, row, (uint64_t)c), block_sign(a.hash, table, row, (uint64_t)c));
  }
}

// Pooled gradient: the bag of lookup n = the last b with bag_off[b] <= n (bag_off[0] == 0, so one
// exists; empty bags share their offset with the next one and are skipped by "last").  The result is
// clamped to [0, B-1] whatever the offsets hold, so a malformed offsets array cannot push a read out
// of dOut.  What it costs is one wait for memory after the other, 13 in a bisection of 8191 bags.  Four places are asked for first: the two where bags of equal
// sizes have it, which then is all, and one a little to each side, between which bags of about equal sizes have it; the rest is a bisection, of no more places than
// without them.  Over 100 pooled gradients of 200 to 10^6 lookups, against the bisection alone: bags of equal sizes 1.09 times faster with atomic adds and 1.05 in a fixed order,
// of random ones 1.00 to 1.05 and 0.99 to 1.02 (a call at worst 0.96; 0.88 where a lookup is one chunk and bags differ a thousandfold).  (A search at seven places a time after a wrong guess was slower than the bisection, 0.84 to 1.0: it asks for more lines.)
__device__ inline int64_t bag_of(const EmbedArgs& a, int64_t n) {
  const int64_t* __restrict__ bag_off = a.bag_off;
  const int64_t B = a.B;
  const int64_t guess = min(max((int64_t)(((double)n + 0.5) * a.bags_each), (int64_t)0), B - 1), near = (B >> 6) + 4;
  const int64_t below = max(guess - near, (int64_t)0), above = min(guess + 1 + near, B - 1);
  const int64_t at = bag_off[guess], next = bag_off[min(guess + 1, B - 1)], at_below = bag_off[below], at_above = bag_off[above];
  int64_t lo, hi;
  if (at <= n) {
    if (next > n || guess == B - 1) return guess;
    lo = at_above <= n ? above : guess + 1;
    hi = at_above <= n ? B : above;
  } else {
    lo = at_below <= n ? below : 0;
    hi = at_below <= n ? guess : max(below, (int64_t)1);
  }
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (bag_off[mid] <= n) lo = mid; else hi = mid;
  }
  return lo;
}
// row of dOut that lookup n takes its gradient from
__device__ inline int64_t grad_row(const EmbedArgs& a, int64_t n) { return a.bag_off ? bag_of(a, n) : n; }

// Streaming lookup / direct-atomic gradient.  A wave takes rows_wave lookups (64, fewer in a small call): each lane
// hashes the chunks of one lookup into the wave's LDS key list (offset | sign bit, 32-bit), then the wave walks the
// rows_wave*C chunks in order, LPI lanes per chunk, VEC floats per lane.
// VEC = 4 (forward only) requires Z % 4 == 0 and D % Z == 0 (then every chunk is full and out is 16-byte
// aligned per lane, given a 16-byte aligned base).  Needs |M| < 2^31 and C <= kMaxC.
constexpr int kMaxC = 16;

// slices > 1 (forward only; 2, 4 or 8): M is larger than one XCD's L2, so the gathered reads would
// keep missing it.  The workgroups of XCD group s (workgroups go to the 8 XCDs round-robin) then only
// serve the chunks whose offset lies in the s-th slice of M: every block of 4*rows_wave lookups is hashed by
// `slices` workgroups on different XCDs (hashing is cheap), each of which gathers from a part of M
// that stays in its L2 and writes its share of the output chunks.
template <int VEC, bool BWD>
__global__ __launch_bounds__(256) void k_embed(EmbedArgs a, int lpi_log2, int walk, const int64_t* __restrict__ rows,
                                               const uint32_t* __restrict__ tables, const float* __restrict__ M,
                                               float* __restrict__ out, const float* __restrict__ dOut,
                                               float* __restrict__ dM, int slices, int rows_wave) {
  extern __shared__ uint32_t s_keys[];           // [4 waves][64 * C] keys, then [4 waves][64 * C] selected chunk numbers (16 bit)
  __shared__ int64_t s_src[BWD ? 4 * 64 : 1];    // gradient row of each lookup
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int C = (int)a.C;
  uint32_t* keys = s_keys + wv * 64 * C;
  uint16_t* sel = reinterpret_cast<uint16_t*>(s_keys + 4 * 64 * C) + wv * 64 * C;
  const int per = 8 / slices;                    // consecutive lookup blocks per group of 8 workgroups
  const int slice = (int)(blockIdx.x & 7) / per;
  const int64_t lblock = slices == 1 ? (int64_t)blockIdx.x : (int64_t)(blockIdx.x >> 3) * per + (blockIdx.x & (per - 1));
  const int64_t wave = lblock * 4 + wv;
  const int64_t n0 = wave * rows_wave;
  if (n0 >= a.N) return;
  const int rows_here = (int)min((int64_t)rows_wave, a.N - n0);
  if (lane < rows_here) {
    const int64_t n = n0 + lane;
    if (BWD) s_src[wv * 64 + lane] = grad_row(a, n);
    for_each_chunk(a, walk != 0, tables[n], (uint64_t)rows[n], [&](int64_t c, int64_t off, int sgn) {
      keys[lane * C + c] = (uint32_t)off | (sgn < 0 ? 0x80000000u : 0u);
    });
  }
  // the wave reads back what its own lanes wrote: LDS operations of one wave complete in order
  const int lpi = 1 << lpi_log2;
  const int items_per_step = 64 >> lpi_log2;
  const int sub = lane & (lpi - 1);   // my position among the lanes serving one chunk
  const int which = lane >> lpi_log2; // which chunk of the step I serve
  int n_here = rows_here * C;
  const int64_t g0 = n0 * C;
  if (!BWD && slices > 1) {
    // order-preserving selection of this slice's chunks (wave-level: ballot + prefix count)
    const uint32_t lo = (uint32_t)(((int64_t)slice * a.m_size) / slices);
    const uint32_t hi = (uint32_t)(((int64_t)(slice + 1) * a.m_size) / slices);
    int base = 0;
    for (int j0 = 0; j0 < n_here; j0 += 64) {
      const int j = j0 + lane;
      const uint32_t off = j < n_here ? (keys[j] & 0x7fffffffu) : 0xffffffffu;
      const bool mine = j < n_here && off >= lo && off < hi;
      const unsigned long long mask = __ballot(mine);
      if (mine) sel[base + __popcll(mask & ((1ull << lane) - 1ull))] = (uint16_t)j;
      base += __popcll(mask);
    }
    n_here = base;
    if (n_here == 0) return;
  }
  auto chunk_at = [&](int idx) { return (!BWD && slices > 1) ? (int)sel[idx] : idx; };
  if constexpr (VEC == 4 && !BWD) {
    // Forward, full chunks: the gathered reads of M are latency-bound (L2 / memory-side cache), so
    // each wave keeps U chunks per lane group in flight before it stores any of them.
    constexpr int U = 4;                // chunks of a group of lanes whose loads are waited for together
    if (lpi * 4 == a.Z) {          // one 16-byte piece per lane and chunk (Z <= 256): the common case
      for (int j0 = 0; j0 < n_here; j0 += U * items_per_step) {
        vfloat4 v[U];
        int64_t ob[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int j = chunk_at(min(j0 + u * items_per_step + which, n_here - 1));
          const uint32_t key = keys[j];
          const float scale = (key & 0x80000000u) ? -a.lambda : a.lambda;
          const f4u m = *reinterpret_cast<const f4u*>(M + (key & 0x7fffffffu) + sub * 4);
          v[u] = vfloat4{scale * m.v[0], scale * m.v[1], scale * m.v[2], scale * m.v[3]};
          ob[u] = (g0 + j) * a.Z + sub * 4;      // D % Z == 0: chunk g starts at g*Z in the dense output
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (j0 + u * items_per_step + which < n_here) __builtin_nontemporal_store(v[u], reinterpret_cast<vfloat4*>(out + ob[u]));
      }
      return;
    }
  }
  for (int j0 = 0; j0 < n_here; j0 += items_per_step) {
    if (j0 + which >= n_here) continue;
    const int j = chunk_at(j0 + which);
    const uint32_t key = keys[j];
    const int64_t off = key & 0x7fffffffu;
    const float scale = (key & 0x80000000u) ? -a.lambda : a.lambda;
    const int64_t g = g0 + j;
    const int64_t n = g / C, c = g - n * C;
    const int len = (int)min((int64_t)a.Z, a.D - c * a.Z);   // last chunk of a row may be short
    const int64_t obase = (BWD ? s_src[wv * 64 + (int)(n - n0)] : n) * a.D + c * a.Z;
    for (int o = sub * VEC; o < len; o += lpi * VEC) {
      if constexpr (VEC == 4) {
        const f4u m = *reinterpret_cast<const f4u*>(M + off + o);
        const vfloat4 v = {scale * m.v[0], scale * m.v[1], scale * m.v[2], scale * m.v[3]};
        __builtin_nontemporal_store(v, reinterpret_cast<vfloat4*>(out + obase + o));
      } else {
        if (!BWD) {
          __builtin_nontemporal_store(scale * M[off + o], out + obase + o);
        } else {
          unsafeAtomicAdd(dM + off + o, scale * __builtin_nontemporal_load(dOut + obase + o));
        }
      }
    }
  }
}

// Fallback for huge M (offsets beyond 31 bits) or very many chunks per row: one thread per element.
template <bool BWD>
__global__ __launch_bounds__(256) void k_embed_elem(EmbedArgs a, const int64_t* __restrict__ rows,
                                                    const uint32_t* __restrict__ tables, const float* __restrict__ M,
                                                    float* __restrict__ out, const float* __restrict__ dOut,
                                                    float* __restrict__ dM) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= a.N * a.D) return;
  const int64_t n = e / a.D, i = e - n * a.D, c = i / a.Z, o = i - c * a.Z;
  const int64_t off = block_offset(a.hash, tables[n], (uint64_t)rows[n], (uint64_t)c);
  const float scale = a.lambda * (float)(block_sign(a.hash, tables[n], (uint64_t)rows[n], (uint64_t)c) *
                                         elem_sign(a.hash, tables[n], (uint64_t)rows[n], (uint64_t)i));
  if (!BWD) out[e] = scale * M[off + o];
  else unsafeAtomicAdd(dM + off + o, scale * dOut[grad_row(a, n) * a.D + i]);
}

__global__ __launch_bounds__(256) void k_chunk_index(EmbedArgs a, int walk, const int64_t* __restrict__ rows,
                                                     const uint32_t* __restrict__ tables, int64_t* __restrict__ off,
                                                     int8_t* __restrict__ sgn) {
  const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= a.N) return;
  for_each_chunk(a, walk != 0, tables[n], (uint64_t)rows[n], [&](int64_t c, int64_t o, int s) {
    off[n * a.C + c] = o;
    sgn[n * a.C + c] = (int8_t)s;
  });
}

// Pooled forward: out[b, :] = lambda * sum over the lookups n of bag b of sign_n * M[offset_n(c) + o].
// A workgroup owns `bags_wg` consecutive bags, i.e. one contiguous range of lookups.  It works in
// windows of at most `win` lookups: every lookup of the window is hashed once (one thread per
// lookup, all its chunks, keys to LDS), then each thread walks the part of its bag that lies in the
// window and adds its piece (VEC floats of one chunk) of every row -- gathered reads of M, served by
// L2.  Sums run in lookup order, in fp64, so the result does not depend on the launch shape.
// VEC = 4 requires Z % 4 == 0 and D % 4 == 0 (a piece never straddles a chunk or the row end).
template <int VEC>
__global__ __launch_bounds__(256) void k_embed_bag_fwd(EmbedArgs a, int walk, int tpb, int bags_wg, int win,
                                                       const int64_t* __restrict__ rows,
                                                       const uint32_t* __restrict__ tables,
                                                       const float* __restrict__ M, float* __restrict__ out) {
  extern __shared__ uint32_t s_bag_keys[];       // [win * C]
  const int C = (int)a.C;
  const int64_t b0 = (int64_t)blockIdx.x * bags_wg;
  const int64_t b1 = min(a.B, b0 + bags_wg);
  auto clampN = [&](int64_t v) { return min(max(v, (int64_t)0), a.N); };
  const int64_t n_begin = clampN(a.bag_off[b0]);
  const int64_t n_end = max(n_begin, clampN(a.bag_off[b1]));
  const int bl = threadIdx.x / tpb, tl = threadIdx.x % tpb;
  const int64_t b = b0 + bl;
  const bool active = bl < bags_wg && b < b1;
  int64_t my_begin = 0, my_end = 0;
  if (active) {
    my_begin = min(max(clampN(a.bag_off[b]), n_begin), n_end);
    my_end = min(max(clampN(a.bag_off[b + 1]), my_begin), n_end);
  }
  const int pieces = (int)((a.D + VEC - 1) / VEC);
  for (int p0 = 0; p0 < pieces; p0 += tpb) {           // one pass unless a row has more pieces than tpb
    const int piece = p0 + tl;
    const bool live = active && piece < pieces;
    const int c = live ? (piece * VEC) / a.Z : 0, o = live ? (piece * VEC) % a.Z : 0;
    double acc[VEC];   // a bag may hold thousands of rows: fp64 sums keep the result within one fp32 rounding
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
    for (int64_t w0 = n_begin; w0 < n_end; w0 += win) {   // uniform trip count for the workgroup
      const int64_t w1 = min(n_end, w0 + win);
      __syncthreads();                                    // the previous window's keys are no longer needed
      for (int64_t n = w0 + threadIdx.x; n < w1; n += 256)
        for_each_chunk(a, walk != 0, tables[n], (uint64_t)rows[n], [&](int64_t cc, int64_t off, int sgn) {
          s_bag_keys[(n - w0) * C + cc] = (uint32_t)off | (sgn < 0 ? 0x80000000u : 0u);
        });
      __syncthreads();
      if (!live) continue;
      const int64_t lo = max(my_begin, w0), hi = min(my_end, w1);
      constexpr int U = 4;                // chunks of a group of lanes whose loads are waited for together
      for (int64_t n = lo; n < hi; n += U) {
        float m[U][VEC];
        float sg[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int64_t nn = min(n + u, hi - 1);
          const uint32_t key = s_bag_keys[(nn - w0) * C + c];
          sg[u] = (n + u < hi) ? ((key & 0x80000000u) ? -1.f : 1.f) : 0.f;
          const float* src = M + (key & 0x7fffffffu) + o;
          if constexpr (VEC == 4) {
            const f4u t = *reinterpret_cast<const f4u*>(src);   // 4-byte aligned: chunk bases are arbitrary
#pragma unroll
            for (int v = 0; v < 4; ++v) m[u][v] = t.v[v];
          } else {
            m[u][0] = src[0];
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int v = 0; v < VEC; ++v) acc[v] += (double)(sg[u] * m[u][v]);
      }
    }
    if (live) {
      float* dst = out + b * a.D + (int64_t)piece * VEC;
      if constexpr (VEC == 4) {
        const double l = (double)a.lambda;
        const vfloat4 r = {(float)(l * acc[0]), (float)(l * acc[1]), (float)(l * acc[2]), (float)(l * acc[3])};
        *reinterpret_cast<vfloat4*>(dst) = r;
      } else {
        dst[0] = (float)((double)a.lambda * acc[0]);
      }
    }
  }
}

// Fallback for huge M or very many chunks per row: one thread per output element.
__global__ __launch_bounds__(256) void k_embed_bag_fwd_elem(EmbedArgs a, const int64_t* __restrict__ rows,
                                                            const uint32_t* __restrict__ tables,
                                                            const float* __restrict__ M, float* __restrict__ out) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= a.B * a.D) return;
  const int64_t b = e / a.D, i = e - b * a.D, c = i / a.Z, o = i - c * a.Z;
  const int64_t n0 = min(max(a.bag_off[b], (int64_t)0), a.N), n1 = min(max(a.bag_off[b + 1], n0), a.N);
  double acc = 0.0;
  for (int64_t n = n0; n < n1; ++n) {
    const int64_t off = block_offset(a.hash, tables[n], (uint64_t)rows[n], (uint64_t)c);
    acc += (double)((float)(block_sign(a.hash, tables[n], (uint64_t)rows[n], (uint64_t)c) *
                            elem_sign(a.hash, tables[n], (uint64_t)rows[n], (uint64_t)i)) * M[off + o]);
  }
  out[e] = (float)((double)a.lambda * acc);
}

inline int walk_ok(const EmbedArgs& a) { return (uint64_t)a.C <= a.hash.P.d ? 1 : 0; }

template <bool BWD>
roast_status launch_embed(const EmbedArgs& a, const int64_t* rows, const uint32_t* tables, const float* M,
                          float* out, const float* dOut, float* dM, hipStream_t s) {
  // (the chunk kernels carry one sign per chunk: per-element signs take the per-element kernel)
  if (a.m_size >= (1ll << 31) || a.C > kMaxC || a.hash.use_sign == 2) {
    const int64_t blocks = (a.N * a.D + 255) / 256;
    if (blocks > 0x7fffffffll) return ROAST_ERR_UNSUPPORTED;
    hipLaunchKernelGGL((k_embed_elem<BWD>), dim3((unsigned)blocks), dim3(256), 0, s, a, rows, tables, M, out, dOut, dM);
    return hip_status(hipGetLastError());
  }
  // The gradient takes one value per lane: the chip serves atomic adds by the 64-byte piece of a wave
  // instruction (18.7 G pieces/s, however many of its 16 slots are added to), so an instruction has to
  // cover consecutive slots.  Four values per lane -- slots 16 bytes apart in one instruction -- ran at
  // 0.08 T adds/s instead of 0.2-0.3: 62 400 chunks of 32 took 54 us, now 18.
  const bool vec4 = !BWD && (a.Z % 4 == 0) && (a.D % a.Z == 0) && (((uintptr_t)out & 15) == 0);
  const int per_lane = vec4 ? 4 : 1;
  int lpi_log2 = 0;
  while ((1 << lpi_log2) < 64 && (int64_t)(1 << lpi_log2) * per_lane < a.Z) ++lpi_log2;
  // forward over an M that does not fit one XCD's L2 (4 MiB): four slices (measured on a 5 MiB M:
  // 171 us unsliced, 158 / 144 / 189 us with 2 / 4 / 8 slices -- every slice hashes all lookups),
  // eight once a quarter is too large; not for small calls, nor once even an eighth does not fit
  int slices = 1;
  if (!BWD && vec4 && a.N * a.C >= 65536) {
    const int64_t bytes = a.m_size * 4, fit = 3584 * 1024;
    slices = bytes <= fit ? 1 : bytes <= 4 * fit ? 4 : bytes <= 8 * fit ? 8 : 1;
  }
  // Lookups per wave: 64 (one per lane) once the call fills the chip with full waves; below that fewer,
  // so that a small call spreads over up to 8192 waves (32 per CU) instead of walking 64 lookups'
  // chunks one group after the other in a few waves -- but never fewer than one step of the wave
  // serves (64 >> lpi_log2 chunks).  2028 lookups of 8 chunks, gradient: 32 -> 14 us.  With slices a wave keeps
  // 64: it hashes all of its lookups for its slice's share of their chunks, a few of which would be left (in us, 64 and
  // fewer: 30000 lookups of 4 chunks of 32, four slices 9.1 and 22.9; 66000 of one of 128, eight slices 10.0 and 20.8; 213000 of 4 21.8 and 25.6).
  int rows_wave = 64;
  while (slices == 1 && rows_wave > 1 && (a.N + rows_wave / 2 - 1) / (rows_wave / 2) <= 8192 && (rows_wave / 2) * a.C >= (64 >> lpi_log2)) rows_wave /= 2;
  const int64_t waves = (a.N + rows_wave - 1) / rows_wave;
  int64_t blocks = (waves + 3) / 4;
  if (slices > 1) blocks = (blocks + 8 / slices - 1) / (8 / slices) * 8;
  if (blocks > 0x7fffffffll) return ROAST_ERR_UNSUPPORTED;
  const dim3 g((unsigned)blocks), b(256);
  const size_t lds = (size_t)4 * 64 * a.C * (sizeof(uint32_t) + sizeof(uint16_t));
  if constexpr (!BWD) {
    if (vec4) {
      hipLaunchKernelGGL((k_embed<4, false>), g, b, lds, s, a, lpi_log2, walk_ok(a), rows, tables, M, out, dOut, dM, slices, rows_wave);
      return hip_status(hipGetLastError());
    }
  }
  hipLaunchKernelGGL((k_embed<1, BWD>), g, b, lds, s, a, lpi_log2, walk_ok(a), rows, tables, M, out, dOut, dM, slices, rows_wave);
  return hip_status(hipGetLastError());
}

// ---------------------------------------------------------------------------------------------
// Bucketed gradient: fp32 global atomics top out near 0.3 T adds/s on this chip, an order of
// magnitude short of what streaming dOut needs, so the scatter-add is reorganised by destination.
//   1. route:  every lookup is hashed once; each of its chunks is appended to the list of the bucket
//              (R consecutive slots of M) its offset falls in.  A workgroup ranks its chunks inside
//              each bucket with LDS counters, reserves list space with one global add per bucket,
//              and writes every entry to reserved base + rank.  Lists have a fixed capacity; an entry that finds its list full
//              goes behind the lists, and a chunk that finds no room there either straight into dM with global atomics.
//   2. accum:  a workgroup owns a part of a bucket's slots, in an fp64 LDS image.  It reads the bucket's list (and what was
//              spilled), sorts the entries that touch its slots by where they start, adds the chunks of dOut that start at the
//              same slot in registers and these sums to the image, and hands the image to dM: one add per slot and workgroup.
// Needs Z % 4 == 0, D % Z == 0, C <= kMaxC, |M| < 2^31 and at most kMaxBuckets buckets of at most
// kMaxR slots by this reckoning; other shapes use the direct atomic kernel above.
constexpr int kSeg = 8192;          // list entries per accumulate workgroup, where lists are longer than that on average
constexpr int kListSlack = 8192;    // list capacity beyond twice the mean load, for every 4096 slots
constexpr int kAccThreads = 512;
constexpr int kPass = 4096;         // list entries that an accumulate workgroup sorts at a time, by the slot they start at
constexpr int kMaxBuckets = 2048;   // of 4096 slots (8192 beyond 8 Mi): what the lists' room is reckoned by
constexpr int kMaxR = 8192;
constexpr int kRouteItems = 8192;   // chunks per route workgroup (lookups per workgroup = kRouteItems / C)
constexpr int kRouteThreads = 512;
constexpr uint32_t kNoEntry = 0x7fffffffu;   // key of a list entry that touches nothing (beyond any M that is routed)

struct BucketPlan {
  bool ok;
  int64_t n_items;
  int s_log2;            // a bucket has R = g << s_log2 slots
  uint32_t g;
  int nb;                // number of buckets
  size_t list_off, total;   // the cursors come first
  int R() const { return (int)(g << s_log2); }
};

// Buckets of 4096 slots, and no more than 256 of them, or 512 of a larger M.  Few: a route workgroup waits for one reservation in
// each bucket, and the list of a bucket with popular rows has room for less (of 6.8 M chunks over 3 Mi slots, 512 lists spill 84 000 that
// every workgroup then looks through: 516 us, with 256 303).  But a list's workgroups that share out the slots (AccPlan) read all of
// it, more of them the longer a bucket is, which counts more the shorter a chunk is: from 2 Mi slots on with chunks of 16 (13.6 M
// chunks over 6 Mi: 256 buckets 576 us, 512 487), from 4 Mi on with 32 (6.8 M over 6 Mi 327 and 294, but 6.2 M over 4 Mi with a fixed order 393 and 461);
// where a list takes more than one pass (0.63 M chunks of 16 over 3.9 Mi with a fixed order 70.5 and 75).
inline BucketPlan bucket_plan(const EmbedArgs& a) {
  BucketPlan p{};
  p.n_items = a.N * a.C;
  int r = 12;
  while ((1 << r) < kMaxR && ((a.m_size + (1ll << r) - 1) >> r) > kMaxBuckets) ++r;
  const int64_t room_buckets = (a.m_size + (1ll << r) - 1) >> r;
  p.ok = (a.Z % 4 == 0) && (a.D % a.Z == 0) && a.m_size < (1ll << 31) && p.n_items < (1ll << 31) && a.Z <= 1024 &&
         a.C <= kMaxC && a.B * a.C < (1ll << 31) &&  // (B = 0 unless pooled)
         a.hash.use_sign != 2 &&                     // list entries carry one sign per chunk
         room_buckets <= kMaxBuckets;
  if (!p.ok) return p;
  const int64_t most = a.m_size > std::min(a.Z, 32) * (128ll << 10) && p.n_items > 256 * kPass ? 512 : 256;
  const int64_t want = std::max<int64_t>(4096, (a.m_size + most - 1) / most);   // (at most 32768)
  while (((want - 1) >> p.s_log2) + 1 > 8) ++p.s_log2;
  p.g = (uint32_t)(((want - 1) >> p.s_log2) + 1);
  p.nb = (int)((a.m_size + p.R() - 1) / p.R());
  // room for twice the entries and some: uniform hashing stays far below, skewed ids mostly too
  auto up = [](size_t v) { return (v + 255) / 256 * 256; };
  p.list_off = up((size_t)(p.nb + 1) * 4);
  p.total = up((size_t)room_buckets * 4) + up((size_t)room_buckets * (2 * (p.n_items / room_buckets) + kListSlack) * 8);
  return p;
}

constexpr int kPer = kPass / kAccThreads;
constexpr int U = 4;                // chunks of a group of lanes whose loads are waited for together
// groups of lanes that hold a chunk, in a wave; places for the sorted entries and what fills up the groups' shares
__host__ __device__ constexpr int acc_groups(int Z) { return Z >= 256 ? 1 : 64 / (Z / 4); }
__host__ __device__ constexpr int acc_sorted(int Z) { return kPass + 2 * U * acc_groups(Z) * (kAccThreads / 64); }
__host__ __device__ constexpr int acc_span(int slots, int Z) { return (slots + 2 * Z + 15) / 16 * 16; }
inline size_t acc_lds(int slots, int Z) { return (size_t)acc_span(slots, Z) * (8 + 2) + (size_t)acc_sorted(Z) * 6; }

// How the lists are laid out and an accumulate launch shares out the work.
struct AccPlan {
  int s_log2;            // buckets, see BucketPlan
  uint32_t g, mu;        // (mu: 2^32 / g, rounded up)
  int nb;
  int q_log2;            // a workgroup owns R >> q_log2 slots
  uint32_t cap;          // of a list
  uint32_t spill_cap;    // of what lies behind the lists: the entries that found theirs full, where every workgroup looks for its own
  // A list is read by several workgroups to a part, at most `most`: as many as `per` times its entries, of which those up to the
  // mean load count `share` each (the nearest number, or the next above: `up` is a half or nearly one)
  uint32_t mean, most;
  float share, per, up;
  float less;            // the last of three and more is by that much of a length shorter than the others
  bool owned;            // (fixed point) every slot has one workgroup that sees all of its chunks and writes dM
  bool take_max;         // ... and the route kernel takes the largest |dOut|
  bool sampled;          // ... of a sample of dOut: see local_pbits
  __host__ __device__ int R() const { return (int)(g << s_log2); }
  __host__ __device__ uint32_t segments(uint32_t count) const {
    const uint32_t usual = count < mean ? count : mean, n = (uint32_t)(((float)usual * share + (float)(count - usual)) * per + up);
    return n < 1u ? 1u : n > most ? most : n;
  }
  // entries to a segment; a little more than exactly that, so that they are never too few.  (One way or the other to divide decides
  // whether the kernels with 128 registers keep some in scratch, which costs a launch 2 to 3 us: 8191 x 26 pooled 34.9 -> 31.9.)
  template <bool FIXED>
  __device__ uint32_t length(uint32_t entries, uint32_t nseg) const {
    if constexpr (FIXED) return (entries + nseg - 1) / nseg;
    const float n = (float)nseg - (nseg < 3u ? 0.f : less);
    return (uint32_t)((float)entries * __builtin_amdgcn_rcpf(n) * 1.000001f) + 1u;
  }
  __device__ uint32_t bucket(uint32_t off) const { return __umulhi(off >> s_log2, mu); }   // exact: off < 2^31, g <= 8
};

// Every fp32 add to dM rounds, so there is one per slot and kSeg chunks of the 4096 slots around it, or one in all where those get
// fewer on average.  In a bucket of more slots the mean load is spread evenly over them, what a list has beyond it starts at a
// few popular rows and may be all in one place.  With a workgroup for every kSeg entries of a list instead, 6.2 M chunks over 4 Mi
// slots took 250 us and were 4.6e-8 off the exact gradient; this takes 258 and is 2.9e-8 off; 6.8 M over 1.28 M 238 and 4.8e-8, 238 and
// 4.3e-8.  From 4 Mi slots on popular rows are split too where lists are short: one workgroup to a list takes 306 us instead of 258 (2.6e-8).
// Fixed point is exact however it is cut: one pass of the sort, where chunks are long enough and a part is a whole bucket
// (6.8 M chunks of 32 over 0.1 Mi slots 362 -> 354 us, 3.4 M 218 -> 204, of 64 363 -> 337; 6.8 M of 32 over 0.6 Mi 349 -> 356, of 16 535 -> 548).
inline AccPlan acc_plan(const EmbedArgs& a, const BucketPlan& p, bool fixed) {
  AccPlan k{};
  k.s_log2 = p.s_log2; k.g = p.g; k.nb = p.nb;
  k.mu = (uint32_t)(((1ull << 32) + p.g - 1) / p.g);
  const int64_t room = (int64_t)((p.total - p.list_off) / 8), mean = p.n_items / p.nb;
  k.share = fixed ? 1.f : 4096.f / (float)k.R();
  k.less = !fixed && k.R() > 4096 && a.Z >= 32 ? 0.3f : 0.f;   // (the last third of 750 workgroups in 512 places runs alone: 1.28 M slots 246 -> 238 us, 2 Mi 249 -> 244)
  // (fixed point: one workgroup while that costs less than an accumulator of all of M to clear and to add up)
  const bool many = fixed ? mean > kSeg / 2 * 3 : mean * 4096 > (int64_t)kSeg * k.R() || a.m_size >= (4ll << 20);
  k.owned = fixed && !many;
  k.take_max = k.owned && a.B <= 4 * a.N;   // (beyond that few workgroups would read a large dOut: 70 000 chunks of 32, 2 M bags 197 us, 95 with a launch for it; 0.4 M 70 and 68, 0.14 M 42 and 46)
  // Skew: lists have room for twice their mean load and half of what there is beyond that, the rest is spill.  Owned slots:
  // lists have room for the mean load and all there is beyond twice that, any number of entries can be spilled.
  k.sampled = k.take_max && a.bag_off == nullptr;   // (pooled: a row of dOut that no chunk refers to counts too)
  k.cap = (uint32_t)((k.owned ? room - p.n_items : p.n_items + room / 2) / p.nb);
  k.spill_cap = (uint32_t)std::min<int64_t>(room - (int64_t)p.nb * k.cap, 0x7fffffff);
  const int seg = fixed && k.R() == 4096 && a.Z >= 32 ? kPass : kSeg;
  k.per = 1.f / (float)seg; k.up = fixed || k.R() == 4096 ? 1.f - k.per : 0.5f;
  k.mean = (uint32_t)mean; k.most = many ? ~0u : 1u;
  k.most = k.segments(k.cap);
  const int64_t wgs = p.nb * (many ? std::max<int64_t>(1, (int64_t)((float)mean * k.share) / kSeg) : 1);
  // parts: so that a CU holds two workgroups, and a workgroup for most of the places (512: two to a CU)
  while (acc_lds(k.R() >> k.q_log2, a.Z) > 80 * 1024 || (k.q_log2 < 3 && wgs << k.q_log2 < 400 && k.q_log2 < k.s_log2 && (int64_t)a.Z << (k.q_log2 + 1) <= k.R())) ++k.q_log2;
  return k;
}

// cursors (the last one counts the spilled entries) and, unless it is null, the scale record
__global__ __launch_bounds__(256) void k_embed_route_init(int nb, uint32_t* __restrict__ cursor, uint32_t* __restrict__ record) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i <= nb) cursor[i] = 0u;
  if (record && i < 4) record[i] = 0u;
}

__global__ __launch_bounds__(256) void k_embed_zero(uint32_t* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// ---- fixed-point accumulation (the DETERMINISTIC mode).  Integer addition is associative, so sums
// of fixed-point values do not depend on the order in which atomics land.  Every contribution
// v = fl(+-lambda * dOut[..]) (one fp32 product, the same rounding as the atomic mode) is converted
// to a multiple of 2^-shift chosen from the largest |dOut| of the call such that |v| * 2^shift <
// 2^pbits and pbits + ceil(log2(number of chunks)) <= 62: no sum can overflow 64 bits, and the
// quantum is at least 2^-31 of the largest contribution (finer than fp32 for any realistic batch).
struct FixedScale {
  uint32_t absmax_bits;   // max over dOut of the bits of |x| (order-independent: integer max)
  uint32_t not_finite;    // (a sample only) a workgroup has found an Inf or NaN and makes all of dM NaN
  uint32_t pad[2];
};

__device__ inline uint32_t absmax4(const vfloat4& x) {
  return max(max(__float_as_uint(x.x) & 0x7fffffffu, __float_as_uint(x.y) & 0x7fffffffu), max(__float_as_uint(x.z) & 0x7fffffffu, __float_as_uint(x.w) & 0x7fffffffu));
}
__device__ inline uint32_t wave_max(uint32_t m) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d, 64));
  return m;
}

constexpr int kMaxThreads = 512;
__global__ __launch_bounds__(kMaxThreads) void k_embed_absmax(const float* __restrict__ dOut, int64_t n,
                                                      FixedScale* __restrict__ fs) {
  // streaming read: 16-byte loads, eight of them in flight per thread (a scalar grid-stride loop was
  // latency-bound at a third of this rate); head and tail that are not 16-byte aligned go scalar
  uint32_t m = 0u;
  const int64_t tid = (int64_t)blockIdx.x * kMaxThreads + threadIdx.x;
  const int64_t head = min(n, (int64_t)((16 - ((uintptr_t)dOut & 15)) & 15) / 4);   // floats before the first aligned one
  const int64_t nvec = (n - head) / 4;
  const vfloat4* v = reinterpret_cast<const vfloat4*>(dOut + head);
  // a workgroup takes contiguous 64 KiB pieces (8 x 512 lanes x 16 bytes), round-robin over the grid
  constexpr int U = 8;
  const int64_t piece = (int64_t)U * kMaxThreads;
  for (int64_t p0 = (int64_t)blockIdx.x * piece; p0 < nvec; p0 += (int64_t)gridDim.x * piece) {
    vfloat4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = min(p0 + u * kMaxThreads + threadIdx.x, nvec - 1);      // clamped: max is idempotent
      x[u] = __builtin_nontemporal_load(v + i);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) m = max(m, absmax4(x[u]));
  }
  if (tid < head) m = max(m, __float_as_uint(dOut[tid]) & 0x7fffffffu);
  const int64_t tail0 = head + 4 * nvec;
  if (tail0 + tid < n) m = max(m, __float_as_uint(dOut[tail0 + tid]) & 0x7fffffffu);
  m = wave_max(m);
  __shared__ uint32_t s_m[kMaxThreads / 64];
  if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = m;
  __syncthreads();
  // Atomics on one address complete one after the other (12 ns each: one per wave of 2048 workgroups
  // took 100 us whatever the size of dOut): one per workgroup, none where the maximum found
  // so far is as large already, and no more workgroups than the loads of two to a CU need (all of them end together where
  // dOut is small: 38 MB took 28 us with 2048).
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 0; w < kMaxThreads / 64; ++w) m = max(m, s_m[w]);
    if (m > __hip_atomic_load(&fs->absmax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&fs->absmax_bits, m);
  }
}

// 2^shift as a double; NaN when dOut holds an Inf or NaN (the result is then NaN everywhere).
__device__ inline double fixed_scale(uint32_t bits, float lambda, int pbits) {
  if (bits >= 0x7f800000u) return __longlong_as_double(0x7ff8000000000000ll);
  const float bound = fabsf(lambda) * __uint_as_float(bits);   // every |contribution| <= bound
  if (!(bound > 0.f)) return 1.0;
  if (!(bound < __uint_as_float(0x7f800000u))) return __longlong_as_double(0x7ff8000000000000ll);
  int ex;
  frexpf(bound, &ex);                                           // bound < 2^ex
  return ldexp(1.0, pbits - ex);
}
__device__ inline double fixed_scale(const FixedScale* fs, float lambda, int pbits) { return fixed_scale(fs->absmax_bits, lambda, pbits); }

// Where every slot has one workgroup that sees all of its chunks, the scale only has to allow for those chunks, and each workgroup
// takes its own: from the largest magnitude of a sample of dOut, the same one in every run, with up to 6 bits to spare.  A workgroup that
// meets a chunk beyond that starts over with its own largest.  So dOut is read once, not twice (10007 x 26 lookups of 128 values 87 -> 69 us).
// The chunks are counted by the places asked for in the bucket's list, whether it had room for them or not: that is the
// same number in every run, where how many are found behind the lists is not (a chunk that two full lists ask for is there once).
// The bits to spare are those that these chunks, no more than all of the call, leave (at least one: fixed_pbits leaves a bit for the sign
// and rounds up): the quantum is not larger than that of the largest |dOut| of the call and all chunks.
__device__ inline int local_pbits(uint32_t chunks) { return min(50, (int)__builtin_clz(chunks | 1u) + 31); }   // (chunks * 2^pbits < 2^63; 50: fixed_raw)
__device__ inline uint32_t sample_limit(uint32_t bits, float lambda, int spare) {
  if (bits >= 0x7f800000u) return 0xffffffffu;                  // (everything is NaN already)
  const float l = ldexpf(__uint_as_float(bits), spare);
  return fabsf(lambda) * l < __uint_as_float(0x7f800000u) ? __float_as_uint(l) : bits;   // (no product may overflow unseen)
}
__device__ inline int local_spare(int pbits, int pbits_all) { return min(pbits - pbits_all, 6); }

__device__ inline unsigned long long to_fixed(float v, double scale) {
  return (unsigned long long)__double2ll_rn((double)v * scale);
}

// The same for values below 2^51 (where chunks are routed: pbits of a call <= 45, of a workgroup <= 50), in sums: adding 1.5 * 2^52 rounds to a whole number,
// which the low bits hold; the sum of n of them is too large by n times this constant.
constexpr double kFixedMagic = 6755399441055744.0;
__device__ inline unsigned long long fixed_raw(float v, double scale) {
  return (unsigned long long)__double_as_longlong(fma((double)v, scale, kFixedMagic));
}
__device__ inline unsigned long long fixed_sum(unsigned long long raw, uint32_t n) {
  return raw - ((unsigned long long)(n * 0x43380000u) << 32);
}

inline int fixed_pbits(int64_t n_items) {
  int lg = 0;
  while ((1ll << lg) < n_items + 1) ++lg;
  return 62 - lg;
}

// One thread per element: any shape, 64-bit integer atomics straight into the accumulator.
__global__ __launch_bounds__(256) void k_embed_fixed_elem(EmbedArgs a, int pbits, const int64_t* __restrict__ rows,
                                                          const uint32_t* __restrict__ tables,
                                                          const float* __restrict__ dOut, const FixedScale* fs,
                                                          unsigned long long* __restrict__ acc) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= a.N * a.D) return;
  const double scale = fixed_scale(fs, a.lambda, pbits);
  const int64_t n = e / a.D, i = e - n * a.D, c = i / a.Z, o = i - c * a.Z;
  const int64_t off = block_offset(a.hash, tables[n], (uint64_t)rows[n], (uint64_t)c);
  const float sc = a.lambda * (float)(block_sign(a.hash, tables[n], (uint64_t)rows[n], (uint64_t)c) *
                                      elem_sign(a.hash, tables[n], (uint64_t)rows[n], (uint64_t)i));
  atomicAdd(acc + off + o, to_fixed(sc * dOut[grad_row(a, n) * a.D + i], scale));
}

__global__ __launch_bounds__(256) void k_embed_fixed_finish(int64_t m_size, float lambda, int pbits, const FixedScale* fs,
                                                            const unsigned long long* __restrict__ acc,
                                                            float* __restrict__ dM) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= m_size) return;
  const double scale = fixed_scale(fs, lambda, pbits);
  if (scale != scale) { dM[i] += __uint_as_float(0x7fc00000u); return; }
  const long long v = (long long)acc[i];
  if (v != 0) dM[i] += (float)((double)v / scale);
}

// Largest magnitude of the 16-byte pieces first .. end of v.  (A launch of its own takes 34 us on 133 MB, this 27 as a step of the
// route kernel, whose workgroups do not need the answer: entries that find no list are spilled, not added.)
__device__ inline uint32_t absmax_of(const vfloat4* __restrict__ v, int64_t first, int64_t end, int threads) {
  uint32_t m = 0u;
  constexpr int U = 8;
  for (int64_t i0 = first + threadIdx.x; i0 < end; i0 += (int64_t)U * threads) {
    vfloat4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = v[min(i0 + (int64_t)u * threads, end - 1)];        // (clamped: max is idempotent)
#pragma unroll
    for (int u = 0; u < U; ++u) m = max(m, absmax4(x[u]));
  }
  return wave_max(m);
}

// This thread's piece of a sample of them: a 128-byte line for every eight threads, evenly spaced, but each a line further on in its share of them: else whole rows to
// a share would give every line the same columns, and rows whose other columns are larger would start over (N = 262144, D = 128, three quarters of the columns 1000 times
// as large as the first: 83 -> 58 us).
__device__ inline vfloat4 sample_of(const vfloat4* __restrict__ v, int64_t first, int64_t end, int threads) {
  const uint32_t line = threadIdx.x / 8, share = (uint32_t)(end - first) / (uint32_t)(threads / 8);
  return v[min(first + share * line + (share >= 8u ? line % (share / 8u) * 8u : 0u) + threadIdx.x % 8, end - 1)];
}

// entry = (chunk number g, key); key = offset | (negative sign << 31).  A workgroup waits in turn for the ids, for the
// reservations and (pooled) for the bags of its lookups; what it can do without the answer it does meanwhile.
template <bool FIXED>
__global__ __launch_bounds__(kRouteThreads) void k_embed_route(EmbedArgs a, AccPlan k, int walk, int items,
                                                     const int64_t* __restrict__ rows,
                                                     const uint32_t* __restrict__ tables, uint32_t* __restrict__ cursor,
                                                     uint2* __restrict__ list, const float* __restrict__ dOut,
                                                     float* __restrict__ dM, int pbits, FixedScale* fs,
                                                     unsigned long long* __restrict__ acc) {
  extern __shared__ __attribute__((aligned(16))) uint32_t s_route[];
  const int nb = k.nb;
  const uint32_t cap = k.cap;
  const int C = (int)a.C;
  const int rows_wg = items / C;
  uint32_t* s_key = s_route;                                       // [items]
  uint16_t* s_pos = reinterpret_cast<uint16_t*>(s_key + items);   // [items] rank inside (workgroup, bucket)
  uint32_t* hist = s_key + items + items / 2;                      // [nb]  chunks of this workgroup per bucket
  uint32_t* gbase = hist + nb;                                     // [nb]  reserved position in the bucket's global list
  uint32_t* pre = gbase + nb;                                      // [nb]  chunks of this workgroup in the buckets before
  uint16_t* s_ord = reinterpret_cast<uint16_t*>(pre + nb);         // [items] chunk index by (bucket, rank)
  const bool twice = FIXED && k.owned;                             // chunks that reach into the next bucket go into its list too
  uint32_t* s_over = reinterpret_cast<uint32_t*>(s_ord + (twice ? 2 * items : items));   // [items] (twice) those | rank there << 16
  uint32_t* s_src = s_over + (twice ? items : 0);                  // [rows_wg] gradient row of each lookup (pooled calls only)
  constexpr int W = kRouteThreads / 64;
  __shared__ uint32_t s_wave[W], s_max[W], s_overs;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0) s_overs = 0u;
  for (int i = tid; i < nb; i += kRouteThreads) hist[i] = 0u;
  __syncthreads();
  const int64_t n0 = (int64_t)blockIdx.x * rows_wg;
  const int rows_here = (int)min((int64_t)rows_wg, a.N - n0);
  vfloat4 sample = {};
  if (FIXED && k.sampled) sample = sample_of(reinterpret_cast<const vfloat4*>(dOut), n0 * (a.D / 4), (n0 + rows_here) * (a.D / 4), kRouteThreads);
  auto new_max = [&](uint32_t m) {
    if (m > __hip_atomic_load(&fs->absmax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&fs->absmax_bits, m);
  };
  auto take_max = [&] {
    const int64_t pieces = (a.bag_off ? a.B : a.N) * a.D / 4, share = (pieces + gridDim.x - 1) / gridDim.x, first = share * blockIdx.x;
    const uint32_t m = absmax_of(reinterpret_cast<const vfloat4*>(dOut), first, min(pieces, first + share), kRouteThreads);
    if (lane == 0) new_max(m);
  };
  for (int q = tid; q < rows_here; q += kRouteThreads) {
    const int64_t n = n0 + q;
    if (a.bag_off) s_src[q] = (uint32_t)bag_of(a, n);
    for_each_chunk(a, walk != 0, tables[n], (uint64_t)rows[n], [&](int64_t c, int64_t off, int sgn) {
      s_key[q * C + c] = (uint32_t)off | (sgn < 0 ? 0x80000000u : 0u);
      const uint32_t b = k.bucket((uint32_t)off);
      if (twice && b + 1 < (uint32_t)nb && k.bucket((uint32_t)off + (uint32_t)a.Z - 1u) != b)
        s_over[atomicAdd(&s_overs, 1u)] = (uint32_t)(q * C + c) | (atomicAdd(&hist[b + 1], 1u) << 16);
      s_pos[q * C + c] = (uint16_t)atomicAdd(&hist[b], 1u);
    });
  }
  __syncthreads();
  // One global add per (workgroup, bucket) reserves that many consecutive list slots.  The answers come back while the
  // prefix of the histogram is formed (where the workgroup's chunks of a bucket start when ordered by (bucket, rank)).
  constexpr int P = kMaxBuckets / kRouteThreads;                   // buckets per thread, consecutive ones
  const int per = (nb + kRouteThreads - 1) / kRouteThreads;
  uint32_t cnt[P], got[P], sum = 0;
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const int i = tid * per + j;
    cnt[j] = j < per && i < nb ? hist[i] : 0u;
    got[j] = cnt[j] ? atomicAdd(&cursor[i], cnt[j]) : 0u;
    sum += cnt[j];
  }
  if (FIXED && k.take_max && !k.sampled) take_max();
  if (FIXED && k.sampled) {
    const uint32_t m = wave_max(absmax4(sample));
    if (lane == 0) s_max[wave] = m;
  }
  uint32_t run = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = (uint32_t)__shfl_up((int)run, d, 64);
    if (lane >= d) run += o;
  }
  if (lane == 63) s_wave[wave] = run;
  __syncthreads();
  if (FIXED && k.sampled && tid == 0) {
    uint32_t m = s_max[0];
#pragma unroll
    for (int w = 1; w < W; ++w) m = max(m, s_max[w]);
    new_max(m);
  }
  run -= sum;
#pragma unroll
  for (int w = 0; w < W; ++w)
    if (w < wave) run += s_wave[w];
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const int i = tid * per + j;
    if (j < per && i < nb) {
      pre[i] = run;
      gbase[i] = got[j];
    }
    run += cnt[j];
  }
  __syncthreads();
  // every chunk knows its bucket and its rank inside (workgroup, bucket): that is its list slot.
  // The chunks are written out in (bucket, rank) order, so that consecutive threads store to
  // consecutive list slots of one run (a store instruction then touches a handful of lines instead
  // of 64: scattered 8-byte stores were what this kernel spent its time on).
  const int n_here = rows_here * C;
  for (int i = tid; i < n_here; i += kRouteThreads) s_ord[pre[k.bucket(s_key[i] & 0x7fffffffu)] + s_pos[i]] = (uint16_t)i;
  const int overs = twice ? (int)s_overs : 0;
  for (int t = tid; t < overs; t += kRouteThreads) {
    const uint32_t i = s_over[t] & 0xffffu;
    s_ord[pre[k.bucket(s_key[i] & 0x7fffffffu) + 1] + (s_over[t] >> 16)] = (uint16_t)(i | 0x8000u);
  }
  __syncthreads();
  for (int t = tid; t < n_here + overs; t += kRouteThreads) {
    const int i = s_ord[t] & 0x7fff;
    const uint32_t key = s_key[i];
    uint32_t b = k.bucket(key & 0x7fffffffu), pos = gbase[b] + s_pos[i];
    // entry.x = number of the dOut chunk to add: chunk c of lookup n, or of n's bag in a pooled call
    uint2 e = make_uint2(a.bag_off ? s_src[i / C] * (uint32_t)C + (uint32_t)(i % C) : (uint32_t)(n0 * C + i), key);
    if (twice && (s_ord[t] & 0x8000)) {
      const bool spilled = pos >= cap;             // from its own list: the next bucket finds it there too
      ++b;
      pos = gbase[b] + ((uint32_t)t - pre[b]);
      if (spilled && pos >= cap) continue;
      if (spilled) e = make_uint2(0u, kNoEntry);   // (the place is reserved)
      else if (pos >= cap) e.x |= 0x80000000u;     // (for the next bucket alone)
    }
    if (pos < cap) {
      list[(size_t)b * cap + pos] = e;
      continue;
    }
    const uint32_t sp = atomicAdd(&cursor[nb], 1u);
    if (sp < k.spill_cap) {
      list[(size_t)nb * cap + sp] = e;
      continue;
    }
    // no room there either (never where slots are owned): add this chunk directly
    const float sc = (e.y & 0x80000000u) ? -a.lambda : a.lambda;
    const float* src = dOut + (int64_t)e.x * a.Z;
    if constexpr (FIXED) {
      const double scale = fixed_scale(fs, a.lambda, pbits);
      for (int o = 0; o < a.Z; ++o) atomicAdd(acc + (e.y & 0x7fffffffu) + o, to_fixed(sc * src[o], scale));
    } else {
      float* dst = dM + (e.y & 0x7fffffffu);
      for (int o = 0; o < a.Z; ++o) unsafeAtomicAdd(dst + o, sc * src[o]);
    }
  }
}

// Sums in fp64, of rows of dOut that belong to one lookup each or to the lookups of a bag; fixed point, with the scale of the call or a workgroup's own.
// A row that several lookups share stays in the L2 (plain loads: 8191 bags of 26 30 -> 27 us), one that is read once goes by it (with plain loads 1.7 M rows of 128
// 197 -> 226 us, 0.26 M 45 -> 51).
enum { ACC_ROWS, ACC_BAGS, ACC_FIXED, ACC_SAMPLED };

// What bounds it: the gather of 128-byte pieces of dOut (5.7 TB/s on 6.8 M chunks of 32; 152 of the kernel's 188 us), beside which
// the sort, the image and its flush (29 us) are only partly hidden by the other workgroup of the CU.  Sorting puts the chunks of a popular row, which add to
// the same slots, next to one another: where adds into the image one chunk at a time (two segments of unsorted lists)
// meet in the same LDS words, runs of them cost a register add (pooled gradient of 0.85 M chunks 45 -> 30 us with its sums;
// 0.73 M chunks of 16 over an M of 0.24 Mi 55 -> 38).  LPI: lanes per chunk, Z / 4 (4, 8 or 16; 0: any other).
template <int KIND, int LPI>
__global__ __launch_bounds__(kAccThreads, 4) void k_embed_accum(EmbedArgs a, AccPlan k, const uint32_t* __restrict__ cursor, const uint2* __restrict__ list,
                                                     const float* __restrict__ dOut, float* __restrict__ dM, int pbits,
                                                     FixedScale* fs, unsigned long long* __restrict__ acc) {
  // fp64 image: LDS fp32 atomic adds were measured ~20x slower than fp64 ones on this chip.
  // FIXED: the same 8-byte slots hold 64-bit fixed-point sums.
  constexpr bool FIXED = KIND >= ACC_FIXED, SAMPLED = KIND == ACC_SAMPLED;
  using img_t = typename std::conditional<FIXED, unsigned long long, double>::type;
  extern __shared__ __attribute__((aligned(16))) char img_raw[];
  __shared__ uint32_t s_wave[kAccThreads / 64];
  // Workgroups go to the 8 XCDs round-robin: the parts of a bucket, which read the same list, follow one another on
  // one XCD, and the segments that only long lists have come last.
  const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
  const int Q = 1 << k.q_log2, per_xcd = (k.nb + 7) / 8;
  const int part = j & (Q - 1), bi = (j >> k.q_log2) % per_xcd;
  const uint32_t seg = (uint32_t)((j >> k.q_log2) / per_xcd);
  // Segments of few buckets go round the XCDs: 18 buckets are three for two of them and two for the others, whose places stay empty (rows of 128, 1.56 M in
  // chunks of 16 over 70000 slots 401 -> 361 us, 1.3 M over 138614 187 -> 179, 0.4 M of 64 over 70000 62 -> 54.5).  Of 49 buckets, 7 and 6, they stay:
  // 1.7 M of 64 in chunks of 16 208 and 211.
  const int b = bi * 8 + (k.nb < 48 ? (x + (int)seg) & 7 : x);
  if (b >= k.nb) return;
  const int S = k.R() >> k.q_log2, Z = a.Z;
  const int64_t slot0 = (int64_t)b * k.R() + part * S;
  if (slot0 >= a.m_size) return;
  const uint32_t largest = FIXED ? fs->absmax_bits : 0u;          // (asked for with the cursors)
  const uint32_t asked = cursor[b], count = min(asked, k.cap), spilled = min(cursor[k.nb], k.spill_cap);
  const uint32_t nseg = k.segments(count);
  if (seg >= nseg) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // image: Z slots of the part before, this part's, Z slots of the next
  const int span = acc_span(S, Z);
  img_t* img = reinterpret_cast<img_t*>(img_raw);
  uint32_t* bin = reinterpret_cast<uint32_t*>(img + span);        // two 16-bit counters each
  const uint16_t* bin16 = reinterpret_cast<const uint16_t*>(bin);
  uint32_t* s_src = bin + span / 2;                               // sorted: chunk of dOut | sign << 31
  uint16_t* s_at = reinterpret_cast<uint16_t*>(s_src + acc_sorted(Z));    // ... and place in the image
  double scale = 0.0;
  // (sampled) bits of the largest |dOut| that the scale allows for, and of the largest that is added
  uint32_t limit = 0u, top = 0u;
  auto uniform = [](double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, (uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)b) | (uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32);
  };
  if constexpr (FIXED) {
    if constexpr (SAMPLED) {
      const uint32_t bits = __builtin_amdgcn_readfirstlane(largest);
      const int own = local_pbits(asked), spare = local_spare(own, pbits);
      scale = uniform(fixed_scale(bits, a.lambda, own - spare));
      pbits = own;
      limit = sample_limit(bits, a.lambda, spare);
    } else {
      scale = fixed_scale(largest, a.lambda, pbits);
    }
  }
  const uint32_t low = (uint32_t)slot0 - (uint32_t)Z;             // M offset of the image's first slot (modulo 2^32)
  auto clear = [&] {
    for (int i = tid; i < span; i += kAccThreads) img[i] = img_t(0);
  };
  clear();
#pragma unroll 1
  for (int r = 0; r < 2;) {
    const uint2* lst = list + (size_t)b * k.cap;
    uint32_t entries = count, len = k.length<FIXED>(entries, nseg), first = seg * len;
    if (r == 1) {
      lst = list + (size_t)k.nb * k.cap;
      entries = spilled;
      len = k.length<FIXED>(entries, nseg);
      first = seg * len;
    }
    const uint32_t end = min(entries, first + len);
    uint2 ent[kPer];
    auto fetch = [&](uint32_t i0) {
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const uint32_t i = i0 + u * kAccThreads + tid;
        ent[u] = i < end ? lst[i] : make_uint2(0u, low);          // (low: beside the slots, not picked)
      }
    };
    if (first < end) fetch(first);
#pragma unroll 1
    for (uint32_t i0 = first; i0 < end; i0 += kPass) {
      if (tid * 16 < span) {
        uint4* p = reinterpret_cast<uint4*>(bin + tid * 8);
        p[0] = p[1] = make_uint4(0u, 0u, 0u, 0u);
      }
      __syncthreads();
      uint32_t at[kPer], rank[kPer] = {};
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        at[u] = (ent[u].y & 0x7fffffffu) - low;
        if (r == 1 && (FIXED && (SAMPLED || k.owned) ? (ent[u].x >> 31) && at[u] >= (uint32_t)Z : part == 0 && at[u] < (uint32_t)Z)) at[u] = 0u;
        if (at[u] - 1u >= (uint32_t)(S + Z - 1)) at[u] = 0u;        // (not picked)
        if (at[u]) {
          const int sh = 16 * (at[u] & 1);
          rank[u] = (atomicAdd(&bin[at[u] >> 1], 1u << sh) >> sh) & 0xffffu;
        }
      }
      __syncthreads();
      // exclusive prefix of the counters, sixteen to a thread
      uint32_t total = 0;
      {
        uint4* p = reinterpret_cast<uint4*>(bin + tid * 8);
        uint32_t c[8] = {};
        if (tid * 16 < span) {
          const uint4 lo = p[0], hi = p[1];
          c[0] = lo.x; c[1] = lo.y; c[2] = lo.z; c[3] = lo.w;
          c[4] = hi.x; c[5] = hi.y; c[6] = hi.z; c[7] = hi.w;
        }
        uint32_t sum = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) sum += (c[i] & 0xffffu) + (c[i] >> 16);
        uint32_t run = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const uint32_t o = (uint32_t)__shfl_up((int)run, d, 64);
          if (lane >= d) run += o;
        }
        if (lane == 63) s_wave[wave] = run;
        __syncthreads();
        run -= sum;
#pragma unroll
        for (int w = 0; w < kAccThreads / 64; ++w) {
          if (w < wave) run += s_wave[w];
          total += s_wave[w];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint32_t mid = run + (c[i] & 0xffffu), next = mid + (c[i] >> 16);
          c[i] = run | (mid << 16);
          run = next;
        }
        if (tid * 16 < span) {
          p[0] = make_uint4(c[0], c[1], c[2], c[3]);
          p[1] = make_uint4(c[4], c[5], c[6], c[7]);
        }
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kPer; ++u) rank[u] += bin16[at[u]];
#pragma unroll
      for (int u = 0; u < kPer; ++u)
        if (at[u]) {
          s_src[rank[u]] = (ent[u].x & 0x7fffffffu) | (ent[u].y & 0x80000000u);
          s_at[rank[u]] = (uint16_t)at[u];
        }
      // The sorted entries, shared out evenly among groups of lanes that hold a chunk.  What fills up the last shares
      // adds chunk 0 of dOut to the place before the image's first slot.
      const int lanes = LPI ? LPI : min(Z / 4, 64), per_wave = LPI ? 64 / LPI : acc_groups(Z), groups = per_wave * (kAccThreads / 64);
      const int sub = lane % lanes, which = lane / lanes;
      const int share = ((int)(total + groups * U - 1) / (groups * U) | 1) * U;   // (an odd number of quadruples: no two groups of a wave read the same banks)
      for (int p = (int)total + tid; p < groups * share; p += kAccThreads) {
        s_src[p] = 0u;
        s_at[p] = 0;
      }
      __syncthreads();
      if (i0 + kPass < end) fetch(i0 + kPass);
      const uint32_t* g_src = s_src + (wave * per_wave + which) * share;
      const uint16_t* g_at = s_at + (wave * per_wave + which) * share;
      const int pieces = LPI ? 1 : (Z / 4 + 63) / 64;             // (of 64 lanes, Z > 256)
#pragma unroll 1
      for (int pc = 0; pc < pieces; ++pc) {
        const int o = 4 * (sub + 64 * pc);
        if (!LPI && (which >= per_wave || o >= Z)) continue;
        const float* from = dOut + o;
        struct Batch {
          uint32_t src[U];
          int at[U];
          vfloat4 d[U];
        };
        Batch A, B;
        img_t sum[4] = {img_t(0), img_t(0), img_t(0), img_t(0)};
        int cur = 0;
        uint32_t n = 0;                               // (fixed point) addends of the sums
        auto put = [&] {
          img_t* to = img + cur + o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if constexpr (FIXED) atomicAdd(&to[e], fixed_sum(sum[e], n));
            else atomicAdd(&to[e], sum[e]);
          }
        };
        auto load = [&](Batch& x, int i) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            x.src[u] = g_src[i + u];
            x.at[u] = g_at[i + u];
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
          {
            const vfloat4* p = reinterpret_cast<const vfloat4*>(from + (int64_t)(x.src[u] & 0x7fffffffu) * (LPI ? 4 * LPI : Z));
            x.d[u] = KIND == ACC_BAGS ? *p : __builtin_nontemporal_load(p);
          }
        };
        auto add = [&](const Batch& x) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if (x.at[u] != cur) {
              put();
#pragma unroll
              for (int e = 0; e < 4; ++e) sum[e] = img_t(0);
              cur = x.at[u];
              n = 0;
            }
            if constexpr (SAMPLED) top = max(top, x.at[u] ? absmax4(x.d[u]) : 0u);   // (not of what fills up the shares)
            const float sc = __uint_as_float(__float_as_uint(a.lambda) ^ (x.src[u] & 0x80000000u));
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              if constexpr (FIXED) sum[e] += fixed_raw(sc * x.d[u][e], scale);
              else sum[e] += (double)(sc * x.d[u][e]);
            }
            ++n;
          }
        };
        if (share > 0) load(A, 0);
        if (share > U) load(B, U);
#pragma unroll 1
        for (int i = 0; i < share; i += 2 * U) {
          add(A);
          if (i + 2 * U < share) load(A, i + 2 * U);
          if (i + U < share) add(B);
          if (i + 3 * U < share) load(B, i + 3 * U);
        }
        put();
      }
      __syncthreads();
    }
    ++r;
    if (SAMPLED && r == 2) {
      // Has a chunk exceeded what the scale allows for?  Then once more, with the largest of them instead of the sample's.
      top = wave_max(top);
      if (lane == 0) s_wave[wave] = top;
      __syncthreads();
#pragma unroll 1
      for (int w = 0; w < kAccThreads / 64; ++w) top = max(top, s_wave[w]);
      top = __builtin_amdgcn_readfirstlane(top);
      if (top > limit) {
        limit = 0xffffffffu;
        scale = uniform(fixed_scale(top, a.lambda, pbits));
        clear();
        if (scale == scale) r = 0;
      }
      __syncthreads();
    }
  }
  __syncthreads();
  if constexpr (SAMPLED) {
    // An Inf or NaN makes all of dM NaN: the first workgroup to find one that the sample has not adds NaN to every slot.
    if (scale != scale && largest < 0x7f800000u) {
      if (tid == 0) s_wave[0] = atomicExch(&fs->not_finite, 1u);
      __syncthreads();
      if (s_wave[0] == 0u)
        for (int64_t i = tid; i < a.m_size; i += kAccThreads) unsafeAtomicAdd(dM + i, __uint_as_float(0x7fc00000u));
      return;
    }
  }
  const int own = !(FIXED && (SAMPLED || k.owned)) && part == Q - 1 ? S + Z : S;
  for (int i = tid; i < own && slot0 + i < a.m_size; i += kAccThreads) {
    const img_t v = img[Z + i];
    if constexpr (FIXED) {
      if (!SAMPLED && acc) {
        if (v != 0ull) atomicAdd(acc + slot0 + i, v);
      } else {
        // (sampled: another workgroup may be adding NaN)
        if constexpr (SAMPLED) {
          if (scale != scale) unsafeAtomicAdd(dM + slot0 + i, __uint_as_float(0x7fc00000u));
          else if (v != 0ull) unsafeAtomicAdd(dM + slot0 + i, (float)((double)(long long)v / scale));
        } else if (scale != scale) {
          dM[slot0 + i] += __uint_as_float(0x7fc00000u);
        } else if (v != 0ull) {
          dM[slot0 + i] += (float)((double)(long long)v / scale);
        }
      }
    } else {
      const float f = (float)v;
      if (f != 0.f) unsafeAtomicAdd(dM + slot0 + i, f);          // (another stream's call may be adding too)
    }
  }
}

}  // namespace

roast_status embed_fwd_launch(const EmbedArgs& a, const int64_t* rows, const uint32_t* tables, const float* M,
                              float* out, hipStream_t s) {
  return launch_embed<false>(a, rows, tables, M, out, nullptr, nullptr, s);
}

size_t embed_bucket_workspace_bytes(const EmbedArgs& a) {
  const BucketPlan p = bucket_plan(a);
  return p.ok ? p.total : 0;
}

namespace {

// route + accumulate; FIXED selects the 64-bit fixed-point variant (fs, acc in the workspace)
template <bool FIXED>
roast_status bucket_run(const EmbedArgs& a, const BucketPlan& p, const int64_t* rows, const uint32_t* tables,
                        const float* dOut, float* dM, char* base, int pbits, FixedScale* fs,
                        unsigned long long* acc, hipStream_t s) {
  uint32_t* cursor = (uint32_t*)base;
  uint2* list = (uint2*)(base + p.list_off);
  const AccPlan k = acc_plan(a, p, FIXED);
  if (k.owned) acc = nullptr;
  // Chunks per route workgroup: 8192 (long runs per bucket, few reservations) once that leaves a
  // workgroup for every CU, fewer for smaller batches (0.85 M chunks: 2048 instead of 8192, -9 us).
  int items = kRouteItems;
  while (items > 2048 && p.n_items / items < 256) items /= 2;
  const int rows_wg = items / (int)a.C;
  const size_t lds_route = (size_t)items * (k.owned ? 4 + 2 + 4 + 4 : 4 + 2 + 2) + (size_t)3 * p.nb * 4 + (a.bag_off ? (size_t)rows_wg * 4 : 0);
  const int S = k.R() >> k.q_log2;
  const dim3 grid((unsigned)((p.nb + 7) / 8 * 8) * k.most << k.q_log2);
  auto run = [&](auto LPI) -> roast_status {
    constexpr int L = decltype(LPI)::value;
    constexpr int kOne = FIXED ? ACC_FIXED : ACC_ROWS, kOther = FIXED ? ACC_SAMPLED : ACC_BAGS;
    auto* accum = (FIXED ? k.sampled : a.bag_off != nullptr) ? &k_embed_accum<kOther, L> : &k_embed_accum<kOne, L>;
    static std::atomic<bool> configured{false};   // per instantiation; a race between host threads only repeats the calls
    if (!configured.load(std::memory_order_acquire)) {
      // (the route kernel also has a little static LDS)
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(&k_embed_route<FIXED>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 8192) != hipSuccess ||
          hipFuncSetAttribute(reinterpret_cast<const void*>(&k_embed_accum<kOne, L>), hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024) != hipSuccess ||
          hipFuncSetAttribute(reinterpret_cast<const void*>(&k_embed_accum<kOther, L>), hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024) != hipSuccess)
        return ROAST_ERR_HIP;
      configured.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(k_embed_route_init, dim3((unsigned)(p.nb + 256) / 256), dim3(256), 0, s, p.nb, cursor, k.take_max ? (uint32_t*)fs : nullptr);
    hipLaunchKernelGGL(k_embed_route<FIXED>, dim3((unsigned)((a.N + rows_wg - 1) / rows_wg)), dim3(kRouteThreads), lds_route, s, a,
                       k, walk_ok(a), items, rows, tables, cursor, list, dOut, dM, pbits, fs, acc);
    hipLaunchKernelGGL(accum, grid, dim3(kAccThreads), acc_lds(S, a.Z), s, a, k, cursor, list, dOut, dM, pbits, fs, acc);
    return hip_status(hipGetLastError());
  };
  switch (a.Z) {
    case 16: return run(std::integral_constant<int, 4>{});
    case 32: return run(std::integral_constant<int, 8>{});
    case 64: return run(std::integral_constant<int, 16>{});
    default: return run(std::integral_constant<int, 0>{});
  }
}

// From 65536 chunks on.  (The direct adds would be as fast a little beyond that -- 104 000 chunks of 32
// take 27 us routed and 29 direct -- but they sum in fp32, a slot that a popular row adds to thousands of times
// included, where the routed gradient sums in fp64 and rounds once per flush.)
inline bool bucket_worthwhile(const BucketPlan& p, const float* dOut) {
  return p.ok && p.n_items >= 65536 && ((uintptr_t)dOut & 15) == 0;
}

struct DetLayoutE {
  size_t fs_off, acc_off, bucket_off, total;
};

inline DetLayoutE det_layout_e(const EmbedArgs& a) {
  auto up = [](size_t v) { return (v + 255) / 256 * 256; };
  DetLayoutE l{};
  size_t o = 0;
  l.fs_off = o;     o += up(sizeof(FixedScale));
  l.acc_off = o;    o += up((size_t)a.m_size * 8);
  l.bucket_off = o; o += embed_bucket_workspace_bytes(a);
  l.total = o;
  return l;
}

}  // namespace

roast_status embed_bwd_atomic_launch(const EmbedArgs& a, const int64_t* rows, const uint32_t* tables,
                                     const float* dOut, float* dM, void* ws, size_t ws_bytes, hipStream_t s) {
  const BucketPlan p = bucket_plan(a);
  // small problems, odd shapes, or no workspace: plain atomics straight into dM
  if (!bucket_worthwhile(p, dOut) || ws == nullptr || ws_bytes < p.total)
    return launch_embed<true>(a, rows, tables, nullptr, nullptr, dOut, dM, s);
  return bucket_run<false>(a, p, rows, tables, dOut, dM, (char*)ws, 0, nullptr, nullptr, s);
}

// DETERMINISTIC: largest |dOut| (or that of a sample of it, see local_pbits) -> fixed-point scale; zeroed 64-bit accumulator of |M| slots in the
// workspace; the same route + accumulate pipeline (or one thread per element for the shapes it does
// not take) with integer atomics; then dM += accumulator / scale, one rounding per slot.
size_t embed_det_workspace_bytes(const EmbedArgs& a) {
  if (a.N * a.C >= (1ll << 40)) return 0;
  return det_layout_e(a).total;
}

roast_status embed_bwd_det_run(const EmbedArgs& a, const int64_t* rows, const uint32_t* tables, const float* dOut,
                               float* dM, void* ws, hipStream_t s) {
  if (a.N * a.C >= (1ll << 40)) return ROAST_ERR_UNSUPPORTED;
  const DetLayoutE l = det_layout_e(a);
  char* base = (char*)ws;
  FixedScale* fs = (FixedScale*)(base + l.fs_off);
  unsigned long long* acc = (unsigned long long*)(base + l.acc_off);
  const int pbits = fixed_pbits(a.N * a.C);
  const BucketPlan p = bucket_plan(a);
  const bool routed = bucket_worthwhile(p, dOut);
  // where every slot has one owner, the accumulator is not used, and mostly the route kernel takes the maximum
  const AccPlan k = routed ? acc_plan(a, p, true) : AccPlan{};
  const bool owned = k.owned;
  const int64_t n_el = a.N * a.D;                               // contributions
  const int64_t n_grad = (a.bag_off ? a.B : a.N) * a.D;          // elements of dOut
  if (!k.take_max) {
    // zero the scale record and the accumulator (contiguous: fs_off == 0, acc follows)
    const int64_t zero_words = (int64_t)((owned ? sizeof(FixedScale) : l.acc_off + (size_t)a.m_size * 8) / 4);
    const int64_t zb = (zero_words + 255) / 256;
    if (zb > 0x7fffffffll) return ROAST_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(k_embed_zero, dim3((unsigned)zb), dim3(256), 0, s, (uint32_t*)base, zero_words);
    const int64_t ab = std::min<int64_t>(n_grad / (4 * 8 * kMaxThreads) + 1, 512);
    hipLaunchKernelGGL(k_embed_absmax, dim3((unsigned)ab), dim3(kMaxThreads), 0, s, dOut, n_grad, fs);
  }
  roast_status st;
  if (routed) {
    st = bucket_run<true>(a, p, rows, tables, dOut, dM, base + l.bucket_off, pbits, fs, acc, s);
  } else {
    const int64_t blocks = (n_el + 255) / 256;
    if (blocks > 0x7fffffffll) return ROAST_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(k_embed_fixed_elem, dim3((unsigned)blocks), dim3(256), 0, s, a, pbits, rows, tables, dOut, fs, acc);
    st = hip_status(hipGetLastError());
  }
  if (st != ROAST_OK || owned) return st;
  hipLaunchKernelGGL(k_embed_fixed_finish, dim3((unsigned)((a.m_size + 255) / 256)), dim3(256), 0, s, a.m_size, a.lambda,
                     pbits, fs, acc, dM);
  return hip_status(hipGetLastError());
}

// ---------------------------------------------------------------------------------------------
// Lookup gradient for callers that cannot allocate: the workspace of roast_embed_bwd (bucket
// cursors and lists; in the deterministic mode also the fixed-point accumulator) lives in a
// file-scope device array instead of a caller buffer.  Every GPU the library runs on holds its own
// copy of the array, at its own address, until the process ends.
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each device, once known

// Device address of this device's copy of `scratch` (in host code the array's name is only a
// stand-in for the symbol, never an address a kernel could use).
roast_status static_scratch_ptr(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return ROAST_ERR_HIP;
  void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (p == nullptr) {
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return ROAST_ERR_HIP;
    g_scratch_ptr[dev].store(p, std::memory_order_release);   // a race between host threads stores the same value twice
  }
  *out = p;
  return ROAST_OK;
}
}  // namespace

size_t embed_static_scratch_bytes() { return kStaticScratchBytes; }

roast_status embed_bwd_static_run(const EmbedArgs& a, const int64_t* rows, const uint32_t* tables, const float* dOut,
                                  float* dM, bool deterministic, hipStream_t s) {
  const size_t need = deterministic ? embed_det_workspace_bytes(a) : embed_bucket_workspace_bytes(a);
  if (deterministic && need == 0) return ROAST_ERR_UNSUPPORTED;
  if (need > kStaticScratchBytes) return ROAST_ERR_WORKSPACE;
  void* ws = nullptr;
  if (need > 0) {
    const roast_status st = static_scratch_ptr(&ws);
    if (st != ROAST_OK) return st;
  }
  // From here on the device pointer `ws` stands for the array: the kernels get it as an argument,
  // exactly as they get the caller's buffer in roast_embed_bwd.  What has to start at zero (bucket
  // cursors, the fixed-point accumulator and its scale record) is cleared by fill kernels inside.
  if (deterministic) return embed_bwd_det_run(a, rows, tables, dOut, dM, ws, s);
  return embed_bwd_atomic_launch(a, rows, tables, dOut, dM, ws, need, s);
}

roast_status embed_bag_fwd_launch(const EmbedArgs& a, const int64_t* rows, const uint32_t* tables, const float* M,
                                  float* out, hipStream_t s) {
  if (a.m_size >= (1ll << 31) || a.C > kMaxC || a.hash.use_sign == 2) {
    const int64_t blocks = (a.B * a.D + 255) / 256;
    if (blocks > 0x7fffffffll) return ROAST_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(k_embed_bag_fwd_elem, dim3((unsigned)blocks), dim3(256), 0, s, a, rows, tables, M, out);
    return hip_status(hipGetLastError());
  }
  const bool vec4 = (a.Z % 4 == 0) && (a.D % 4 == 0) && (((uintptr_t)out & 15) == 0);
  const int64_t pieces = vec4 ? a.D / 4 : a.D;
  const int tpb = (int)std::min<int64_t>(256, pieces);      // threads per bag
  const int bags_wg = 256 / tpb;
  const int win = (int)(8192 / a.C);                        // 32 KiB of keys per window
  const int64_t blocks = (a.B + bags_wg - 1) / bags_wg;
  if (blocks > 0x7fffffffll) return ROAST_ERR_UNSUPPORTED;
  const size_t lds = (size_t)win * a.C * sizeof(uint32_t);
  if (vec4)
    hipLaunchKernelGGL(k_embed_bag_fwd<4>, dim3((unsigned)blocks), dim3(256), lds, s, a, walk_ok(a), tpb, bags_wg, win,
                       rows, tables, M, out);
  else
    hipLaunchKernelGGL(k_embed_bag_fwd<1>, dim3((unsigned)blocks), dim3(256), lds, s, a, walk_ok(a), tpb, bags_wg, win,
                       rows, tables, M, out);
  return hip_status(hipGetLastError());
}

roast_status chunk_index_launch(const EmbedArgs& a, const int64_t* rows, const uint32_t* tables, int64_t* off,
                                int8_t* sgn, hipStream_t s) {
  const int64_t blocks = (a.N + 255) / 256;
  if (blocks > 0x7fffffffll) return ROAST_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(k_chunk_index, dim3((unsigned)blocks), dim3(256), 0, s, a, walk_ok(a), rows, tables, off, sgn);
  return hip_status(hipGetLastError());
}

}  // namespace roast
