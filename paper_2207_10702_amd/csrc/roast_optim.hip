// Optimizer step on the shared array M: the "update weights" leg of the paper's training workload
// (Appendix tables "update weights (optim.step())": SGD, Adagrad and Adam on the |M|-sized
// parameter).  One streaming pass over |M| floats that also does what would otherwise be two more
// passes: it clears the gradient for the next step and refreshes the bf16 shadow of M that the bf16
// ROAST-MM kernels read.  HBM-bound: 8 (SGD) to 24 (Adam) bytes read and 4 to 16 bytes written per
// parameter, 4 parameters per thread.
#include "roast_internal.hpp"

namespace roast {
namespace {

typedef float vfloat4 __attribute__((ext_vector_type(4)));

struct OptimArgs {
  int kind;
  float lr, wd, b1, b2, eps;
  float omb1, omb2;       // 1 - beta, computed on the host in double (1.f - 0.999f is off by 1e-5)
  float bc1, bc2;         // Adam bias corrections 1 - beta^t, computed on the host in double
  int zero_grad;
  int copies;             // of the shadow
  int64_t n, stride;      // |M|, distance between the copies
};

__device__ inline float update(const OptimArgs& a, float m, float g, float* s1, float* s2) {
  g = fmaf(a.wd, m, g);
  if (a.kind == ROAST_OPT_SGD) return m - a.lr * g;
  if (a.kind == ROAST_OPT_ADAGRAD) {
    *s1 = fmaf(g, g, *s1);
    return m - a.lr * g / (sqrtf(*s1) + a.eps);
  }
  *s1 = a.b1 * *s1 + a.omb1 * g;
  *s2 = a.b2 * *s2 + a.omb2 * g * g;
  return m - a.lr * (*s1 / a.bc1) / (sqrtf(*s2 / a.bc2) + a.eps);
}

typedef uint32_t vuint2 __attribute__((ext_vector_type(2)));

__device__ inline uint32_t pack(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 r = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, r);
}
__device__ inline uint16_t to_bf16(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }

// Four parameters per thread, 16-byte accesses.  The shadow's copies are written 8 bytes at a time (2-byte
// stores took half as long again as the rest of the pass): the one that is shifted by a parameter needs
// the next thread's first (from the next lane; across waves the value's owner stores it).
__global__ __launch_bounds__(256) void k_optim(OptimArgs a, float* __restrict__ M, float* __restrict__ dM,
                                               float* __restrict__ st1, float* __restrict__ st2,
                                               uint16_t* __restrict__ shadow) {
  const int64_t i0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  const int lane = threadIdx.x & 63;
  const bool full = i0 + 4 <= a.n;
  vfloat4 m = {0.f, 0.f, 0.f, 0.f}, g = m, s1 = m, s2 = m;
  if (full) {
    m = *reinterpret_cast<const vfloat4*>(M + i0);
    g = *reinterpret_cast<const vfloat4*>(dM + i0);
    if (a.kind != ROAST_OPT_SGD) s1 = *reinterpret_cast<const vfloat4*>(st1 + i0);
    if (a.kind == ROAST_OPT_ADAM) s2 = *reinterpret_cast<const vfloat4*>(st2 + i0);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (i0 + k < a.n) {
        m[k] = M[i0 + k];
        g[k] = dM[i0 + k];
        if (a.kind != ROAST_OPT_SGD) s1[k] = st1[i0 + k];
        if (a.kind == ROAST_OPT_ADAM) s2[k] = st2[i0 + k];
      }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float x = s1[k], y = s2[k];
    const float v = update(a, m[k], g[k], &x, &y);
    m[k] = i0 + k < a.n ? v : 0.f;
    s1[k] = x; s2[k] = y;
  }
  if (full) {
    *reinterpret_cast<vfloat4*>(M + i0) = m;
    if (a.kind != ROAST_OPT_SGD) *reinterpret_cast<vfloat4*>(st1 + i0) = s1;
    if (a.kind == ROAST_OPT_ADAM) *reinterpret_cast<vfloat4*>(st2 + i0) = s2;
    if (a.zero_grad) *reinterpret_cast<vfloat4*>(dM + i0) = vfloat4{0.f, 0.f, 0.f, 0.f};
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (i0 + k < a.n) {
        M[i0 + k] = m[k];
        if (a.kind != ROAST_OPT_SGD) st1[i0 + k] = s1[k];
        if (a.kind == ROAST_OPT_ADAM) st2[i0 + k] = s2[k];
        if (a.zero_grad) dM[i0 + k] = 0.f;
      }
  }
  if (shadow == nullptr) return;
  const float next = __shfl_down(m[0], 1, 64);     // (every lane of the wave is still here)
  if (i0 >= a.n) return;                           // the padding beyond M was written when the shadow was made
  const uint32_t c0 = pack(m[0], m[1]), c1 = pack(m[2], m[3]);
  const uint32_t x0 = pack(m[1], m[2]), x1 = pack(m[3], next);
  for (int c = 0; c < a.copies; c += 2) {          // M and M shifted by one; where there are four copies, the same of -M
    const uint32_t flip = c ? 0x80008000u : 0u;
    uint16_t* o = shadow + c * a.stride + i0;
    if (full) {
      *reinterpret_cast<vuint2*>(o) = vuint2{c0 ^ flip, c1 ^ flip};
      if (lane < 63) {
        *reinterpret_cast<vuint2*>(o + a.stride) = vuint2{x0 ^ flip, x1 ^ flip};
      } else {
        *reinterpret_cast<uint32_t*>(o + a.stride) = x0 ^ flip;
        o[a.stride + 2] = (uint16_t)(x1 ^ flip);
      }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (i0 + k < a.n) {
          o[k] = to_bf16(m[k]) ^ (uint16_t)flip;
          o[a.stride + k] = (k < 3 ? to_bf16(m[k < 3 ? k + 1 : 3]) : (uint16_t)0) ^ (uint16_t)flip;
        }
    }
    if (lane == 0 && i0 > 0) o[a.stride - 1] = to_bf16(m[0]) ^ (uint16_t)flip;
  }
}

}  // namespace

roast_status optim_launch(const roast_optim_desc& d, int64_t m_size, float* M, float* dM, float* st1, float* st2,
                          void* shadow, hipStream_t s) {
  OptimArgs a{};
  a.kind = (int)d.kind; a.lr = d.lr; a.wd = d.weight_decay; a.b1 = d.beta1; a.b2 = d.beta2; a.eps = d.eps;
  a.omb1 = (float)(1.0 - (double)d.beta1);
  a.omb2 = (float)(1.0 - (double)d.beta2);
  a.bc1 = (float)(1.0 - pow((double)d.beta1, (double)d.step));
  a.bc2 = (float)(1.0 - pow((double)d.beta2, (double)d.step));
  a.zero_grad = d.zero_grad ? 1 : 0;
  a.n = m_size; a.stride = shadow_stride(m_size); a.copies = shadow_copies(m_size);
  const int64_t blocks = (m_size + 1023) / 1024;
  if (blocks > 0x7fffffffll) return ROAST_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(k_optim, dim3((unsigned)blocks), dim3(256), 0, s, a, M, dM, st1, st2, (uint16_t*)shadow);
  return hip_status(hipGetLastError());
}

}  // namespace roast
