// Adam update of a flat parameter vector and the helpers of the replica weight
// synchronisation.  HBM-bound: 16 bytes read and 12 + sizeof(storage) bytes
// written per parameter, 16-byte accesses, no reductions.
//
// The paper names the optimizer (Adam, Section 7) and requires the replica to
// carry the successor's parameters and optimizer state (Section 5.1); the update
// is the textbook one: m <- b1 m + (1-b1) g, v <- b2 v + (1-b2) g^2,
// w <- w - lr (m / (1-b1^t)) / (sqrt(v / (1-b2^t)) + eps), on fp32 master
// weights, with the storage-dtype copy that the layer kernels read rewritten in
// the same pass.
#include <math.h>

#include "common.h"

namespace bamboo {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kAdamGroups = 2;    // groups of four parameters per lane

template <typename T> struct Store4;
template <> struct Store4<float> {
  __device__ static __forceinline__ void put(float* p, const float4& v) { *(float4*)p = v; }
  __device__ static __forceinline__ float4 get(const float* p) { return *(const float4*)p; }
};
template <> struct Store4<bf16_t> {
  typedef __attribute__((ext_vector_type(4))) __bf16 raw;
  __device__ static __forceinline__ void put(bf16_t* p, const float4& v) {
    raw t;
    t[0] = (bf16_t)v.x; t[1] = (bf16_t)v.y; t[2] = (bf16_t)v.z; t[3] = (bf16_t)v.w;
    *(raw*)p = t;
  }
  __device__ static __forceinline__ float4 get(const bf16_t* p) {
    const raw t = *(const raw*)p;
    return make_float4((float)t[0], (float)t[1], (float)t[2], (float)t[3]);
  }
};

// Sixteen bytes per lane that may bypass the caches: STREAM marks the access as not to be kept.
template <bool STREAM> __device__ __forceinline__ f32x4 load4(const f32x4* p) {
  return STREAM ? __builtin_nontemporal_load(p) : *p;
}
template <bool STREAM> __device__ __forceinline__ void store4(f32x4* p, const f32x4& v) {
  if (STREAM) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// inv_c1 = 1 / (1 - beta1^t), inv_c2 = 1 / (1 - beta2^t), computed on the host in double.
// Bound by HBM: 30 bytes per bf16 parameter.  A workgroup takes 2 x 256 groups of four parameters once, with the
// eight loads of a lane requested together, and the dispatcher walks the arrays in order; 2048 workgroups striding
// through them kept as many streams open and took 464 us for 75.6 M parameters (4.8 TB/s), this form 388 us
// (5.85 TB/s) with STREAM, 422 us without.
template <typename T, bool STREAM>
__global__ __launch_bounds__(256) void adam_kernel(long n4, const f32x4* __restrict__ g, f32x4* __restrict__ master,
                                                   f32x4* __restrict__ m, f32x4* __restrict__ v, T* __restrict__ w,
                                                   float lr, float beta1, float beta2, float eps, float inv_c1,
                                                   float inv_c2) {
  const long i0 = (long)blockIdx.x * (256 * kAdamGroups) + threadIdx.x;
  f32x4 gg[kAdamGroups], ww[kAdamGroups], mm[kAdamGroups], vv[kAdamGroups];
#pragma unroll
  for (int u = 0; u < kAdamGroups; ++u) {
    const long i = i0 + u * 256;
    if (i < n4) {
      gg[u] = load4<STREAM>(g + i);
      mm[u] = load4<STREAM>(m + i);
      vv[u] = load4<STREAM>(v + i);
      ww[u] = load4<STREAM>(master + i);
    }
  }
#pragma unroll
  for (int u = 0; u < kAdamGroups; ++u) {
    const long i = i0 + u * 256;
    if (i >= n4) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      mm[u][j] = beta1 * mm[u][j] + (1.0f - beta1) * gg[u][j];
      vv[u][j] = beta2 * vv[u][j] + (1.0f - beta2) * gg[u][j] * gg[u][j];
      ww[u][j] -= lr * (mm[u][j] * inv_c1) / (sqrtf(vv[u][j] * inv_c2) + eps);
    }
    store4<STREAM>(m + i, mm[u]);
    store4<STREAM>(v + i, vv[u]);
    store4<STREAM>(master + i, ww[u]);
    Store4<T>::put(w + 4 * i, make_float4(ww[u][0], ww[u][1], ww[u][2], ww[u][3]));   // read by the next iteration
  }
}

// master[i] = (float) w[i]
template <typename T>
__global__ __launch_bounds__(256) void widen_kernel(long n4, const T* __restrict__ w, float* __restrict__ master) {
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n4; i += (long)gridDim.x * 256)
    ((float4*)master)[i] = Store4<T>::get(w + 4 * i);
}

__global__ __launch_bounds__(256) void fill_zero_kernel(long n4, float* __restrict__ p) {
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < n4; i += (long)gridDim.x * 256)
    ((float4*)p)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

static unsigned grid_for(long n4) {
  long blocks = (n4 + 255) / 256;
  if (blocks > 256 * 8) blocks = 256 * 8;
  if (blocks < 1) blocks = 1;
  return (unsigned)blocks;
}

template <typename T>
static hipError_t adam_launch(hipStream_t s, long n4, const float* g, float* master, float* m, float* v, T* w, float lr,
                              float beta1, float beta2, float eps, float inv_c1, float inv_c2) {
  const auto kern = streams_past_cache(n4 * 4 * (16 + (long)sizeof(T))) ? adam_kernel<T, true> : adam_kernel<T, false>;
  const long blocks = (n4 + 256 * kAdamGroups - 1) / (256 * kAdamGroups);
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), 0, s, n4, (const f32x4*)g, (f32x4*)master, (f32x4*)m,
                     (f32x4*)v, w, lr, beta1, beta2, eps, inv_c1, inv_c2);
  return hipGetLastError();
}

hipError_t launch_adam(hipStream_t s, int dtype, long n, const float* g, float* master, float* m, float* v, void* w,
                       float lr, float beta1, float beta2, float eps, int step) {
  if (n % 4 || step < 1) return hipErrorInvalidValue;
  const float inv_c1 = (float)(1.0 / (1.0 - pow((double)beta1, (double)step)));
  const float inv_c2 = (float)(1.0 / (1.0 - pow((double)beta2, (double)step)));
  const long n4 = n / 4;
  if (n4 == 0) return hipSuccess;
  return dtype == 0 ? adam_launch<float>(s, n4, g, master, m, v, (float*)w, lr, beta1, beta2, eps, inv_c1, inv_c2)
                    : adam_launch<bf16_t>(s, n4, g, master, m, v, (bf16_t*)w, lr, beta1, beta2, eps, inv_c1, inv_c2);
}

hipError_t launch_widen(hipStream_t s, int dtype, long n, const void* w, float* master) {
  if (n % 4) return hipErrorInvalidValue;
  const long n4 = n / 4;
  if (dtype == 0)
    hipLaunchKernelGGL(widen_kernel<float>, dim3(grid_for(n4)), dim3(256), 0, s, n4, (const float*)w, master);
  else
    hipLaunchKernelGGL(widen_kernel<bf16_t>, dim3(grid_for(n4)), dim3(256), 0, s, n4, (const bf16_t*)w, master);
  return hipGetLastError();
}

hipError_t launch_fill_zero(hipStream_t s, long n, float* p) {
  if (n % 4) return hipErrorInvalidValue;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(grid_for(n / 4)), dim3(256), 0, s, n / 4, p);
  return hipGetLastError();
}

}  // namespace bamboo
