// Softmax attention forward/backward on the vector ALUs (fp32 arithmetic, any
// sequence length, head size up to 128).  Used by the fp32 configuration and as
// the fallback of the bf16 path.  Online softmax over key tiles; the forward
// keeps only the per-row log-sum-exp, the backward recomputes the
// probabilities from it.  No atomics: dQ and dK/dV come from two kinds of
// workgroups, of one launch, that each own their output rows, so results are
// bitwise reproducible.
//
// The fp32 configuration has a few dozen tokens: its launches are one or a few
// workgroups whose time is a chain of memory round trips, so a thread requests
// all it needs of a tile before it waits (8 tokens, 2 samples x 2 heads of 32:
// forward 8.0 us with one load per trip), and the backward is one launch that
// forms delta = rowsum(ctx * dctx) where it is needed (three launches of 5.6,
// 8.6 and 13.0 us before).
#include "common.h"

namespace bamboo {

constexpr int QT = 16;  // rows owned by a block
constexpr int KT = 32;  // rows streamed per tile

// dst0/dst1[r][c] = src0/src1[(row0 + r) * stride + c] for r < nrows, zero from row_limit on: eight elements of each
// per thread in flight.  Rows past the limit are read from the last valid one, so that no load sits behind a branch.
template <typename T>
__device__ __forceinline__ void load_tiles(float* dst0, const T* src0, long stride0, float* dst1, const T* src1,
                                           long stride1, int ld, int row0, int nrows, int row_limit, int D) {
  const int n = nrows * D, dr = 256 / D, dc = 256 % D;
  int r = threadIdx.x / D, c = threadIdx.x % D;
  for (int i0 = threadIdx.x; i0 < n; i0 += 8 * 256) {
    T v0[8], v1[8];
    int at[8];
    bool live[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const long row = min(row0 + r, row_limit - 1);
      v0[u] = src0[row * stride0 + c];
      v1[u] = src1[row * stride1 + c];
      at[u] = r * ld + c;
      live[u] = row0 + r < row_limit;
      r += dr;
      c += dc;
      if (c >= D) { c -= D; ++r; }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i0 + u * 256 < n) {
        dst0[at[u]] = live[u] ? to_f32<T>(v0[u]) : 0.f;
        dst1[at[u]] = live[u] ? to_f32<T>(v1[u]) : 0.f;
      }
  }
}

__device__ __forceinline__ float group16_max(float v) {
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float group16_sum(float v) {
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// sum of x[c] y[c] over c = first, first + STEP, ... < n, four products in flight
template <int STEP, typename T>
__device__ __forceinline__ float strided_dot(const T* x, const T* y, int first, int n) {
  float s = 0.f;
  for (int c0 = first; c0 < n; c0 += 4 * STEP) {
    T p[4], q[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = min(c0 + u * STEP, n - 1);
      p[u] = x[c];
      q[u] = y[c];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) s += c0 + u * STEP < n ? to_f32<T>(p[u]) * to_f32<T>(q[u]) : 0.f;
  }
  return s;
}

template <typename T>
__global__ __launch_bounds__(256) void attn_fwd_simple_kernel(AttnDesc a) {
  extern __shared__ float smem[];
  const int D = a.d, ld = D + 1, H = a.heads * D;
  float* Qs = smem;
  float* Ks = Qs + QT * ld;
  float* Vs = Ks + KT * ld;
  float* Ps = Vs + KT * ld;  // [QT][KT+1]
  const int b = blockIdx.y / a.heads, h = blockIdx.y % a.heads;
  const int q0 = blockIdx.x * QT;
  const int q = threadIdx.x / 16, t = threadIdx.x % 16;
  const T* base = (const T*)a.qkv + (long)b * a.S * 3 * H + h * D;
  const float scale = rsqrtf((float)D);
  load_tiles<T>(Qs, base, 3 * H, Qs, base, 3 * H, ld, q0, QT, a.S, D);
  const int qrow = q0 + q;
  float m = -INFINITY, l = 0.f, o[8] = {};
  const int kend = a.causal ? min(a.S, q0 + QT) : a.S;
  for (int k0 = 0; k0 < kend; k0 += KT) {
    __syncthreads();
    load_tiles<T>(Ks, base + H, 3 * H, Vs, base + 2 * H, 3 * H, ld, k0, min(KT, kend - k0), a.S, D);
    const int jn = min(KT, kend - k0);              // keys of this tile that any of the block's queries sees
    __syncthreads();
    float sc[2];
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      const int j = t + 16 * jj, key = k0 + j;
      const bool valid = key < a.S && qrow < a.S && (!a.causal || key <= qrow);
      float dot = 0.f;
      if (j < jn) {
#pragma unroll 8
        for (int c = 0; c < D; ++c) dot = fmaf(Qs[q * ld + c], Ks[j * ld + c], dot);
      }
      sc[jj] = valid ? dot * scale : -INFINITY;
    }
    const float mnew = fmaxf(m, group16_max(fmaxf(sc[0], sc[1])));
    const float corr = (m == -INFINITY) ? 0.f : __expf(m - mnew);
    float psum = 0.f;
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      const float p = (sc[jj] == -INFINITY) ? 0.f : __expf(sc[jj] - mnew);
      Ps[q * (KT + 1) + t + 16 * jj] = p;
      psum += p;
    }
    l = l * corr + group16_sum(psum);
    m = mnew;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = t + 16 * e;
      if (c < D) {
        float acc = o[e] * corr;
#pragma unroll 8
        for (int j = 0; j < jn; ++j) acc = fmaf(Ps[q * (KT + 1) + j], Vs[j * ld + c], acc);
        o[e] = acc;
      }
    }
  }
  if (qrow < a.S) {
    const float inv = 1.f / l;
    T* out = (T*)a.ctx + ((long)b * a.S + qrow) * H + h * D;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = t + 16 * e;
      if (c < D) out[c] = from_f32<T>(o[e] * inv);
    }
    if (t == 0) a.lse[((long)b * a.heads + h) * a.S + qrow] = m + __logf(l);
  }
}

// dQ: a block owns QT query rows and streams the keys.
template <typename T>
__device__ __forceinline__ void bwd_dq_block(const AttnDesc& a, int blk, float* smem) {
  const int D = a.d, ld = D + 1, H = a.heads * D;
  float* Qs = smem;
  float* dOs = Qs + QT * ld;
  float* Ks = dOs + QT * ld;
  float* Vs = Ks + KT * ld;
  float* dSs = Vs + KT * ld;  // [QT][KT+1]
  const int b = blockIdx.y / a.heads, h = blockIdx.y % a.heads;
  const int q0 = blk * QT;
  const int q = threadIdx.x / 16, t = threadIdx.x % 16;
  const T* base = (const T*)a.qkv + (long)b * a.S * 3 * H + h * D;
  const T* dbase = (const T*)a.dctx + (long)b * a.S * H + h * D;
  const float scale = rsqrtf((float)D);
  load_tiles<T>(Qs, base, 3 * H, dOs, dbase, H, ld, q0, QT, a.S, D);
  const int qrow = q0 + q, qv = min(qrow, a.S - 1);
  const float lse = a.lse[((long)b * a.heads + h) * a.S + qv];
  // delta of the row: its sixteen threads take every sixteenth feature
  float delta;
  {
    const T* o = (const T*)a.ctx + ((long)b * a.S + qv) * H + h * D;
    const T* dO = dbase + (long)qv * H;
    delta = group16_sum(strided_dot<16>(o, dO, t, D));
    if (t == 0 && qrow < a.S) a.delta[((long)b * a.heads + h) * a.S + qrow] = delta;   // for the caller
  }
  float dq[8] = {};
  const int kend = a.causal ? min(a.S, q0 + QT) : a.S;
  for (int k0 = 0; k0 < kend; k0 += KT) {
    __syncthreads();
    load_tiles<T>(Ks, base + H, 3 * H, Vs, base + 2 * H, 3 * H, ld, k0, min(KT, kend - k0), a.S, D);
    const int jn = min(KT, kend - k0);              // keys of this tile that any of the block's queries sees
    __syncthreads();
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      const int j = t + 16 * jj, key = k0 + j;
      const bool valid = key < a.S && qrow < a.S && (!a.causal || key <= qrow);
      float dot = 0.f, dp = 0.f;
      if (j < jn) {
#pragma unroll 8
        for (int c = 0; c < D; ++c) {
          dot = fmaf(Qs[q * ld + c], Ks[j * ld + c], dot);
          dp = fmaf(dOs[q * ld + c], Vs[j * ld + c], dp);
        }
      }
      const float p = valid ? __expf(dot * scale - lse) : 0.f;
      dSs[q * (KT + 1) + j] = p * (dp - delta);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = t + 16 * e;
      if (c < D) {
        float acc = dq[e];
#pragma unroll 8
        for (int j = 0; j < jn; ++j) acc = fmaf(dSs[q * (KT + 1) + j], Ks[j * ld + c], acc);
        dq[e] = acc;
      }
    }
  }
  if (qrow < a.S) {
    T* out = (T*)a.dqkv + ((long)b * a.S + qrow) * 3 * H + h * D;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = t + 16 * e;
      if (c < D) out[c] = from_f32<T>(dq[e] * scale);
    }
  }
}

// dK, dV: a block owns QT key rows and streams the queries.
template <typename T>
__device__ __forceinline__ void bwd_dkv_block(const AttnDesc& a, int blk, float* smem) {
  const int D = a.d, ld = D + 1, H = a.heads * D;
  float* Ks = smem;
  float* Vs = Ks + QT * ld;
  float* Qs = Vs + QT * ld;
  float* dOs = Qs + KT * ld;
  float* Ps = dOs + KT * ld;      // [KT][QT+1]
  float* dSs = Ps + KT * (QT + 1);  // [KT][QT+1]
  float* lse_s = dSs + KT * (QT + 1);  // [KT]
  float* del_s = lse_s + KT;           // [KT]
  const int b = blockIdx.y / a.heads, h = blockIdx.y % a.heads;
  const int k0 = blk * QT;
  const int j = threadIdx.x / 16, t = threadIdx.x % 16;
  const T* base = (const T*)a.qkv + (long)b * a.S * 3 * H + h * D;
  const T* dbase = (const T*)a.dctx + (long)b * a.S * H + h * D;
  const float scale = rsqrtf((float)D);
  load_tiles<T>(Ks, base + H, 3 * H, Vs, base + 2 * H, 3 * H, ld, k0, QT, a.S, D);
  const int key = k0 + j;
  float dk[8] = {}, dv[8] = {};
  const int qbeg = a.causal ? (k0 / KT) * KT : 0;
  for (int q0 = qbeg; q0 < a.S; q0 += KT) {
    __syncthreads();
    const int in = min(KT, a.S - q0);               // queries of this tile
    {
      // delta and the log-sum-exp of the tile's queries: eight threads a row, straight from memory, so that these
      // loads travel with those of the tile
      const int i = threadIdx.x >> 3, e = threadIdx.x & 7, row = min(q0 + i, a.S - 1);
      const T* o = (const T*)a.ctx + ((long)b * a.S + row) * H + h * D;
      const T* dO = dbase + (long)row * H;
      const float lse = a.lse[((long)b * a.heads + h) * a.S + row];
      float delta = strided_dot<8>(o, dO, e, D);
#pragma unroll
      for (int x = 4; x > 0; x >>= 1) delta += __shfl_xor(delta, x, 64);
      if (e == 0) {
        lse_s[i] = lse;
        del_s[i] = delta;
      }
    }
    load_tiles<T>(Qs, base, 3 * H, dOs, dbase, H, ld, q0, in, a.S, D);
    __syncthreads();
#pragma unroll
    for (int ii = 0; ii < 2; ++ii) {
      const int i = t + 16 * ii, qrow = q0 + i;
      const bool valid = key < a.S && qrow < a.S && (!a.causal || key <= qrow);
      float dot = 0.f, dp = 0.f;
      if (i < in) {
#pragma unroll 8
        for (int c = 0; c < D; ++c) {
          dot = fmaf(Qs[i * ld + c], Ks[j * ld + c], dot);
          dp = fmaf(dOs[i * ld + c], Vs[j * ld + c], dp);
        }
      }
      float p = 0.f, ds = 0.f;
      if (valid) {
        p = __expf(dot * scale - lse_s[i]);
        ds = p * (dp - del_s[i]);
      }
      Ps[i * (QT + 1) + j] = p;
      dSs[i * (QT + 1) + j] = ds;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = t + 16 * e;
      if (c < D) {
        float av = dv[e], ak = dk[e];
#pragma unroll 8
        for (int i = 0; i < in; ++i) {
          av = fmaf(Ps[i * (QT + 1) + j], dOs[i * ld + c], av);
          ak = fmaf(dSs[i * (QT + 1) + j], Qs[i * ld + c], ak);
        }
        dv[e] = av;
        dk[e] = ak;
      }
    }
  }
  if (key < a.S) {
    T* out = (T*)a.dqkv + ((long)b * a.S + key) * 3 * H + h * D;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = t + 16 * e;
      if (c < D) {
        out[H + c] = from_f32<T>(dk[e] * scale);
        out[2 * H + c] = from_f32<T>(dv[e]);
      }
    }
  }
}

// Both passes in one launch: workgroups 0 .. nblk-1 of a (sample, head) own query rows, the others key rows.
template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_simple_kernel(AttnDesc a, int nblk) {
  extern __shared__ float smem[];
  if ((int)blockIdx.x < nblk) bwd_dq_block<T>(a, blockIdx.x, smem);
  else bwd_dkv_block<T>(a, (int)blockIdx.x - nblk, smem);
}

template <typename T>
static hipError_t fwd_impl(hipStream_t s, const AttnDesc& a) {
  const size_t sh = ((size_t)(QT + 2 * KT) * (a.d + 1) + QT * (KT + 1)) * sizeof(float);
  dim3 grid((a.S + QT - 1) / QT, a.B * a.heads);
  hipLaunchKernelGGL(attn_fwd_simple_kernel<T>, grid, dim3(256), sh, s, a);
  return hipGetLastError();
}

template <typename T>
static hipError_t bwd_impl(hipStream_t s, const AttnDesc& a) {
  const int nblk = (a.S + QT - 1) / QT;
  const size_t tiles = (size_t)(2 * QT + 2 * KT) * (a.d + 1);
  constexpr size_t kOwn = 2 * KT * (QT + 1) + 2 * KT;      // scores and row statistics of a key owner
  static_assert(kOwn >= QT * (KT + 1), "the key owners need the most LDS");
  hipLaunchKernelGGL(attn_bwd_simple_kernel<T>, dim3(2 * nblk, a.B * a.heads), dim3(256),
                     (tiles + kOwn) * sizeof(float), s, a, nblk);
  return hipGetLastError();
}

hipError_t launch_attention_fwd_simple(hipStream_t s, int dtype, const AttnDesc& a) {
  if (a.d > 128) return hipErrorInvalidValue;
  return dtype == 0 ? fwd_impl<float>(s, a) : fwd_impl<bf16_t>(s, a);
}
hipError_t launch_attention_bwd_simple(hipStream_t s, int dtype, const AttnDesc& a) {
  if (a.d > 128) return hipErrorInvalidValue;
  return dtype == 0 ? bwd_impl<float>(s, a) : bwd_impl<bf16_t>(s, a);
}

hipError_t launch_attention_fwd(hipStream_t s, int dtype, const AttnDesc& a) {
  if (dtype == 1) {
    hipError_t e = launch_attention_fwd_mfma(s, a);
    if (e != hipErrorNotSupported) return e;
  }
  return launch_attention_fwd_simple(s, dtype, a);
}
hipError_t launch_attention_bwd(hipStream_t s, int dtype, const AttnDesc& a) {
  if (dtype == 1) {
    hipError_t e = launch_attention_bwd_mfma(s, a);
    if (e != hipErrorNotSupported) return e;
  }
  return launch_attention_bwd_simple(s, dtype, a);
}

}  // namespace bamboo
