// Whole layers of the fp32 configuration in one launch: a workgroup takes one sample through the forward of all layers
// of a stack, or through the input-gradient chain of one layer.
//
// With a few tokens per sample a layer is a chain of seven to ten kernels that each have microseconds of launch, of
// arguments and of memory round trips around well under a microsecond of work, and the host cannot enqueue them as fast
// as they run.  Samples do not meet before the weight gradients, so nothing but barriers inside a workgroup is needed
// between those steps: activations stay in LDS, memory sees the stash record and what the weight gradients read.
// See small_layers_fit for the figures and where the line lies.
//
// Products: v_mfma_f32_16x16x4_f32, sixteen wavefronts over column tiles of 16 and, where there are fewer tiles than
// wavefronts, over the contraction; the partial sums meet in LDS and are added in order by the threads that apply the
// epilogue.  Lane l of a step of 16 holds k = 4 (l / 16) .. + 3 of both operands, register j feeds instruction j.
// Bound by latency: a barrier, a trip to the L2 for weights and one through LDS per step.
#include "common.h"

namespace bamboo {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kThreads = 1024, kWaves = kThreads / 64;
constexpr int kChunk = 16 * kWaves;                    // output columns per pass of a product
constexpr int kPartLd = kChunk + 4;            // floats per row of partial sums

// The wavefronts meet, and what they have put in LDS is there.  Not __syncthreads, which also waits for every load and
// store on its way to memory; nothing that one thread writes to memory here is read by another.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__host__ __device__ inline int rows16(int S) { return (S + 15) / 16 * 16; }

// How the wavefronts share nc <= 256 output columns: tile, part of the contraction, columns a part's sums take
struct Share { int tile, part, parts, stride; bool idle; };
__device__ __forceinline__ Share share_of(int nc) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), tiles = (nc + 15) / 16;
  int p2 = 1;
  while (p2 < tiles) p2 *= 2;
  return {wave & (p2 - 1), wave / p2, kWaves / p2, p2 * 16, (wave & (p2 - 1)) >= tiles};
}

// Four steps of W for this lane, from step s0 on: b[u][j] = W at k = 16 (s0 + u) + 4 (lane / 16) + j, this lane's column.
// ROWS: W holds a row per output column (dX = dY W^T), else a row per k.  Its rows are 16-byte aligned, K a multiple of 8.
struct Frags { f32x4 b[4]; };
template <bool ROWS>
__device__ __forceinline__ void small_fetch(Frags& f, const float* W, int ldw, int K, int col, int s0) {
  const int kq = 4 * ((threadIdx.x & 63) >> 4);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int kc = min((s0 + u) * 16 + kq, K - 4);
    if (ROWS) {
      f.b[u] = *(const f32x4*)(W + (unsigned)(col * ldw + kc));
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) f.b[u][j] = W[(unsigned)((kc + j) * ldw + col)];
    }
  }
}
struct Span { int begin, end; };
__device__ __forceinline__ Span span_of(const Share& sh, int K) {
  const int steps = (K + 15) / 16, per = (steps + sh.parts - 1) / sh.parts;
  return {sh.part * per, min(steps, (sh.part + 1) * per)};
}
__device__ __forceinline__ int column_of(const Share& sh, int n0, int N) {
  return min(n0 + sh.tile * 16 + ((int)threadIdx.x & 15), N - 1);
}
// one product: its matrix, output columns and contraction
struct Product { const float* W; int ldw, N, K; };
// the first fragments of a product, requested while the step before it still runs
template <bool ROWS>
__device__ __forceinline__ void small_ahead(Frags& f, const Product& p) {
  const Share sh = share_of(min(kChunk, p.N));
  if (!sh.idle) small_fetch<ROWS>(f, p.W, p.ldw, p.K, column_of(sh, 0, p.N), span_of(sh, p.K).begin);
}

// part[row][part of K][column] = act[row][K] W over columns n0 .. n0 + nc - 1.  act in LDS, rows of lda floats, of which
// 16 TT may be read.  f: the first fragments.
template <int TT, bool ROWS>
__device__ __forceinline__ void small_gemm(Frags f, const float* act, int lda, const float* W, int ldw, int N, int K,
                                           int n0, int nc, float* part) {
  const Share sh = share_of(nc);
  if (sh.idle) return;
  const int lane = threadIdx.x & 63, i16 = lane & 15, kq = 4 * (lane >> 4);
  const int col = column_of(sh, n0, N);
  const Span sp = span_of(sh, K);
  f32x4 acc[TT][4] = {};        // every fourth k a sum of its own: short chains, and less rounding than one long one
  for (int s0 = sp.begin; s0 < sp.end; s0 += 4) {
    Frags next = f;
    if (s0 + 4 < sp.end) small_fetch<ROWS>(next, W, ldw, K, col, s0 + 4);
    const f32x4 zero = {};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (s0 + u >= sp.end) break;                    // uniform
      const int kb = (s0 + u) * 16 + kq, kc = min(kb, K - 4);
      const f32x4 b = kb < K ? f.b[u] : zero;
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        f32x4 a = *(const f32x4*)(act + (t * 16 + i16) * lda + kc);
        a = kb < K ? a : zero;
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], acc[t][j], 0, 0, 0);
      }
    }
    f = next;
  }
  // D[row][col]: lane holds col = lane % 16, rows 4 (lane / 16) .. + 3
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    const f32x4 v = (acc[t][0] + acc[t][1]) + (acc[t][2] + acc[t][3]);
#pragma unroll
    for (int r = 0; r < 4; ++r) part[(t * 16 + kq + r) * kPartLd + sh.part * sh.stride + sh.tile * 16 + i16] = v[r];
  }
}

// out(row, column, value, in(row, column)) once per output element of act W: a wavefront takes every 16th row, a lane
// every 64th column, so no index needs a division.  `in` is what the epilogue reads from memory, requested before the
// barrier, and so are the first fragments of the product after this one.  Ends behind a barrier.
template <int TT, bool ROWS, typename IN, typename OUT>
__device__ __forceinline__ void small_product(Frags& f, const float* act, int lda, const Product& g, const Product& after,
                                              int S, float* part, IN in, OUT out) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
#pragma unroll 1
  for (int n0 = 0; n0 < g.N; n0 += kChunk) {
    const int nc = min(kChunk, g.N - n0);
    const Share sh = share_of(nc);
    constexpr int RW = 16 * TT / kWaves, CW = kChunk / 64;     // rows a wavefront, columns a lane takes
    float pre[RW][CW];
#pragma unroll
    for (int i = 0; i < RW; ++i)
      if (wave + kWaves * i < S)
#pragma unroll
        for (int j = 0; j < CW; ++j) pre[i][j] = in(wave + kWaves * i, min(n0 + lane + 64 * j, g.N - 1));
    small_gemm<TT, ROWS>(f, act, lda, g.W, g.ldw, g.N, g.K, n0, nc, part);
    {
      const bool more = n0 + kChunk < g.N;
      const Product p = more ? g : after;
      const int m0 = more ? n0 + kChunk : 0;
      const Share sn = share_of(min(kChunk, p.N - m0));
      if (!sn.idle) small_fetch<ROWS>(f, p.W, p.ldw, p.K, column_of(sn, m0, p.N), span_of(sn, p.K).begin);
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < RW; ++i) {
      const int row = wave + kWaves * i;
      if (row < S) {
#pragma unroll
        for (int j = 0; j < CW; ++j) {
          const int c = lane + 64 * j;
          if (c < nc) {
            const float* q = part + row * kPartLd + c;
            float v = q[0];
#pragma unroll 1
            for (int k = 1; k < sh.parts; ++k) v += q[k * sh.stride];      // in order
            out(row, n0 + c, v, pre[i][j]);
          }
        }
      }
    }
    lds_barrier();
  }
}

__device__ __forceinline__ float half_sum(float v) {
  v = sum16(v);
  const float lo = of_lane(v, 0) + of_lane(v, 16), hi = of_lane(v, 32) + of_lane(v, 48);
  return (threadIdx.x & 32) ? hi : lo;
}
__device__ __forceinline__ float half_max(float v) {
  v = max16(v);
  const float lo = fmaxf(of_lane(v, 0), of_lane(v, 16)), hi = fmaxf(of_lane(v, 32), of_lane(v, 48));
  return (threadIdx.x & 32) ? hi : lo;
}
// sum over j < n of x[j * ld] times the weight that lane j of this half-wave holds; n <= most (uniform) <= 32
__device__ __forceinline__ float half_weighted(float weight, const float* x, int ld, int n, int most) {
  float o = 0.f;
#pragma unroll 1
  for (int j = 0; j < most; j += 4) {
    float y[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) y[u] = x[min(j + u, n - 1) * ld];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float lo = of_lane(weight, (j + u) & 31), hi = of_lane(weight, 32 + ((j + u) & 31));
      o = j + u < n ? fmaf((threadIdx.x & 32) ? hi : lo, y[u], o) : o;
    }
  }
  return o;
}

// A layer's vectors, in LDS: 9 H + F floats
struct SmallVectors {
  const float *bqkv, *bo, *g1, *be1, *b1, *b2, *g2, *be2;
};
__device__ __forceinline__ SmallVectors small_vectors(const SmallLayers& a, const float* w, float* v) {
  const int H = a.H, F = a.F;
  for (int c = threadIdx.x; c < 3 * H; c += kThreads) {
    v[c] = w[a.bqkv + c];                                  // bqkv
    v[3 * H + c] = w[a.bo + c];                            // bo, g1, be1 follow each other
    v[6 * H + c] = w[a.b2 + c];                            // b2, g2, be2
  }
  for (int c = threadIdx.x; c < F; c += kThreads) v[9 * H + c] = w[a.b1 + c];
  return {v, v + 3 * H, v + 4 * H, v + 5 * H, v + 9 * H, v + 6 * H, v + 7 * H, v + 8 * H};
}

// LayerNorm of the rows of `in` (LDS), a wavefront per row: out(row, column, value), stats[2 row], [2 row + 1]
template <typename OUT>
__device__ __forceinline__ void small_ln_fwd(const float* in, int ld, int S, int H, float eps, const float* gamma,
                                             const float* beta, float* stats, OUT out) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const bool live = lane < H;
  const float g = gamma[min(lane, H - 1)], b = beta[min(lane, H - 1)];
  for (int row = wave; row < S; row += kWaves) {
    const float v = live ? in[row * ld + lane] : 0.f;
    const float mean = wave_sum(v) / (float)H;
    const float rstd = rsqrtf(wave_sum(live ? (v - mean) * (v - mean) : 0.f) / (float)H + eps);
    if (live) out(row, lane, g * ((v - mean) * rstd) + b);
    if (lane == 0) {
      stats[2 * row] = mean;
      stats[2 * row + 1] = rstd;
    }
  }
}

struct SmallRecord {      // one layer's tensors of the sample at hand
  float *x, *ain, *qkv, *ctx, *r1, *fin, *g, *dg, *r2, *lse, *ln1, *ln2;
};
__device__ __forceinline__ SmallRecord record_of(const SmallLayers& a, int layer) {
  char* r = a.rec + layer * a.rec_bytes;
  const long t0 = (long)blockIdx.x * a.S;
  auto at = [&](long off, long per_token) { return (float*)(r + off) + t0 * per_token; };
  SmallRecord k;
  k.x = at(a.x, a.H); k.ain = at(a.ain, a.H); k.qkv = at(a.qkv, 3 * a.H); k.ctx = at(a.ctx, a.H);
  k.r1 = at(a.r1, a.H); k.fin = at(a.fin, a.H); k.g = at(a.g, a.F); k.dg = at(a.dg, a.F); k.r2 = at(a.r2, a.H);
  k.lse = at(a.lse, a.heads); k.ln1 = at(a.ln1, 2); k.ln2 = at(a.ln2, 2);
  return k;
}

// The steps are written out (one pass through common code for all of them: 27 instead of 22 us).
// TT: token tiles of 16 rows
template <int TT>
__global__ __launch_bounds__(kThreads) void small_fwd_kernel(SmallLayers a) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int S = a.S, H = a.H, F = a.F, R = 16 * TT, d = H / a.heads;
  const int LH = H + 4, LQ = 3 * H + 4, LF = F + 4;
  float* X = lds;                       // layer input
  float* A = X + R * LH;                // attention input (pre-LN), later FFN input
  float* C = A + R * LH;                // attention output
  float* Q = C + R * LH;                // queries | keys | values, later GELU(h)
  float* part = Q + R * max(LQ, LF);
  float* vec = part + R * kPartLd;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const long t0 = (long)blockIdx.x * S * H;
  const bool pre = a.pre_ln != 0;
  auto product = [&](const float* w, int step) __attribute__((always_inline)) {
    return step == 0 ? Product{w + a.Wqkv, 3 * H, 3 * H, H} : step == 1 ? Product{w + a.Wo, H, H, H}
         : step == 2 ? Product{w + a.W1, F, F, H} : Product{w + a.W2, H, H, F};
  };
  Frags f;
  small_ahead<false>(f, product(a.w, 0));
  {
    float* rx = record_of(a, 0).x;
    for (int row = wave; row < S; row += kWaves)
      for (int c = lane; c < H; c += 64) {
        const float v = a.in[t0 + row * H + c];
        X[row * LH + c] = v;
        rx[row * H + c] = v;
      }
  }
#pragma unroll 1
  for (int l = 0; l < a.n; ++l) {
    const SmallRecord k = record_of(a, l);
    const float* w = a.w + l * a.w_stride;
    float* next = l == a.n - 1 ? a.out + t0 : record_of(a, l + 1).x;
    const SmallVectors v = small_vectors(a, w, vec);
    lds_barrier();
    // step -1: LayerNorm ahead of the attention (pre-LN); 0: Q|K|V and attention; 1: its output, LayerNorm; 2, 3: FFN
#pragma unroll
    for (int step = -1; step < 4; ++step) {
      if (step == -1 && !pre) continue;
      if (step >= 0) {
        const float* act = step == 0 ? (pre ? A : X) : step == 1 ? C : step == 2 ? A : Q;
        const Product after = step < 3 ? product(w, step + 1) : product(l + 1 < a.n ? w + a.w_stride : w, 0);
        const float* bias = step == 0 ? v.bqkv : step == 1 ? v.bo : step == 2 ? v.b1 : v.b2;
        small_product<TT, false>(f, act, step == 3 ? LF : LH, product(w, step), after, S, part,
                                 [](int, int) { return 0.f; },
                                 [&](int row, int c, float y, float) {
          y += bias[c];
          if (step == 0) {
            Q[row * LQ + c] = y;
            k.qkv[row * 3 * H + c] = y;
          } else if (step == 2) {
            const float e = 0.5f * (1.0f + erff(y * 0.70710678118654752f)), g = y * e;
            Q[row * LF + c] = g;
            k.g[row * F + c] = g;
            k.dg[row * F + c] = e + y * __expf(-0.5f * y * y) * 0.39894228040143268f;
          } else {
            // r1 replaces the layer input (post-LN: no longer needed; pre-LN: it is the next residual), and r2 / the
            // layer's output replaces r1
            y += (step == 3 && !pre ? A : X)[row * LH + c];
            X[row * LH + c] = y;
            (step == 1 ? k.r1 : pre ? next : k.r2)[row * H + c] = y;
          }
        });
      }
      if (step == 0) {
        // attention: half a wavefront per (head, query), a key per lane, then a feature per lane
        const float scale = rsqrtf((float)d);
#pragma unroll 1
        for (int r0 = 2 * wave; r0 < a.heads * S; r0 += 2 * kWaves) {
          const int r = min(r0 + (lane >> 5), a.heads * S - 1), i32 = lane & 31;
          const int h = (int)(((float)r + 0.5f) / (float)S), q = r - h * S;
          const bool live = r == r0 + (lane >> 5);
          const float* qp = Q + q * LQ + h * d;
          const float* kp = Q + min(i32, S - 1) * LQ + H + h * d;
          float dot = 0.f;
#pragma unroll 4
          for (int c = 0; c < d; c += 4) {
            const f32x4 x = *(const f32x4*)(qp + c), y = *(const f32x4*)(kp + c);
#pragma unroll
            for (int j = 0; j < 4; ++j) dot = fmaf(x[j], y[j], dot);
          }
          const bool valid = i32 < S && (!pre || i32 <= q);
          const float sc = valid ? dot * scale : -INFINITY;
          const float m = half_max(sc);
          const float p = sc == -INFINITY ? 0.f : __expf(sc - m);
          const float sum = half_sum(p), inv = 1.f / sum;
#pragma unroll 1
          for (int c0 = 0; c0 < d; c0 += 32) {
            const int c = c0 + i32;
            const float o = half_weighted(p, Q + 2 * H + h * d + min(c, d - 1), LQ, pre ? q + 1 : S, S) * inv;
            if (c < d && live) {
              C[q * LH + h * d + c] = o;
              k.ctx[q * H + h * d + c] = o;
            }
          }
          if (i32 == 0 && live) k.lse[h * S + q] = m + __logf(sum);
        }
        lds_barrier();
      }
      if (step == -1 || step == 1 || (step == 3 && !pre)) {
        // its first or second LayerNorm; a wavefront's row is its own, so in place where the layer's output is made
        const bool second = pre ? step == 1 : step == 3;
        float* dst = step == 3 ? X : A;
        float* mem = step == -1 ? k.ain : step == 1 ? k.fin : next;
        small_ln_fwd(X, LH, S, H, a.eps, second ? v.g2 : v.g1, second ? v.be2 : v.be1, second ? k.ln2 : k.ln1,
                     [&](int row, int c, float y) {
                       dst[row * LH + c] = y;
                       mem[row * H + c] = y;
                     });
        lds_barrier();
      }
    }
  }
}

// Column sums over the sample's rows: out[c] = sum of x[row][c] (times y[row][c]), every fourth row in a sum of its own
struct Sum { const float *x, *y; float* out; int ld, N; };
// up to three of them, by threads 0 .., 256 .. and 512 .. of the workgroup
__device__ __forceinline__ void small_colsums(const Sum (&s)[3], int S) {
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if (s[q].out == nullptr) continue;              // uniform
#pragma unroll 1
    for (int c = ((int)threadIdx.x - 256 * q) & (kThreads - 1); c < s[q].N; c += kThreads) {
      float t[4] = {};
#pragma unroll 1
      for (int row = 0; row < S; row += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int at = min(row + u, S - 1) * s[q].ld + c;
          const float x = s[q].x[at], v = s[q].y != nullptr ? x * s[q].y[at] : x;
          t[u] += row + u < S ? v : 0.f;
        }
      }
      s[q].out[c] = (t[0] + t[1]) + (t[2] + t[3]);
    }
  }
}

// The input-gradient chain of one layer (the record at a.rec, weights at a.w); what the weight gradients read goes to
// the buffers of b, one row of column sums per sample to its partial rows.
template <int TT>
__global__ __launch_bounds__(kThreads) void small_bwd_kernel(SmallLayers a, SmallBackward b) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const int S = a.S, H = a.H, F = a.F, R = 16 * TT, d = H / a.heads;
  const int LH = H + 4, LQ = 3 * H + 4, LF = F + 4;
  float* D0 = lds;                      // gradient at the FFN output
  float* D2 = D0 + R * LH;              // gradient at the FFN input, later at the attention input
  float* DA = D2 + R * LH;              // gradient at the attention block's output
  float* DC = DA + R * LH;              // r1, its normalised rows, then the gradient at ctx
  float* CT = DC + R * LH;              // ctx
  float* Q = CT + R * LH;               // queries | keys | values
  float* DH = Q + R * LQ;               // gradient at h, later
  float* DQ = DH;                       // at queries | keys | values
  float* part = DH + R * max(LF, LQ);
  float* vec = part + R * kPartLd;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const SmallRecord k = record_of(a, 0);
  const float* w = a.w;
  const long s = blockIdx.x, t0 = s * S;
  const bool pre = a.pre_ln != 0;
  auto product = [&](int step) __attribute__((always_inline)) {
    return step == 0 ? Product{w + a.W2, H, F, H} : step == 1 ? Product{w + a.W1, F, H, F}
         : step == 2 ? Product{w + a.Wo, H, H, H} : Product{w + a.Wqkv, 3 * H, H, 3 * H};
  };
  Frags f;
  small_ahead<true>(f, product(0));
  for (int row = wave; row < S; row += kWaves) {
    for (int c = lane; c < H; c += 64) {
      (pre ? D0 : D2)[row * LH + c] = a.in[(t0 + row) * H + c];
      DC[row * LH + c] = k.r1[row * H + c];
      CT[row * LH + c] = k.ctx[row * H + c];
      if (!pre) DA[row * LH + c] = k.r2[row * H + c];
    }
    for (int c = lane; c < 3 * H; c += 64) Q[row * LQ + c] = k.qkv[row * 3 * H + c];
  }
  const SmallVectors v = small_vectors(a, w, vec);
  lds_barrier();
  // step -1: LayerNorm behind the FFN (post-LN); 0, 1: FFN, LayerNorm; 2: attention; 3: its input, LayerNorm (pre-LN)
#pragma unroll
  for (int step = -1; step < 4; ++step) {
    if (step == -1 && pre) continue;
    Sum sums[3] = {};
    if (step >= 0) {
      const float* act = step == 0 ? D0 : step == 1 ? DH : step == 2 ? DA : DQ;
      small_product<TT, true>(f, act, step == 1 ? LF : step == 3 ? LQ : LH, product(step), product(step < 3 ? step + 1 : 3),
                              S, part, [&](int row, int c) { return step == 0 ? k.dg[row * F + c] : 0.f; },
                              [&](int row, int c, float y, float dg) {
        if (step == 0) {
          y *= dg;
          DH[row * LF + c] = y;
          b.dh[(t0 + row) * F + c] = y;
        } else {
          if (!pre && step != 2) y += (step == 1 ? D0 : DA)[row * LH + c];
          (step == 2 ? DC : D2)[row * LH + c] = y;
          (step == 2 ? b.dctx : step == 1 ? (pre ? b.d1 : b.d2) : pre ? b.d1 : a.out)[(t0 + row) * H + c] = y;
        }
      });
    }
    if (step == 0) {
      sums[0] = {DH, nullptr, b.p_dh + s * F, LF, F};
      if (pre) sums[1] = {D0, nullptr, b.p_df + s * H, LH, H};
    }
    if (step == 2) {
      // attention, a group of heads at a time: probabilities and score gradients of the group in the place of `part`
      const float scale = rsqrtf((float)d);
      const int LS = S + 1, group = kPartLd / (2 * LS);        // S <= 32: at least three heads
#pragma unroll 1
      for (int h0 = 0; h0 < a.heads; h0 += group) {
        const int hn = min(group, a.heads - h0);
        float* P = part;
        float* dS = part + hn * S * LS;
#pragma unroll 1
        for (int r0 = 2 * wave; r0 < hn * S; r0 += 2 * kWaves) {       // as in the forward
          const int r = min(r0 + (lane >> 5), hn * S - 1), i32 = lane & 31;
          const int hh = (int)(((float)r + 0.5f) / (float)S), q = r - hh * S, h = h0 + hh;
          const bool live = r == r0 + (lane >> 5);
          const float* qp = Q + q * LQ + h * d;
          const float* gp = DC + q * LH + h * d;
          const float* kp = Q + min(i32, S - 1) * LQ + H + h * d;
          const float lse = k.lse[h * S + q];
          float dot = 0.f, dp = 0.f, delta = 0.f;
#pragma unroll 1
          for (int c = i32; c < d; c += 32) delta += CT[q * LH + h * d + c] * gp[c];
#pragma unroll 4
          for (int c = 0; c < d; c += 4) {
            const f32x4 x = *(const f32x4*)(qp + c), y = *(const f32x4*)(kp + c);
            const f32x4 g = *(const f32x4*)(gp + c), z = *(const f32x4*)(kp + H + c);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              dot = fmaf(x[j], y[j], dot);
              dp = fmaf(g[j], z[j], dp);
            }
          }
          delta = half_sum(delta);
          const bool valid = i32 < S && (!pre || i32 <= q);
          const float p = valid ? __expf(dot * scale - lse) : 0.f;
          const float ds = valid ? p * (dp - delta) : 0.f;
          if (i32 < S && live) {
            P[r * LS + i32] = p;
            dS[r * LS + i32] = ds;
          }
#pragma unroll 1
          for (int c0 = 0; c0 < d; c0 += 32) {
            const int c = c0 + i32;
            const float o = half_weighted(ds, Q + H + h * d + min(c, d - 1), LQ, pre ? q + 1 : S, S) * scale;
            if (c < d && live) DQ[q * LQ + h * d + c] = o;
          }
        }
        lds_barrier();
#pragma unroll 1
        for (int r = 2 * wave + (lane >> 5); r < hn * S; r += 2 * kWaves) {
          const int hh = (int)(((float)r + 0.5f) / (float)S), j = r - hh * S;
#pragma unroll 1
          for (int c = lane & 31; c < d; c += 32) {
            const int i = (h0 + hh) * d + c;
            float dk = 0.f, dv = 0.f;
#pragma unroll 4
            for (int q = pre ? j : 0; q < S; ++q) {
              dk = fmaf(dS[(hh * S + q) * LS + j], Q[q * LQ + i], dk);
              dv = fmaf(P[(hh * S + q) * LS + j], DC[q * LH + i], dv);
            }
            DQ[j * LQ + H + i] = dk * scale;
            DQ[j * LQ + 2 * H + i] = dv;
          }
        }
        lds_barrier();
      }
      for (int row = wave; row < S; row += kWaves)
        for (int c = lane; c < 3 * H; c += 64) b.dqkv[(t0 + row) * 3 * H + c] = DQ[row * LQ + c];
      sums[0] = {DQ, nullptr, b.p_dqkv + s * 3 * H, LQ, 3 * H};
    }
    if (step == -1 || step == 1 || (step == 3 && pre)) {
      // LayerNorm backward of D2's rows, a wavefront per row; the rows it normalised go in place of its input `xh`, from
      // which and from D2 the gain and shift gradients are summed, and from its result the bias gradient before it
      const bool second = pre ? step == 1 : step == -1;
      const float* stats = second ? k.ln2 : k.ln1;
      const float* gamma = second ? v.g2 : v.g1;
      const float* add = pre ? (step == 1 ? D0 : DA) : nullptr;
      float* xh = step == -1 ? DA : DC;
      float* dr = step == 1 ? DA : D0;
      float* mem = (step == -1 ? b.d3 : step == 1 ? (pre ? b.d2 : b.d1) : a.out) + t0 * H;
#pragma unroll 1
      for (int row = wave; row < S; row += kWaves) {
        const float mean = stats[2 * row], rstd = stats[2 * row + 1];
        const bool live = lane < H;
        const float in = live ? (step == 3 ? k.x[row * H + lane] : xh[row * LH + lane]) : 0.f;
        const float x = live ? (in - mean) * rstd : 0.f;
        const float dh = live ? D2[row * LH + lane] * gamma[lane] : 0.f;
        const float m1 = wave_sum(dh) / (float)H, m2 = wave_sum(dh * x) / (float)H;
        if (live) {
          float o = (dh - m1 - x * m2) * rstd;
          if (add != nullptr) o += add[row * LH + lane];
          xh[row * LH + lane] = x;
          dr[row * LH + lane] = o;
          mem[row * H + lane] = o;
        }
      }
      const int set = second ? 1 : 0;
      sums[0] = {D2, xh, b.p_ln[set][0] + s * H, LH, H};
      sums[1] = {D2, nullptr, b.p_ln[set][1] + s * H, LH, H};
      if (step != 3) sums[2] = {dr, nullptr, b.p_ln[set][2] + s * H, LH, H};
      lds_barrier();
    }
    small_colsums(sums, S);
    if (step == -1 || step == 1) lds_barrier();       // the buffers that were summed are written again
  }
}

static int fwd_lds_bytes(int S, int H, int F) {
  return 4 * (rows16(S) * (3 * (H + 4) + (3 * H > F ? 3 * H : F) + 4 + kPartLd) + 9 * H + F);
}
static int bwd_lds_bytes(int S, int H, int F) {
  return 4 * (rows16(S) * (5 * (H + 4) + 3 * H + 4 + (3 * H > F ? 3 * H : F) + 4 + kPartLd) + 9 * H + F);
}

// A wavefront holds a row of a LayerNorm in one register and half of one the keys of a query; beyond that the line lies
// where a CU per sample stops being faster than the chip per step: the products of a row tile (up to 16 rows: more passes over
// the FFN's columns still pay; 32 rows: one pass of 256 does), and the scores, of which a CU takes 32 queries' at a time.
// An iteration of 3 micro-batches through 2 + 2 layers, 1 x tokens, H, heads, F, steps launched one by one / this, us:
//   12,  64,  1, 256 (144 scores)   535 / 372      20, 64,  4, 256 (1600)  538 / 545      32, 64,  1,  256 (1024)  628 / 589
//   16,  64,  4, 256 (1024)         534 / 413      24, 64,  4, 256 (2304)  534 / 591      32, 64,  2,  256 (2048)  540 / 588
//   16,  64,  8, 256 (2048)         503 / 502      32, 64,  4, 256 (4096)  538 / 712      32, 64, 16,  256 (16384) 701 / 1492
//   16,  64,  8, 640 (2048)         590 / 614      17, 64,  1, 512 (289)   633 / 702      17, 32,  1, 1024 (289)   613 / 725
//   16,  64,  4, 640 (1024)         592 / 535      26, 64,  2, 256 (1352)  615 / 549      13, 64,  8,  640 (1352)  568 / 570
// The steps are bound by the host, which is up to a quarter faster on one machine than on another; the line is drawn for a
// fast one.  Over 158 configurations inside it, 1 and 8 samples: 0.47 to 1.02 of the steps' time, 0.72 at the median.  With
// 256 samples of 16 tokens 704 / 624, wider layers (96 columns, 1.8 M multiply-adds) 843 / 1026.
// The forward of 2 x 16 tokens, 64, 2, 256 is one launch of 22 us, the backward 29 us and the weight gradients.  Sums split
// four ways (small_gemm, small_colsums) cost 1 % at 16 tokens a sample and 5 % at 32 over one sum each, with which weight
// gradients were 1.3 and bias gradients up to 1.9 times as far from 64 bits as the single kernels' (1.5e-7, 1.6e-7), now 1.04
// and 1.0.  128 registers a thread at 1024 threads: small_fwd_kernel<2> spills 32 of them (84 bytes), the others one or two.
bool small_layers_fit(int B, int S, int H, int heads, int F) {
  const long macs = rows16(S) * (4L * H * H + 2L * H * F), scores = (long)heads * S * S;
  const bool brief = S <= 16 ? macs <= 2000000 && scores + macs / 2000 <= 2000 : F <= 256 && scores <= 1400;
  return S <= 32 && H <= 64 && (H / heads) % 4 == 0 && brief &&
         (size_t)B <= reduce_max_partials() && bwd_lds_bytes(S, H, F) <= 160 * 1024;
}

template <int TT>
static hipError_t fwd_launch(hipStream_t s, int B, const SmallLayers& a) {
  const hipError_t e = ensure_lds_attribute<small_fwd_kernel<TT>, 160 * 1024>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(small_fwd_kernel<TT>, dim3(B), dim3(kThreads), fwd_lds_bytes(a.S, a.H, a.F), s, a);
  return hipGetLastError();
}
template <int TT>
static hipError_t bwd_launch(hipStream_t s, int B, const SmallLayers& a, const SmallBackward& b) {
  const hipError_t e = ensure_lds_attribute<small_bwd_kernel<TT>, 160 * 1024>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(small_bwd_kernel<TT>, dim3(B), dim3(kThreads), bwd_lds_bytes(a.S, a.H, a.F), s, a, b);
  return hipGetLastError();
}
hipError_t launch_small_fwd(hipStream_t s, int B, const SmallLayers& a) {
  return a.S <= 16 ? fwd_launch<1>(s, B, a) : fwd_launch<2>(s, B, a);
}
hipError_t launch_small_bwd(hipStream_t s, int B, const SmallLayers& a, const SmallBackward& b) {
  return a.S <= 16 ? bwd_launch<1>(s, B, a, b) : bwd_launch<2>(s, B, a, b);
}

}  // namespace bamboo
