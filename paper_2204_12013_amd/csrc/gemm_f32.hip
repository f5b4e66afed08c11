// fp32 GEMM on the gfx950 matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, fp32 accumulation) for the fp32
// configuration.  One wavefront owns a 32 x 32 output tile and takes its operands straight from memory: a 32-bit
// matrix instruction works 64 clocks on two fragments, so the vector L1 feeds all four SIMDs without LDS in
// between.  Which k a fragment register stands for is free as long as both operands agree: lane l of a step of 8
// holds row (column) l % 32 and k = 4 * (l / 32) .. + 3, i.e. one 16-byte load of a K-contiguous operand, and four
// loads of 128 contiguous bytes per half-wave of a row-contiguous one; register j of both feeds instruction j.
//
// A layer of the fp32 configuration has 32 tokens and matrices of 64 x 64 to 64 x 256: a launch is a handful of
// tiles, and its time is the serial chain through K.  So the NW wavefronts of a workgroup share ONE tile and take
// every NW-th step; their partial tiles are summed through LDS in wavefront order.  Larger outputs (more tiles than
// wavefront slots) take one wavefront per tile instead.
#include <string.h>

#include "common.h"
#include "reduce_device.h"

namespace bamboo {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// Four k values (kb .. kb+3) of row `row`; KC: contraction index contiguous.  Zero beyond the edges.
template <bool KC, bool VEC>
__device__ __forceinline__ f32x4 frag4(const float* p, long s_row, long s_k, int row, int rows, int kb, int K) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (row >= rows) return v;
  if (KC) {
    const float* q = p + (long)row * s_row + kb;
    if (VEC) {                                    // K a multiple of 4 and 16-byte rows
      if (kb < K) v = *(const f32x4*)q;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) if (kb + j < K) v[j] = q[j];
    }
  } else {
    const float* q = p + (long)kb * s_k + row;
#pragma unroll
    for (int j = 0; j < 4; ++j) if (kb + j < K) v[j] = q[(long)j * s_k];
  }
  return v;
}

__device__ __forceinline__ void epilogue1(const GemmDesc& d, int m, int n, float acc) {
  const long i = (long)m * d.N + n;
  float* C = (float*)d.C;
  switch (d.epi) {
    case EPI_STORE: C[i] = acc; break;
    case EPI_BIAS: C[i] = acc + ((const float*)d.bias)[n]; break;
    case EPI_BIAS_RES: C[i] = acc + ((const float*)d.bias)[n] + ((const float*)d.res)[i]; break;
    case EPI_BIAS_GELU: {
      const float h = acc + ((const float*)d.bias)[n];
      C[i] = gelu_grad_f(h);
      ((float*)d.aux_out)[i] = gelu_f(h);
      break;
    }
    case EPI_RES: C[i] = acc + ((const float*)d.res)[i]; break;
    case EPI_MUL: C[i] = acc * ((const float*)d.aux_in)[i]; break;
    case EPI_ACC_F32: C[i] += acc; break;
  }
}

constexpr int kStepK = 8;      // k of one step (four matrix instructions)
constexpr int kAhead = 4;      // steps whose operands a wavefront requests together

// SPLIT: the workgroup's NW wavefronts share one tile; otherwise each has a tile of its own.  blk: workgroup of the problem
template <bool A_K, bool B_K, bool VEC, int NW, bool SPLIT>
__device__ __forceinline__ void gemm_f32_block(const GemmDesc& d, int blk, float (*part)[32 * 33]) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tiles_n = (d.N + 31) / 32, tiles = ((d.M + 31) / 32) * tiles_n;
  const int tile = SPLIT ? blk : blk * NW + wave;
  if (!SPLIT && tile >= tiles) return;
  const int m0 = (tile / tiles_n) * 32, n0 = (tile % tiles_n) * 32;
  const float* A = (const float*)d.A;
  const float* B = (const float*)d.B;
  const int row = m0 + (lane & 31), col = n0 + (lane & 31), kh = 4 * (lane >> 5);
  f32x16 acc = {};
  const int first = SPLIT ? wave : 0, stride = SPLIT ? NW : 1;
  const int steps = (d.K + kStepK - 1) / kStepK;
  for (int s0 = first; s0 < steps; s0 += stride * kAhead) {
    f32x4 a[kAhead], b[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int kb = (s0 + u * stride) * kStepK + kh;      // beyond K: zeros
      a[u] = frag4<A_K, VEC>(A, d.a_sm, d.a_sk, row, d.M, kb, d.K);
      b[u] = frag4<B_K, VEC>(B, d.b_sn, d.b_sk, col, d.N, kb, d.K);
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][j], b[u][j], acc, 0, 0, 0);
  }
  // D[row][col]: lane holds col = lane % 32, rows 8 * (r / 4) + 4 * (lane / 32) + r % 4
  if (SPLIT) {
#pragma unroll
    for (int r = 0; r < 16; ++r) part[wave][(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * 33 + (lane & 31)] = acc[r];
    __syncthreads();
    for (int o = threadIdx.x; o < 1024; o += 64 * NW) {
      const int m = m0 + (o >> 5), n = n0 + (o & 31);
      float s = part[0][(o >> 5) * 33 + (o & 31)];
#pragma unroll
      for (int w = 1; w < NW; ++w) s += part[w][(o >> 5) * 33 + (o & 31)];
      if (m < d.M && n < d.N) epilogue1(d, m, n, s);
    }
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = m0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), n = n0 + (lane & 31);
      if (m < d.M && n < d.N) epilogue1(d, m, n, acc[r]);
    }
  }
}

template <bool A_K, bool B_K, bool VEC, int NW, bool SPLIT>
__global__ __launch_bounds__(64 * NW) void gemm_f32_kernel(GemmDesc d) {
  __shared__ float part[SPLIT ? NW : 1][32 * 33];
  gemm_f32_block<A_K, B_K, VEC, NW, SPLIT>(d, blockIdx.x, part);
}

constexpr long kSplitTiles = 1024;      // up to this many tiles a workgroup of eight wavefronts takes each

// The weight gradients of a layer and the ordered sums of its partial rows in one launch (g.first as in GemmGroup):
// with 32 tokens each of the five launches was 4 us of kernel for less than one step of work per wavefront.
__global__ __launch_bounds__(512) void gemm_f32_group_kernel(GemmGroup g) {
  __shared__ float part[8][32 * 33];
  static_assert(8 * 32 * 33 >= kReduceLdsFloats, "the reductions use the partial tiles' area");
  const int b = blockIdx.x, total = g.first[GemmGroup::MAX];
  if (b >= total) {
    colreduce_batch_block(g.tail, b - total, &part[0][0]);
    return;
  }
  int p = 0;
#pragma unroll
  for (int q = 1; q < GemmGroup::MAX; ++q)
    if (q < g.n && b >= g.first[q]) p = q;
  gemm_f32_block<false, false, false, 8, true>(g.d[p], b - g.first[p], part);
}

template <bool A_K, bool B_K, bool VEC>
static hipError_t launch(hipStream_t s, const GemmDesc& d) {
  const long tiles = (long)((d.M + 31) / 32) * ((d.N + 31) / 32);
  if (tiles <= kSplitTiles) {
    hipLaunchKernelGGL((gemm_f32_kernel<A_K, B_K, VEC, 8, true>), dim3((unsigned)tiles), dim3(512), 0, s, d);
  } else {
    hipLaunchKernelGGL((gemm_f32_kernel<A_K, B_K, VEC, 4, false>), dim3((unsigned)((tiles + 3) / 4)), dim3(256), 0, s, d);
  }
  return hipGetLastError();
}

// Where the vector-ALU kernel, whose 64 x 64 tiles reuse their operands in LDS, is the faster one for the forward and
// input-gradient forms: outputs that give every CU several of its tiles, fewer where the operands here come one float at a
// time.  Vector ALU / this kernel in us, forward / input gradient (rows, K, N; tiles of 64 x 64):
//   16-byte loads  4096 x 1024 x 1024 (1024)  215 / 152, 194 / 148     8192 x 1024 x 1024 (2048)  282 / 302, 277 / 305
//                  8192 x  512 x 2048 (4096)  279 / 298, 274 / 304     8192 x 1024 x 4096 (8192)  984 / 1108, 1050 / 1178
//                  4096 x  128 x 4096 (4096)   82 / 78,  79 / 88
//   4-byte loads   2048 x 1023 x 1025 (544)   211 / 174, 203 / 171     4096 x 1023 x 1025 (1088 / 1024)  218 / 305, 216 / 360
//                  4096 x  513 x 1025 (1088 / 576)  124 / 163, 220 / 260
// Weight gradients (both operands row-contiguous) are faster here at every size.
static bool vector_alu_is_faster(const GemmDesc& d, bool b_k, bool vec) {
  const long tiles = (long)((d.M + 63) / 64) * ((d.N + 63) / 64);
  if (vec) return tiles >= 2048 && (d.K >= 512 || (b_k && tiles >= 4096));
  return tiles >= (b_k ? 560 : 800);
}

// any M, N, K and the operand strides of the three forms a layer needs
hipError_t launch_gemm_f32(hipStream_t s, const GemmDesc& d) {
  if (d.M <= 0 || d.N <= 0) return hipSuccess;
  const bool a_k = d.a_sk == 1, b_k = d.b_sk == 1;
  if ((!a_k && d.a_sm != 1) || (!b_k && d.b_sn != 1)) return hipErrorNotSupported;
  const bool vec = d.K % 4 == 0 && (!a_k || (d.a_sm % 4 == 0 && ((uintptr_t)d.A & 15) == 0)) &&
                   (!b_k || (d.b_sn % 4 == 0 && ((uintptr_t)d.B & 15) == 0));
  if (a_k && vector_alu_is_faster(d, b_k, vec)) return hipErrorNotSupported;
  if (a_k && !b_k) return vec ? launch<true, false, true>(s, d) : launch<true, false, false>(s, d);
  if (a_k && b_k) return vec ? launch<true, true, true>(s, d) : launch<true, true, false>(s, d);
  if (!a_k && !b_k) return launch<false, false, false>(s, d);
  return launch<false, true, false>(s, d);
}

// n weight-gradient products (both operands with the contraction index strided) as one launch where each of them
// would be one workgroup per tile; hipErrorNotSupported otherwise (the caller launches them singly)
hipError_t launch_gemm_group_f32(hipStream_t s, const GemmDesc* d, int n, const GradReduceBatch* tail) {
  if (n < 1 || n > GemmGroup::MAX) return hipErrorNotSupported;
  GemmGroup g;
  memset(&g, 0, sizeof(g));
  g.n = n;
  if (tail != nullptr) g.tail = *tail;
  long total = 0;
  for (int i = 0; i < n; ++i) {
    if (d[i].M <= 0 || d[i].N <= 0 || d[i].a_sk == 1 || d[i].b_sk == 1 || d[i].a_sm != 1 || d[i].b_sn != 1)
      return hipErrorNotSupported;
    const long tiles = (long)((d[i].M + 31) / 32) * ((d[i].N + 31) / 32);
    if (tiles > kSplitTiles) return hipErrorNotSupported;
    g.d[i] = d[i];
    g.first[i] = (int)total;
    total += tiles;
  }
  for (int i = n; i <= GemmGroup::MAX; ++i) g.first[i] = (int)total;
  hipLaunchKernelGGL(gemm_f32_group_kernel, dim3((unsigned)(total + grad_reduce_blocks(g.tail))), dim3(512), 0, s, g);
  return hipGetLastError();
}

}  // namespace bamboo
