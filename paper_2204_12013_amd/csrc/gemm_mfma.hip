// bf16 GEMM on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16), fp32
// accumulation, fused epilogues.  One kernel template covers the three forms
// the layer needs:
//   forward          Y  = X W      A K-contiguous,  B N-contiguous
//   input gradient   dX = dY W^T   A K-contiguous,  B K-contiguous
//   weight gradient  dW += X^T dY  A M-contiguous,  B N-contiguous
//
// A workgroup of 4 wavefronts (2 x 2) owns a (64*WM) x (64*WN) output tile and
// walks K in slices of 64 that stream global -> LDS directly through a ring of
// buffers, under a hand-ordered, software-pipelined loop (see gemm_pl_tile).
// Row counts and the contraction length may be anything (the last slice's
// missing part is loaded as zeros by the buffer range check); only the
// contiguous dimension of every operand has to be a multiple of 8.  Operands whose contraction index is contiguous
// in memory are kept as [row][k] in LDS and read with ds_read_b128; operands
// whose contraction index is strided are kept in their memory order [k][row]
// and read with the transposing LDS load (ds_read_b64_tr_b16), which hands each
// lane four consecutive k of its row, so no operand is ever transposed in
// registers or re-laid-out in HBM.  The accumulators leave through a
// wavefront-private LDS staging area so that bias / residual / GELU inputs are
// read and results written with 16-byte row-contiguous accesses.
#include <math.h>
#include <stdlib.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include <string.h>

#include "common.h"
#include "reduce_device.h"

namespace bamboo {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short short4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// ---- GELU table -------------------------------------------------------------------------------
// The forward epilogue of the first FFN GEMM needs GELU(h) and GELU'(h) for 16.8 M values per call at
// the BERT-large stage; evaluated with exp and rcp that is ~28 vector instructions per value and as
// long as the GEMM's main loop.  Both results are stored as bf16, so it is enough to know
// Phi(h) = GELU(h) / h and GELU'(h) at the bf16 value nearest to h: a table over the bf16 values with
// 2^-11 <= |h| < 16 (15 exponents x 128 mantissas x 2 signs, fp32 pairs, 30 KB, kept in LDS) replaces
// the arithmetic by one LDS read.  Below 2^-11 Phi and GELU' are 0.5 to within 4e-4, above 16 they
// are 0 or 1 to fp32 precision, so clamping the index is exact enough at both ends.
constexpr int kGeluExpLo = 116, kGeluExpHi = 131;          // biased bf16 exponents covered
constexpr int kGeluN = (kGeluExpHi - kGeluExpLo) * 128;    // entries per sign
constexpr int kGeluBytes = 2 * kGeluN * 8;
__device__ float2 g_gelu_table[2 * kGeluN];

__global__ void gelu_table_init_kernel() {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= 2 * kGeluN) return;
  const unsigned bits = ((unsigned)(i / kGeluN) << 15) | (unsigned)((kGeluExpLo << 7) + i % kGeluN);
  const float h = __uint_as_float(bits << 16);
  const float phi = 0.5f * (1.0f + erff(h * 0.70710678118654752f));
  g_gelu_table[i] = make_float2(phi, phi + h * expf(-0.5f * h * h) * 0.39894228040143268f);
}

// Fills the table once per device and waits for the fill: done by prepare_gemm_tables at set-up
// (stage_init); a GEMM with a GELU epilogue that finds it missing (the kernel used on its own, without a
// stage) does it on its first launch, the one launcher call that waits for the device.  A failed fill
// is tried again by the next caller.
static hipError_t ensure_gelu_table(hipStream_t s) {
  static std::mutex lock;
  static bool ready[kMaxDevices];
  const int dev = current_device_index();
  std::lock_guard<std::mutex> hold(lock);
  if (ready[dev]) return hipSuccess;
  hipLaunchKernelGGL(gelu_table_init_kernel, dim3((2 * kGeluN + 255) / 256), dim3(256), 0, s);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e == hipSuccess) ready[dev] = true;
  return e;
}

// Set-up hook: fill the table now (and wait), so that no later launch has to.
hipError_t prepare_gemm_tables(hipStream_t s) { return ensure_gelu_table(s); }

// (GELU(h), GELU'(h)) from the table in LDS at byte address `tab`
__device__ __forceinline__ void gelu_pair_lookup(float h, unsigned tab, float* g, float* dg) {
  const bf16_t hb = (bf16_t)h;
  const unsigned b = __builtin_bit_cast(unsigned short, hb);
  int rel = (int)(b & 0x7fffu) - (kGeluExpLo << 7);
  rel = min(max(rel, 0), kGeluN - 1);
  const unsigned addr = tab + ((b & 0x8000u) ? kGeluN * 8 : 0) + rel * 8;
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  const f32x2 t = *(__attribute__((address_space(3))) const f32x2*)(uintptr_t)addr;
  *g = h * t[0];
  *dg = t[1];
}

// EPI_BIAS_GELU with the table taken to first order around its points, for row counts that are no multiple of 8: those
// ran on the vector-ALU kernel once, which evaluates both functions at the fp32 pre-activation, and lose nothing here
// (standard normal h, relative L2 error of the stored GELU / GELU': 1.667e-3 / 1.916e-3, the rounding to bf16, as with
// erf; 1.722e-3 / 1.996e-3 at the nearest point).  4095 x 1024 x 4096: 47.1 us, 42.4 at the nearest point, 82 with erf in the
// epilogue.  A form of its own, so that it costs the others nothing.
constexpr int EPI_BIAS_GELU_FINE = 7;
constexpr bool is_gelu(int epi) { return epi == EPI_BIAS_GELU || epi == EPI_BIAS_GELU_FINE; }

// With the point p nearest to h and e = h - p:
//   GELU(h) = h (Phi(p) + phi(p) e),  GELU'(h) = GELU'(p) + GELU''(p) e,  GELU'' = phi(p) (2 - p^2),
// and the density comes from the table as well: p phi(p) = GELU'(p) - Phi(p).  Second-order terms are below 2e-6 of the
// results (relative L2).  Beyond the table's last point phi is 0; e is held to 1 there so that GELU(inf) stays inf.
__device__ __forceinline__ void gelu_pair_fine(float h, unsigned tab, float* g, float* dg) {
  const unsigned b = __builtin_bit_cast(unsigned short, (bf16_t)h);
  int rel = (int)(b & 0x7fffu) - (kGeluExpLo << 7);
  rel = min(max(rel, 0), kGeluN - 1);
  const unsigned addr = tab + ((b & 0x8000u) ? kGeluN * 8 : 0) + rel * 8;
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  const f32x2 t = *(__attribute__((address_space(3))) const f32x2*)(uintptr_t)addr;
  const float p = __uint_as_float((unsigned)(rel + (kGeluExpLo << 7)) << 16 | (b & 0x8000u) << 16);
  const float e = h - p, density = (t[1] - t[0]) * __builtin_amdgcn_rcpf(p);
  *g = h * fmaf(density, fminf(fmaxf(e, -1.f), 1.f), t[0]);
  *dg = fmaf(density * fmaf(-p, p, 2.f), e, t[1]);
}

constexpr int BK = 64;          // k-slice
__host__ __device__ __forceinline__ int k_slices(int K) { return (K + BK - 1) / BK; }

// ---- direct global -> LDS copies (buffer_load_dwordx4 ... lds) --------------------
// The load writes 16 bytes per lane to consecutive LDS addresses starting at a
// wavefront-uniform base, so a slice cannot be padded per row.  Bank conflicts
// are avoided instead by choosing WHICH 16-byte chunk of global memory each
// lane fetches: chunks are XOR-swizzled inside their LDS row, and the fragment
// readers apply the same XOR.  Out-of-range output rows / columns are clamped to a valid one (they
// only feed outputs that are never stored).  What lies beyond K in the last slice has to be zero: those
// lanes' offsets are moved out of the buffer's range, for which the hardware delivers zeros
// (Loop::begin_slice), so K needs no padding and no kernel of its own.  A separate register-staged kernel
// used to take K that is not a multiple of 64, and shapes whose row count is not a multiple of 8 ran on the
// vector ALUs: a stage iteration with 999 tokens per micro-batch (H 1024, F 4096, 2 + 2 layers) took
// 34.3 ms against 2.87 ms now.
// The load is inline assembly so that the compiler's wait-count insertion does
// not see an LDS write that "may alias" every later LDS read and serialise the
// copy with the MFMAs; the kernel waits on vmcnt itself before the barrier
// that publishes a slice.  M0 carries the wavefront-uniform LDS base.

// ---- epilogue ---------------------------------------------------------------------------
// The accumulators leave through a wavefront-private LDS staging area, one 32-row block of the
// wave's sub-tile at a time; afterwards lane l owns, for pass `it`, the 8 consecutive outputs of
// chunk idx = l + 64 * it of the staged 32 x (32 * WN) block (row idx / CHUNKS, columns
// 8 * (idx % CHUNKS) ..); fp32 outputs in chunks of 4, so that an access is 16 bytes a lane and
// neighbouring lanes' accesses touch (see accumulate4).  What the epilogue has to read from memory for those outputs (residual,
// stored activation derivative, fp32 gradient to add to) is known long before the accumulators are
// final: EpiOperands::issue requests one row block's worth.  The kernel calls it for row block 0
// ahead of the last slices of the main loop, so the latency is covered by MFMAs, and write_tile
// requests row block i + 1 before it works on row block i.
template <int WM, int WN, int EPI>
struct EpiOperands {
  static constexpr int CHUNKS = 4 * WN, ITS = 32 * CHUNKS / 64;
  static constexpr bool BF = EPI == EPI_BIAS_RES || EPI == EPI_RES || EPI == EPI_MUL;
  static constexpr bool F32 = EPI == EPI_ACC_F32;
  static constexpr bool PRE = BF || F32;
  static constexpr bool HASB = EPI == EPI_BIAS || EPI == EPI_BIAS_RES || is_gelu(EPI);
  static constexpr int NLOADS = BF ? ITS : (F32 ? 2 * ITS : 0);   // load instructions per lane and row block
  bf16x8 b[BF ? ITS : 1];
  f32x4 f[F32 ? ITS : 1][2];
  // The bias of a lane's columns is the same for every row block: fetched once per tile, at its start
  // (a load inside the row-block loop would put its latency on every block).
  bf16x8 bias[HASB ? ITS : 1];
  __device__ __forceinline__ void issue_bias(const GemmDesc& d, int n0) {
    if (!HASB) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int wn = wave & 1;
#pragma unroll
    for (int it = 0; it < ITS; ++it) {
      const int n = min(n0 + wn * 32 * WN + ((lane + it * 64) % CHUNKS) * 8, d.N - 8);
      bias[it] = *(const bf16x8*)((const bf16_t*)d.bias + n);
    }
  }
  // Rows / columns past the edge are clamped to the last valid ones (their values are never used), so
  // that every lane issues exactly NLOADS loads: the main loop counts them in its vmcnt waits.
  __device__ __forceinline__ void issue(const GemmDesc& d, int m0, int n0, int i) {
    if (!PRE) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const void* src = EPI == EPI_MUL ? d.aux_in : (F32 ? (const void*)d.C : d.res);
#pragma unroll
    for (int it = 0; it < ITS; ++it) {
      const int idx = lane + it * 64;
      const int m = min(m0 + wm * 32 * WM + i * 32 + idx / CHUNKS, d.M - 1);
      const int n = min(n0 + wn * 32 * WN + (idx % CHUNKS) * 8, d.N - 8);
      const long e = (long)m * d.N + n;
      if (BF) b[it] = *(const bf16x8*)((const bf16_t*)src + e);
      if (F32) {      // a gradient is met again a layer stack later: past the caches (see accumulate4)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int q = lane + (2 * it + h) * 64;
          const int mq = min(m0 + wm * 32 * WM + i * 32 + q / (2 * CHUNKS), d.M - 1);
          const int nq = min(n0 + wn * 32 * WN + (q % (2 * CHUNKS)) * 4, d.N - 4);
          f[it][h] = __builtin_nontemporal_load((const f32x4*)((const float*)src + (long)mq * d.N + nq));
        }
      }
    }
  }
};

// 4 consecutive fp32 outputs of one row, added to what was fetched ahead.  Read and written once per micro-batch,
// hundreds of MB of other accesses apart: kept out of the caches it leaves them to the operands (GPT-2 stage
// 65.1 -> 64.3 ms, both ends merged 17.65 -> 17.51).  With two such accesses 32 bytes apart a lane, as the bf16 forms'
// chunks of 8 would have it, each touched every other 16 bytes of twice as many cache lines.  A layer's four weight
// gradients in one launch, before -> after: 2048 tokens of 12288 x 49152 7590 -> 7195 us, 4096 of 1024 x 4096 107 -> 103,
// 2048 of the same 68 -> 63.5, 1024 of 1600 x 6400 99 -> 93.5, 128 of the same 52.5 -> 48.2; 4096 of 1600 x 6400 alone
// 274 -> 281 (in the whole stage, traced in turn, 274.7 -> 277.5).  With plain loads, stores or both: 1-12 % slower but for
// the 12288-wide layer.
__device__ __forceinline__ void accumulate4(const GemmDesc& d, int m, int n, const f32x4& acc, const f32x4& old) {
  f32x4 v;
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = old[j] + acc[j];
  __builtin_nontemporal_store(v, (f32x4*)((float*)d.C + (long)m * d.N + n));
}

// epilogue on 8 consecutive bf16 outputs of one row; `pb` is the operand fetched ahead
template <int EPI>
__device__ __forceinline__ void epilogue8(const GemmDesc& d, int m, int n, const float (&acc)[8], const bf16x8& pb,
                                          const bf16x8& pbias, unsigned gelu_tab, float* stored = nullptr) {
  const long i = (long)m * d.N + n;
  float v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = acc[j];
  if (EPI == EPI_BIAS || EPI == EPI_BIAS_RES || is_gelu(EPI)) {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] += (float)pbias[j];
  }
  if (EPI == EPI_BIAS_RES || EPI == EPI_RES) {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] += (float)pb[j];
  }
  bf16x8 o;
  if (EPI == EPI_MUL) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      o[j] = (bf16_t)(v[j] * (float)pb[j]);
      if (stored != nullptr) stored[j] = (float)o[j];
    }
  } else if (is_gelu(EPI)) {
    bf16x8 g;
#pragma unroll
    for (int j = 0; j < 8; ++j) {   // activation and its derivative, looked up at the nearest bf16 value
      float gv, dgv;
      if (EPI == EPI_BIAS_GELU_FINE) gelu_pair_fine(v[j], gelu_tab, &gv, &dgv);
      else gelu_pair_lookup(v[j], gelu_tab, &gv, &dgv);
      g[j] = (bf16_t)gv;
      o[j] = (bf16_t)dgv;
    }
    *(bf16x8*)((bf16_t*)d.aux_out + i) = g;
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) o[j] = (bf16_t)v[j];
  }
  // Streaming stores where the next reader takes the output once (a LayerNorm, the elementwise part of a later
  // epilogue, the backward pass): what stays dirty in the eight L2s has to be written back before the next kernel
  // starts.  4096 x 4096 outputs, K = 1024: 37.8 -> 35.2 us per launch, all of it in the gap to the next one.
  // Outputs that the next kernel reads as a matrix operand, many times over (Q|K|V, GELU(h), the gradient at h),
  // stay cacheable: streaming those too gains nothing at the BERT-large-shaped iteration (22.25 against 22.30 ms,
  // 22.52 with no streaming) and costs 1.6 % at the GPT-2-shaped one (49.92 against 49.12 ms, 49.34 with none).
  if (EPI == EPI_BIAS || EPI == EPI_MUL) *(bf16x8*)((bf16_t*)d.C + i) = o;
  else __builtin_nontemporal_store(o, (bf16x8*)((bf16_t*)d.C + i));
}

// Accumulators -> wavefront-private LDS rows -> 16-byte global accesses.  `first` holds the operands
// of row block 0 (requested by the caller).
template <int WM, int WN, int EPI, int EPI_LD>
__device__ __forceinline__ void write_tile(const GemmDesc& d, f32x16 (&acc)[WM][WN], float* stage_all, int m0, int n0,
                                           const EpiOperands<WM, WN, EPI>& first, unsigned gelu_tab) {
  typedef EpiOperands<WM, WN, EPI> Ops;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int wm = wave >> 1, wn = wave & 1;
  float* stage = stage_all + wave * 32 * EPI_LD;
  Ops ops[2];
  ops[0] = first;
  // Column sums of the stored outputs (EPI_MUL with d.tile_colsum): where 64 is a multiple of the chunks per
  // staged row, a lane meets the same 8 columns in every pass, so it keeps 8 running sums over its rows.
  constexpr bool CAN_SUM = EPI == EPI_MUL && 64 % Ops::CHUNKS == 0;
  const bool sum_cols = CAN_SUM && d.tile_colsum != nullptr;
  float cs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < WM; ++i) {
    if (i + 1 < WM) ops[(i + 1) & 1].issue(d, m0, n0, i + 1);
    const Ops& cur = ops[i & 1];
    // D[row][col]: lane holds col = lane%32, rows 8*(r/4) + 4*(lane/32) + r%4
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        stage[(8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * EPI_LD + j * 32 + (lane & 31)] = acc[i][j][r];
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): the wave's own LDS writes have landed
    __builtin_amdgcn_wave_barrier();
    constexpr int CHUNKS = Ops::CHUNKS;   // 8-float chunks per staged row
#pragma unroll
    for (int it = 0; it < (Ops::F32 ? 2 * Ops::ITS : 0); ++it) {
      const int idx = lane + it * 64;
      const int row = idx / (2 * CHUNKS), ch = idx % (2 * CHUNKS);
      const int m = m0 + wm * 32 * WM + i * 32 + row;
      const int n = n0 + wn * 32 * WN + ch * 4;
      const f32x4 v = *(const f32x4*)(stage + row * EPI_LD + ch * 4);
      if (m < d.M && n < d.N) accumulate4(d, m, n, v, cur.f[it >> 1][it & 1]);
    }
#pragma unroll
    for (int it = 0; it < (Ops::F32 ? 0 : Ops::ITS); ++it) {
      const int idx = lane + it * 64;
      const int row = idx / CHUNKS, ch = idx % CHUNKS;
      const int m = m0 + wm * 32 * WM + i * 32 + row;
      const int n = n0 + wn * 32 * WN + ch * 8;
      const f32x4 lo = *(const f32x4*)(stage + row * EPI_LD + ch * 8);
      const f32x4 hi = *(const f32x4*)(stage + row * EPI_LD + ch * 8 + 4);
      if (m < d.M && n < d.N) {
        const float v[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        if (CAN_SUM) {
          float st8[8];
          epilogue8<EPI>(d, m, n, v, cur.b[Ops::BF ? it : 0], first.bias[Ops::HASB ? it : 0], gelu_tab, st8);
#pragma unroll
          for (int j = 0; j < 8; ++j) cs[j] += st8[j];
        } else {
          epilogue8<EPI>(d, m, n, v, cur.b[Ops::BF ? it : 0], first.bias[Ops::HASB ? it : 0], gelu_tab);
        }
      }
    }
    __builtin_amdgcn_wave_barrier();      // reads done before the next row block overwrites the stage
  }
  if (CAN_SUM) {
    if (sum_cols) {     // uniform over the workgroup
      // lanes that share a chunk (same lane % CHUNKS), in a fixed order; then the two wavefronts that share
      // the columns (wm = 0, 1), again in a fixed order
#pragma unroll
      for (int o = Ops::CHUNKS; o < 64; o <<= 1)
#pragma unroll
        for (int j = 0; j < 8; ++j) cs[j] += __shfl_xor(cs[j], o, 64);
      float* xch = stage_all;               // [2 wn][CHUNKS][8]: the staging area is free now
      __syncthreads();
      if (wm == 1 && lane < Ops::CHUNKS)
#pragma unroll
        for (int j = 0; j < 8; ++j) xch[(wn * Ops::CHUNKS + lane) * 8 + j] = cs[j];
      __syncthreads();
      if (wm == 0 && lane < Ops::CHUNKS) {
        const int n = n0 + wn * 32 * WN + lane * 8;
        if (n < d.N) {
          float* dst = d.tile_colsum + (long)(m0 / (64 * WM)) * d.N + n;
#pragma unroll
          for (int j = 0; j < 8; ++j) dst[j] = cs[j] + xch[(wn * Ops::CHUNKS + lane) * 8 + j];
        }
      }
    }
  }
}

// Tile order: consecutive workgroup ids are spread round-robin over the 8 XCDs,
// each with its own L2.  Give every XCD a contiguous range of tiles (xcd_range), and inside
// the range walk down GROUP rows of tiles before moving to the next column (tile_walk), so
// that the tiles an XCD works on at one time share operand slices in its L2.
__device__ __forceinline__ int xcd_range(int pid, int total) {
  const int per = total / 8;
  return pid < per * 8 ? (pid % 8) * per + pid / 8 : pid;
}
__device__ __forceinline__ void tile_walk(int pid, int tiles_m, int tiles_n, int* tm, int* tn) {
  constexpr int GROUP = 8;
  const int width = GROUP * tiles_n;
  const int group = pid / width;
  const int first_m = group * GROUP;
  const int rows = min(tiles_m - first_m, GROUP);
  *tm = first_m + (pid % width) % rows;
  *tn = (pid % width) / rows;
}

// ---- software-pipelined kernel with direct global -> LDS loads ------
// Per-thread address tables are set up once; inside the K loop a slice costs
// one scalar pointer bump per operand.  The instruction order of the loop body
// is fixed by hand (scheduling barriers between the groups):
//   k-step s of a slice issues its MFMAs interleaved with the LDS reads of the
//   fragments of k-step s+1 (two fragment register sets), so no MFMA waits on LDS;
//   all LDS reads of a slice are complete after k-step 2, where the one
//   workgroup barrier of the slice sits; k-step 3 then runs its MFMAs
//   interleaved with the fragment reads of the next slice (other buffer) and
//   with the global -> LDS loads of the slice after that (into the buffer just
//   vacated), which therefore have a whole slice of MFMA time to land.
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef __attribute__((address_space(3))) const bf16x8* lds_bf16x8_ptr;
typedef __attribute__((address_space(3))) short4_t* lds_short4_ptr;

typedef __attribute__((ext_vector_type(4))) unsigned buf_rsrc;   // 128-bit buffer descriptor, wavefront-uniform
constexpr unsigned kBufRange = 0x80000000u;                       // bytes addressable from a descriptor's base
constexpr unsigned kBufOutside = 0x80000000u;                     // an offset beyond them: the load delivers zeros
// Whether the offsets of a bm x bn output tile stay inside that range.  They count from the tile's first row: rows
// are a leading dimension apart where the contraction index is contiguous (256 of them reach 2 GiB at 4.2 M elements a
// row), otherwise the 64 steps of a slice are.  A tile that reaches beyond would be given zeros for its last rows, so it
// is not offered for such operands; smaller ones are, and at last the vector-ALU kernel.
static bool tile_in_reach(const GemmDesc& d, int bm, int bn) {
  auto reach = [&](bool k_contiguous, long ld, int rows, int tile) {
    const long steps = k_contiguous ? std::min(rows, tile) : std::min(d.K, BK);
    return (steps - 1) * ld * 2 + (k_contiguous ? BK : tile) * 2;
  };
  const bool a_k = d.a_sk == 1, b_k = d.b_sk == 1;
  return reach(a_k, a_k ? d.a_sm : d.a_sk, d.M, bm) <= (long)kBufRange &&
         reach(b_k, b_k ? d.b_sn : d.b_sk, d.N, bn) <= (long)kBufRange;
}

__device__ __forceinline__ buf_rsrc make_rsrc(const void* base) {
  const unsigned long b = (unsigned long)base;
  buf_rsrc r = {(unsigned)b, (unsigned)(b >> 32) & 0xffffu, kBufRange, 0x00020000u};
  return r;
}
__device__ __forceinline__ void bump_rsrc(buf_rsrc& r, long bytes) {
  const unsigned long b = (((unsigned long)r[1] << 32) | r[0]) + bytes;
  r[0] = (unsigned)b;
  r[1] = (unsigned)(b >> 32);
}
__device__ __forceinline__ void bload_lds16(unsigned voff, const buf_rsrc& r, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
               :
               : "v"(voff), "s"(r), "s"(lds_addr)
               : "memory", "m0");
}
__device__ __forceinline__ void gload_lds16(unsigned voff, const void* sbase, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(voff), "s"(sbase), "s"(lds_addr)
               : "memory", "m0");
}

// K-contiguous operand, ROWS x 64 per slice; LDS row r = 128 bytes, 16-byte chunk c at position
// c ^ ((r / 2) % 8).  The LDS has 64 four-byte banks and serves a 16-byte read for 16 lanes per
// cycle: 16 consecutive rows then cover every bank exactly once (rows 2j and 2j+1 share a position
// in the two 128-byte halves of the 256-byte bank line).
template <int ROWS>
struct PlK {
  static constexpr int NLOAD = ROWS / 32;
  static constexpr int BYTES = ROWS * BK * 2;
  // byte offsets of this thread's chunks relative to row row0, k 0 of the slice
  __device__ static __forceinline__ void load_offsets(unsigned (&off)[NLOAD], long ld, int row0, int row_lim) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const int r = i * 32 + (tid >> 3), p = tid & 7;
      const int row = min(row0 + r, row_lim - 1) - row0;
      off[i] = (unsigned)((long)row * ld * 2 + ((p ^ ((r >> 1) & 7)) << 4));
    }
  }
  // half h of a 256-row operand as ROWS = 128 rows: of every 128 rows the first (h = 0) or second 64
  __device__ static __forceinline__ void load_offsets_half(unsigned (&off)[NLOAD], long ld, int row0, int row_lim, int h) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const int r = i * 32 + (tid >> 3), p = tid & 7;
      const int row = min(row0 + (r >> 6) * 128 + h * 64 + (r & 63), row_lim - 1) - row0;
      off[i] = (unsigned)((long)row * ld * 2 + ((p ^ ((r >> 1) & 7)) << 4));
    }
  }
  __device__ static __forceinline__ const char* base(const bf16_t* g, long ld, int row0) {
    return (const char*)(g + (long)row0 * ld);
  }
  __device__ static __forceinline__ long slice_bytes(long ld) { return BK * 2; }
  // drop the chunks at or beyond the rem-th k of the slice (rem a multiple of 8, or <= 0)
  __device__ static __forceinline__ void mask_tail(unsigned (&off)[NLOAD], int rem) {
    const int k = (((int)threadIdx.x & 7) ^ (((int)threadIdx.x >> 4) & 7)) * 8;   // the same for all i: 32 rows = 16 pairs
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) off[i] = k < rem ? off[i] : kBufOutside;
  }
  // fragment address table: entry ks = address (within the operand's LDS area) of block 0 for k-step ks
  __device__ static __forceinline__ void frag_table(unsigned (&t)[4], int wave_row0) {
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
      t[ks] = (unsigned)((wave_row0 + (l & 31)) * (BK * 2) + (((2 * ks + (l >> 5)) ^ ((l >> 1) & 7)) << 4));
  }
  __device__ static __forceinline__ bf16x8 frag(const unsigned (&t)[4], unsigned lds_base, int blk, int ks) {
    return *(lds_bf16x8_ptr)(lds_base + t[ks] + blk * 32 * BK * 2);
  }
};
// Row-contiguous operand, 64 k-rows x ROWS per slice; the 16-byte chunk g of k-row k sits at chunk position
// place(g, k) of that row.  A transposing 8-byte read is served for 32 lanes per cycle, which address 4
// consecutive k-rows x 64 bytes: the placement moves those four 64-byte pieces to distinct quarters of the
// 256-byte bank line.  Rows of 128 or 256 bytes and more: XOR with a k-dependent chunk offset.  Rows of 384
// bytes (ROWS = 192) already alternate between the two halves of the bank line from one k-row to the
// next; rotating every second pair of k-rows by 64 bytes (modulo the row) separates the rest.
template <int ROWS>
struct PlMN {
  static constexpr int NLOAD = ROWS / 32;
  static constexpr int BYTES = ROWS * BK * 2;
  static constexpr int CPR = ROWS / 8;
  static constexpr bool ROTATE = (CPR & (CPR - 1)) != 0;
  static_assert(!ROTATE || ROWS == 192, "placement derived for rows of 384 bytes only");
  __device__ static __forceinline__ int swz(int k) {
    return ROTATE ? 4 * ((k >> 1) & 1) : (ROWS >= 128 ? 4 * (k & 3) : 4 * ((k >> 1) & 1));
  }
  // position of chunk g in k-row k, and the chunk found at position p
  __device__ static __forceinline__ int place(int g, int k) {
    if (!ROTATE) return g ^ swz(k);
    const int p = g + swz(k);
    return p >= CPR ? p - CPR : p;
  }
  __device__ static __forceinline__ int chunk_at(int p, int k) {
    if (!ROTATE) return p ^ swz(k);
    const int g = p - swz(k);
    return g < 0 ? g + CPR : g;
  }
  __device__ static __forceinline__ void load_offsets(unsigned (&off)[NLOAD], long ld, int row0, int row_lim) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const int c = i * 256 + tid;
      const int kr = c / CPR, p = c % CPR;
      const int col = min(row0 + (chunk_at(p, kr) << 3), row_lim - 8) - row0;
      off[i] = (unsigned)((long)kr * ld * 2 + col * 2);
    }
  }
  __device__ static __forceinline__ void load_offsets_half(unsigned (&off)[NLOAD], long ld, int row0, int row_lim, int h) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const int c = i * 256 + tid;
      const int kr = c / CPR, r = chunk_at(c % CPR, kr) << 3;
      const int col = min(row0 + (r >> 6) * 128 + h * 64 + (r & 63), row_lim - 8) - row0;
      off[i] = (unsigned)((long)kr * ld * 2 + col * 2);
    }
  }
  __device__ static __forceinline__ const char* base(const bf16_t* g, long ld, int row0) {
    return (const char*)(g + row0);
  }
  __device__ static __forceinline__ long slice_bytes(long ld) { return BK * ld * 2; }
  __device__ static __forceinline__ void mask_tail(unsigned (&off)[NLOAD], int rem) {
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) off[i] = (i * 256 + (int)threadIdx.x) / CPR < rem ? off[i] : kBufOutside;
  }
  // entry blk = address of k-step 0 for 32-row block blk
  __device__ static __forceinline__ void frag_table(unsigned (&t)[4], int wave_row0) {
    const int l = threadIdx.x & 63, i = l & 15;
    const int k = (l >> 5) * 8 + (i >> 2);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int col = wave_row0 + b * 32 + ((l >> 4) & 1) * 16 + (i & 3) * 4;
      t[b] = (unsigned)(k * ROWS * 2 + (place(col >> 3, k) << 4) + (col & 7) * 2);
    }
  }
  __device__ static __forceinline__ bf16x8 frag(const unsigned (&t)[4], unsigned lds_base, int blk, int ks) {
    const unsigned a = lds_base + t[blk] + ks * 16 * ROWS * 2;
    union { short4_t s4[2]; bf16x8 b; } u;
    u.s4[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(a));
    u.s4[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(a + 4 * ROWS * 2));
    return u.b;
  }
};

template <int WM, int WN, int NS, bool GELU = false>
struct SmemPl {
  static constexpr int BM = 64 * WM, BN = 64 * WN;
  static constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int EPI_LD = 32 * WN + 4;
  static constexpr int EPI_BYTES = 4 * 32 * EPI_LD * 4;
  static constexpr int MAIN_BYTES = NS * STAGE_BYTES;
  static constexpr int TABLE_OFF = (MAIN_BYTES > EPI_BYTES ? MAIN_BYTES : EPI_BYTES);   // GELU table behind the rest
  static constexpr int BYTES = TABLE_OFF + (GELU ? kGeluBytes : 0);
};

#define BAMBOO_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

template <int WM, int WN, bool A_K, bool B_K>
struct PlLoop {
  typedef SmemPl<WM, WN, 2> SM;
  typedef typename std::conditional<A_K, PlK<SM::BM>, PlMN<SM::BM>>::type OpA;
  typedef typename std::conditional<B_K, PlK<SM::BN>, PlMN<SM::BN>>::type OpB;
  static constexpr int NLA = OpA::NLOAD, NLB = OpB::NLOAD, NL = NLA + NLB;

  unsigned offA[NLA], offB[NLB];      // per-thread global byte offsets
  unsigned tabA[4], tabB[4];          // per-thread LDS fragment addresses
  buf_rsrc rA, rB;                    // descriptors based at the next slice to load
  long stepA, stepB;
  int rem;                            // contraction length left from that slice on
  unsigned lds0;                      // LDS address of stage 0
  unsigned wave_lds;                  // wave * 1024: where this wave's lanes of a 256-chunk group land

  __device__ __forceinline__ void issue_one(int n, unsigned stage) const {
    // n-th load of a slice: A chunks first, then B chunks
    if (n < NLA) bload_lds16(offA[n], rA, lds0 + stage + n * 4096 + wave_lds);
    else bload_lds16(offB[n - NLA], rB, lds0 + stage + SM::A_BYTES + (n - NLA) * 4096 + wave_lds);
  }
  // before the first load of a slice: its part beyond K is dropped (uniform branch, taken by the last slice only)
  __device__ __forceinline__ void begin_slice() {
    if (rem < BK) {
      OpA::mask_tail(offA, rem);
      OpB::mask_tail(offB, rem);
    }
    rem -= BK;
  }
  __device__ __forceinline__ void end_slice() {
    bump_rsrc(rA, stepA);
    bump_rsrc(rB, stepB);
  }
  __device__ __forceinline__ void issue_slice(unsigned stage) {
    begin_slice();
#pragma unroll
    for (int n = 0; n < NL; ++n) issue_one(n, stage);
    end_slice();
  }
  __device__ __forceinline__ void read_one(int n, unsigned stage, int ks, bf16x8 (&fa)[WM], bf16x8 (&fb)[WN]) const {
    if (n < WM) fa[n] = OpA::frag(tabA, lds0 + stage, n, ks);
    else fb[n - WM] = OpB::frag(tabB, lds0 + stage + SM::A_BYTES, n - WM, ks);
  }
  // One k-step: MFMAs on (ca, cb); if READ, the fragments (na, nb) of k-step ks_next of the slice
  // in `rstage` are fetched meanwhile, all of them behind the first MFMAs so that they have the
  // rest of this k-step and all of the next one to return; LOADPART 1 / 2 issues the first / second
  // half of the global loads of a slice into `lstage`, spread over the MFMAs.
  template <bool READ, int LOADPART>
  __device__ __forceinline__ void kstep(f32x16 (&acc)[WM][WN], const bf16x8 (&ca)[WM], const bf16x8 (&cb)[WN],
                                        bf16x8 (&na)[WM], bf16x8 (&nb)[WN], unsigned rstage, int ks_next,
                                        unsigned lstage) {
    constexpr int NMFMA = WM * WN, NR = WM + WN;
    constexpr int RSPAN = NMFMA >= 4 ? NMFMA / 2 : 1;           // MFMAs that carry the reads
    constexpr int RPM = (NR + RSPAN - 1) / RSPAN;               // reads per MFMA
    constexpr int NLH = (NL + 1) / 2;                           // loads per half
    constexpr int LPM = (NLH + NMFMA - 1) / NMFMA;              // loads per MFMA
    constexpr int L0 = LOADPART == 2 ? NLH : 0, L1 = LOADPART == 1 ? NLH : NL;
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        const int n = i * WN + j;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ca[i], cb[j], acc[i][j], 0, 0, 0);
        if (READ) {
#pragma unroll
          for (int q = 0; q < RPM; ++q)
            if (n < RSPAN && n * RPM + q < NR) read_one(n * RPM + q, rstage, ks_next, na, nb);
        }
        if (LOADPART != 0) {
#pragma unroll
          for (int q = 0; q < LPM; ++q)
            if (L0 + n * LPM + q < L1) issue_one(L0 + n * LPM + q, lstage);
        }
        BAMBOO_SCHED_FENCE();
      }
    if (LOADPART == 2) end_slice();
  }
};

// vmcnt(n) lgkmcnt(0): at most n of this wave's global loads still in flight, every LDS read returned
// (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4 left at its maximum, lgkmcnt 11:8)
template <int N>
__device__ __forceinline__ void wait_loads_and_lds() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
}

// Slices are kept in NS LDS buffers used round-robin; the global -> LDS loads of slice kt + NS - 1 ... are
// in flight while slice kt feeds the MFMAs, i.e. a load has NS - 1 slices of MFMA time to land.
// The tile whose first row and column are m0 and n0.
template <int WM, int WN, bool A_K, bool B_K, int EPI, int NS>
__device__ __forceinline__ void gemm_pl_tile(const GemmDesc& d, int m0, int n0) {
  typedef SmemPl<WM, WN, NS, is_gelu(EPI)> SM;
  typedef PlLoop<WM, WN, A_K, B_K> Loop;
  constexpr int NL = Loop::NL;
  constexpr unsigned STAGE = SM::STAGE_BYTES, RING = NS * STAGE;
  static_assert((NS - 1) * NL + (WM * WN <= 8 ? EpiOperands<WM, WN, EPI>::NLOADS : 0) < 64,
                "too many loads in flight for the vmcnt counter");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const long lda = A_K ? d.a_sm : d.a_sk;
  const long ldb = B_K ? d.b_sn : d.b_sk;

  Loop L;
  Loop::OpA::load_offsets(L.offA, lda, m0, d.M);
  Loop::OpB::load_offsets(L.offB, ldb, n0, d.N);
  Loop::OpA::frag_table(L.tabA, wm * 32 * WM);
  Loop::OpB::frag_table(L.tabB, wn * 32 * WN);
  L.rA = make_rsrc(Loop::OpA::base((const bf16_t*)d.A, lda, m0));
  L.rB = make_rsrc(Loop::OpB::base((const bf16_t*)d.B, ldb, n0));
  L.rem = d.K;
  L.stepA = Loop::OpA::slice_bytes(lda);
  L.stepB = Loop::OpB::slice_bytes(ldb);
  L.lds0 = (unsigned)(uintptr_t)(lds_void_ptr)smem_raw;
  L.wave_lds = wave * 1024;

  f32x16 acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk = max(k_slices(d.K), NS);   // the ring is filled once: slices wholly beyond K are zeros
  if (is_gelu(EPI)) {
    // GELU table -> its own LDS region, by the same direct loads as the slices and ahead of them: the
    // wait for slice 0 below covers these older loads too.  A wavefront copies 1 KB per load.
#pragma unroll
    for (int it = 0; it < (kGeluBytes / 16 + 255) / 256; ++it) {
      const int c0 = it * 256 + wave * 64;            // first chunk of this wavefront, uniform
      if (c0 < kGeluBytes / 16)
        gload_lds16((unsigned)(((threadIdx.x & 63)) << 4), (const char*)g_gelu_table + (long)c0 * 16,
                    L.lds0 + SM::TABLE_OFF + c0 * 16);
    }
  }
  // The bias is requested before any slice load: the waits below count the loads that are YOUNGER than
  // the slice they wait for, so however many bias loads the compiler keeps (the columns of a lane often
  // repeat) and wherever it puts them before this point, they can never stand in for a slice load there.
  EpiOperands<WM, WN, EPI> ops;
  ops.issue_bias(d, n0);
  BAMBOO_SCHED_FENCE();
  // four fragment register sets: k-step s of a slice computes from set s while set (s + 2) % 4 is
  // filled for the k-step after the next one, so an LDS read has more than a whole k-step to return
  bf16x8 fa[4][WM], fb[4][WN];
#pragma unroll
  for (int j = 0; j < NS; ++j) L.issue_slice(j * STAGE);
  wait_loads_and_lds<(NS - 1) * NL>();     // slice 0 has landed
  __syncthreads();
#pragma unroll
  for (int n = 0; n < WM + WN; ++n) L.read_one(n, 0, 0, fa[0], fb[0]);
#pragma unroll
  for (int n = 0; n < WM + WN; ++n) L.read_one(n, 0, 1, fa[1], fb[1]);

  // Steady state: slice kt computes from buffer cur.  During its first two k-steps the fragments of
  // its last two are read, so after them every LDS read of cur has been issued; once they have
  // returned and slice kt+1 has landed for every wave, the barrier frees cur for the loads of slice
  // kt+NS (issued between the MFMAs of the last two k-steps) and opens buffer nxt for reading.
  unsigned cur = 0;
  for (int kt = 0; kt < nk - NS; ++kt) {
    const unsigned nxt = cur + STAGE == RING ? 0 : cur + STAGE;
    L.template kstep<true, 0>(acc, fa[0], fb[0], fa[2], fb[2], cur, 2, 0);
    L.template kstep<true, 0>(acc, fa[1], fb[1], fa[3], fb[3], cur, 3, 0);
    wait_loads_and_lds<(NS - 2) * NL>();
    __syncthreads();
    L.begin_slice();
    BAMBOO_SCHED_FENCE();
    L.template kstep<true, 1>(acc, fa[2], fb[2], fa[0], fb[0], nxt, 0, cur);
    L.template kstep<true, 2>(acc, fa[3], fb[3], fa[1], fb[1], nxt, 1, cur);
    cur = nxt;
  }
  // The last NS slices issue no slice loads; instead the epilogue's operands for the first row block
  // are requested now, so that they arrive under the remaining MFMAs.  They are younger than every
  // slice load, hence simply add to the number of loads that may still be in flight at the waits below.
  // (256 x 256 tiles have no registers to spare for them until the fragments are dead.)
  constexpr bool EARLY = WM * WN <= 8;
  if (EARLY) ops.issue(d, m0, n0, 0);
  constexpr int NEPI = EARLY ? EpiOperands<WM, WN, EPI>::NLOADS : 0;
  // the waits below assume these NEPI loads are in flight from here on: keep the compiler from moving them
  asm volatile("" ::: "memory");
  BAMBOO_SCHED_FENCE();
  // slice nk-1-J still has J slices after it, J-1 of which may be in flight
  auto tail = [&](auto jc) __attribute__((always_inline)) {
    constexpr int J = decltype(jc)::value;
    const unsigned nxt = cur + STAGE == RING ? 0 : cur + STAGE;
    L.template kstep<true, 0>(acc, fa[0], fb[0], fa[2], fb[2], cur, 2, 0);
    L.template kstep<true, 0>(acc, fa[1], fb[1], fa[3], fb[3], cur, 3, 0);
    if (J > 0) {
      wait_loads_and_lds<(J > 1 ? J - 1 : 0) * NL + NEPI>();
      __syncthreads();
      BAMBOO_SCHED_FENCE();
    }
    L.template kstep<(J > 0), 0>(acc, fa[2], fb[2], fa[0], fb[0], nxt, 0, 0);
    L.template kstep<(J > 0), 0>(acc, fa[3], fb[3], fa[1], fb[1], nxt, 1, 0);
    cur = nxt;
  };
  if constexpr (NS >= 4) tail(std::integral_constant<int, 3>());
  if constexpr (NS >= 3) tail(std::integral_constant<int, 2>());
  tail(std::integral_constant<int, 1>());
  tail(std::integral_constant<int, 0>());
  // every wave is done with the slice buffers before the staging area reuses them
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __syncthreads();
  BAMBOO_SCHED_FENCE();
  if (!EARLY) ops.issue(d, m0, n0, 0);
  write_tile<WM, WN, EPI, SM::EPI_LD>(d, acc, (float*)smem_raw, m0, n0, ops, L.lds0 + SM::TABLE_OFF);
}

// ---- 256 x 256 tile: quarter-tile phases ---------------------------------------------------------
// One 256 x 256 tile per CU reads the fewest LDS fragments and L1 bytes per matrix instruction, but two slices are
// all the LDS holds (128 of 160 KB).  With whole slices as the unit of reuse a buffer was refilled half a slice time
// before it was needed, less than a trip to memory: 2048 x 12288 x 49152 took 2450 us.  Here the unit is half an
// operand slice (128 rows x 64): a wavefront works through the four quarters of its 128 x 128 in phases of 16 matrix
// instructions,
//     phase   multiplies   reads for later      loads (slice + 2, + 3) into what the previous phase read last
//       1      A0 x B0      B1                   B0 (+2)
//       2      A0 x B1      A1                   B1 (+2)
//       3      A1 x B0      A0 of the next       A1 (+2)
//       4      A1 x B1      B0 of the next       A0 (+3)
// so every half is on its way for seven phases, 1.75 slice times, in the same LDS and with the same four fragment
// register sets.  One barrier per phase tells that the half read in the phase before is free everywhere and that the
// one to be read now has landed everywhere: 2120 us for the shape above, 97 -> 78 us for 64 tiles over K = 4096.
// The order of the sums is that of the other tiles.
// What bounds it now: the matrix cores at the clock the chip holds under them.  The loop is 89 % busy (2300 clocks per
// 2048 of matrix work; taking waits and barriers out of a copy changes nothing), but the clock falls to 1.3-1.6 GHz
// with 256 CUs on random data; without loads and LDS reads the same instructions reach 1.9 PFLOP/s, with them 1.47.
template <bool A_K, bool B_K>
struct PhLoop {
  typedef typename std::conditional<A_K, PlK<128>, PlMN<128>>::type OpA;
  typedef typename std::conditional<B_K, PlK<128>, PlMN<128>>::type OpB;
  static constexpr int QUARTER = 16384;               // bytes of one half-operand slice: 128 rows x 64
  static constexpr unsigned A0 = 0, A1 = QUARTER, B0 = 2 * QUARTER, B1 = 3 * QUARTER, STAGE = 4 * QUARTER;
  unsigned offA[2][4], offB[2][4];                    // per-thread byte offsets of the halves' loads
  unsigned tabA[4], tabB[4];                          // per-thread LDS fragment addresses inside a half
  buf_rsrc rA, rB;                                    // based at the next slice to load
  long stepA, stepB;
  int remA[2], remB[2];                               // contraction left from each half's next slice on
  unsigned lds0, wave_lds;

  template <int H>
  __device__ __forceinline__ void begin_a() {
    if (remA[H] < BK) OpA::mask_tail(offA[H], remA[H]);
    remA[H] -= BK;
  }
  template <int H>
  __device__ __forceinline__ void begin_b() {
    if (remB[H] < BK) OpB::mask_tail(offB[H], remB[H]);
    remB[H] -= BK;
  }
  template <int H> __device__ __forceinline__ void load_a(int n, unsigned stage) const {
    bload_lds16(offA[H][n], rA, lds0 + stage + (H ? A1 : A0) + n * 4096 + wave_lds);
  }
  template <int H> __device__ __forceinline__ void load_b(int n, unsigned stage) const {
    bload_lds16(offB[H][n], rB, lds0 + stage + (H ? B1 : B0) + n * 4096 + wave_lds);
  }
  template <int H> __device__ __forceinline__ void issue_a(unsigned stage) {
    begin_a<H>();
#pragma unroll
    for (int n = 0; n < 4; ++n) load_a<H>(n, stage);
  }
  template <int H> __device__ __forceinline__ void issue_b(unsigned stage) {
    begin_b<H>();
#pragma unroll
    for (int n = 0; n < 4; ++n) load_b<H>(n, stage);
  }
};

template <int N>
__device__ __forceinline__ void phase_barrier() {
  BAMBOO_SCHED_FENCE();
  wait_loads_and_lds<N>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  BAMBOO_SCHED_FENCE();
}

template <bool A_K, bool B_K, int EPI>
__device__ __forceinline__ void gemm_ph_tile(const GemmDesc& d, int m0, int n0) {
  typedef SmemPl<4, 4, 2, is_gelu(EPI)> SM;
  typedef PhLoop<A_K, B_K> Loop;
  static_assert(SM::MAIN_BYTES == 2 * Loop::STAGE, "");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const long lda = A_K ? d.a_sm : d.a_sk;
  const long ldb = B_K ? d.b_sn : d.b_sk;

  Loop L;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    Loop::OpA::load_offsets_half(L.offA[h], lda, m0, d.M, h);
    Loop::OpB::load_offsets_half(L.offB[h], ldb, n0, d.N, h);
    L.remA[h] = L.remB[h] = d.K;
  }
  Loop::OpA::frag_table(L.tabA, wm * 64);
  Loop::OpB::frag_table(L.tabB, wn * 64);
  L.rA = make_rsrc(Loop::OpA::base((const bf16_t*)d.A, lda, m0));
  L.rB = make_rsrc(Loop::OpB::base((const bf16_t*)d.B, ldb, n0));
  L.stepA = Loop::OpA::slice_bytes(lda);
  L.stepB = Loop::OpB::slice_bytes(ldb);
  L.lds0 = (unsigned)(uintptr_t)(lds_void_ptr)smem_raw;
  L.wave_lds = wave * 1024;

  f32x16 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  const int nk = k_slices(d.K);
  if (is_gelu(EPI)) {     // the table: requested ahead of the slices, covered by the first wait
#pragma unroll
    for (int it = 0; it < (kGeluBytes / 16 + 255) / 256; ++it) {
      const int c0 = it * 256 + wave * 64;
      if (c0 < kGeluBytes / 16)
        gload_lds16((unsigned)(((threadIdx.x & 63)) << 4), (const char*)g_gelu_table + (long)c0 * 16,
                    L.lds0 + SM::TABLE_OFF + c0 * 16);
    }
  }
  EpiOperands<4, 4, EPI> ops;
  ops.issue_bias(d, n0);
  BAMBOO_SCHED_FENCE();

  bf16x8 fa[2][4][2], fb[2][4][2];      // [half][k-step][32-row block]
  auto read_a = [&](auto hc, int n, unsigned stage) __attribute__((always_inline)) {
    constexpr int H = decltype(hc)::value;
    fa[H][n >> 1][n & 1] = Loop::OpA::frag(L.tabA, L.lds0 + stage + (H ? Loop::A1 : Loop::A0), n & 1, n >> 1);
  };
  auto read_b = [&](auto hc, int n, unsigned stage) __attribute__((always_inline)) {
    constexpr int H = decltype(hc)::value;
    fb[H][n >> 1][n & 1] = Loop::OpB::frag(L.tabB, L.lds0 + stage + (H ? Loop::B1 : Loop::B0), n & 1, n >> 1);
  };
  // 16 matrix instructions on the quarter (HA, HB); rd(n): n-th of the 8 fragment reads for a later phase, behind the
  // first instructions; ld(n): n-th of the 4 loads into the half whose last reader has passed
  auto quarter = [&](auto hac, auto hbc, auto rd, auto ld) __attribute__((always_inline)) {
    constexpr int HA = decltype(hac)::value, HB = decltype(hbc)::value;
#pragma unroll
    for (int n = 0; n < 16; ++n) {
      const int ks = n >> 2, i = (n >> 1) & 1, j = n & 1;
      acc[2 * HA + i][2 * HB + j] =
          __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[HA][ks][i], fb[HB][ks][j], acc[2 * HA + i][2 * HB + j], 0, 0, 0);
      if (n < 8) rd(n);
      else if (n < 12) ld(n - 8);
      BAMBOO_SCHED_FENCE();
    }
  };
  std::integral_constant<int, 0> c0;
  std::integral_constant<int, 1> c1;

  L.template issue_a<0>(0);
  L.template issue_b<0>(0);
  L.template issue_b<1>(0);
  L.template issue_a<1>(0);
  bump_rsrc(L.rA, L.stepA);
  bump_rsrc(L.rB, L.stepB);
  L.template issue_a<0>(Loop::STAGE);
  L.template issue_b<0>(Loop::STAGE);
  L.template issue_b<1>(Loop::STAGE);
  L.template issue_a<1>(Loop::STAGE);
  bump_rsrc(L.rA, L.stepA);
  bump_rsrc(L.rB, L.stepB);
  phase_barrier<24>();                  // A0, B0 of slice 0 have landed
#pragma unroll
  for (int n = 0; n < 8; ++n) read_a(c0, n, 0);
#pragma unroll
  for (int n = 0; n < 8; ++n) read_b(c0, n, 0);
  phase_barrier<63>();
  L.template issue_a<0>(0);             // slice 2

  unsigned cur = 0;
  for (int kt = 0; kt < nk; ++kt) {
    const unsigned nxt = cur ^ Loop::STAGE;
    phase_barrier<24>();
    L.template begin_b<0>();
    quarter(c0, c0, [&](int n) { read_b(c1, n, cur); }, [&](int n) { L.template load_b<0>(n, cur); });
    phase_barrier<24>();
    L.template begin_b<1>();
    quarter(c0, c1, [&](int n) { read_a(c1, n, cur); }, [&](int n) { L.template load_b<1>(n, cur); });
    bump_rsrc(L.rB, L.stepB);
    phase_barrier<24>();
    L.template begin_a<1>();
    quarter(c1, c0, [&](int n) { read_a(c0, n, nxt); }, [&](int n) { L.template load_a<1>(n, cur); });
    bump_rsrc(L.rA, L.stepA);
    phase_barrier<24>();
    L.template begin_a<0>();
    quarter(c1, c1, [&](int n) { read_b(c0, n, nxt); }, [&](int n) { L.template load_a<0>(n, nxt); });
    cur = nxt;
  }
  // what is still on its way into the ring are zeros beyond K; every wavefront is done with it
  phase_barrier<0>();
  ops.issue(d, m0, n0, 0);
  write_tile<4, 4, EPI, SM::EPI_LD>(d, acc, (float*)smem_raw, m0, n0, ops, L.lds0 + SM::TABLE_OFF);
}

template <int WM, int WN, bool A_K, bool B_K, int EPI, int NS, int MINB>
__global__ __launch_bounds__(256, MINB) void gemm_mfma_pl_kernel(GemmDesc d) {
  constexpr int BM = 64 * WM, BN = 64 * WN;
  const int pid = xcd_range(blockIdx.x, ((d.M + BM - 1) / BM) * ((d.N + BN - 1) / BN));
  int tile_m, tile_n;
  tile_walk(pid, (d.M + BM - 1) / BM, (d.N + BN - 1) / BN, &tile_m, &tile_n);
  if constexpr (WM == 4 && WN == 4) gemm_ph_tile<A_K, B_K, EPI>(d, tile_m * BM, tile_n * BN);
  else gemm_pl_tile<WM, WN, A_K, B_K, EPI, NS>(d, tile_m * BM, tile_n * BN);
}

// Several weight-gradient problems in one launch: workgroup b works on problem p where
// first[p] <= b < first[p+1].  The problems of a layer's backward are independent of each other and
// most of them do not fill a whole number of rounds of the 256 CUs on their own (1024 x 1024 outputs
// are 64 tiles of 128 x 128); launched together their tiles pack, and a CU goes from one problem's
// tile to the next one's without the chip draining in between.
// With 256 x 256 tiles a remainder of up to 128 rows or columns at a matrix' edge is covered by 128 x 256 or 256 x 128
// tiles (see edge_strips): a launch of 1600-wide matrices has 456 tiles and 76 strips instead of 532 tiles, i.e. two
// rounds of the 256 CUs instead of three.  4096 tokens, 1600 x 6400 layers: 293 us as 128 x 256 tiles, 286 us like this,
// 266 us with the gradients past the caches (see accumulate4): 133 us a round, 90 us of them main loop at the clock that
// 256 busy CUs leave, the rest fp32 reads and writes.
template <int WM, int WN, int NS, int MINB>
__global__ __launch_bounds__(256, MINB) void gemm_mfma_pl_group_kernel(GemmGroup g) {
  const int total = g.first[GemmGroup::MAX], wg = (int)blockIdx.x - g.chains;
  if (wg >= total) {                               // behind the GEMM tiles: the reductions riding along
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    colreduce_batch_block(g.tail, wg - total, (float*)smem_raw);
    return;
  }
  if constexpr (WM == 4 && WN == 4) {
    if (wg < 0) {
      const int begin = (int)blockIdx.x * g.chain, end = min(begin + g.chain, g.strip0[GemmGroup::MAX]);
      for (int i = begin; i < end; ++i) {
        int p = 0;
#pragma unroll
        for (int q = 1; q < GemmGroup::MAX; ++q)
          if (q < g.n && i >= g.strip0[q]) p = q;
        const GemmDesc& d = g.d[p];
        const int along_n = g.tiles_m[p] * 256 < d.M ? (d.N + 255) / 256 : 0;   // strips of the last rows come first
        const int j = i - g.strip0[p];
        // the loads of a tile are counted from nothing in flight, and its LDS is free in every wavefront
        __builtin_amdgcn_s_waitcnt(0x0070);
        __syncthreads();
        if (j < along_n) gemm_pl_tile<2, 4, false, false, EPI_ACC_F32, 3>(d, g.tiles_m[p] * 256, j * 256);
        else gemm_pl_tile<4, 2, false, false, EPI_ACC_F32, 3>(d, (j - along_n) * 256, g.tiles_n[p] * 256);
      }
      return;
    }
  }
  // g.whole_launch_ranges: every XCD takes one contiguous range of the CONCATENATED tile sequences, so that
  // a problem's operands go to the L2s of the two or three XCDs its range spans instead of to all eight
  // (launches of one round); otherwise each problem is spread over all XCDs, a range per XCD inside it.
  const int b = g.whole_launch_ranges ? xcd_range(wg, total) : wg;
  int p = 0;
#pragma unroll
  for (int q = 1; q < GemmGroup::MAX; ++q)
    if (q < g.n && b >= g.first[q]) p = q;
  int local = b - g.first[p];
  if (!g.whole_launch_ranges) {
    int end = total;
#pragma unroll
    for (int q = GemmGroup::MAX - 1; q >= 1; --q)
      if (q > p && q < g.n) end = g.first[q];
    local = xcd_range(local, end - g.first[p]);
  }
  int tile_m, tile_n;
  tile_walk(local, g.tiles_m[p], g.tiles_n[p], &tile_m, &tile_n);
  if constexpr (WM == 4 && WN == 4) gemm_ph_tile<false, false, EPI_ACC_F32>(g.d[p], tile_m * 256, tile_n * 256);
  else gemm_pl_tile<WM, WN, false, false, EPI_ACC_F32, NS>(g.d[p], tile_m * 64 * WM, tile_n * 64 * WN);
}

template <int WM, int WN, bool A_K, bool B_K, int EPI, int NS>
static hipError_t launch_pl(hipStream_t s, const GemmDesc& d, int tiles) {
  typedef SmemPl<WM, WN, NS, is_gelu(EPI)> SM;
  constexpr auto kern = gemm_mfma_pl_kernel<WM, WN, A_K, B_K, EPI, NS, (2 * SM::BYTES <= 160 * 1024 ? 2 : 1)>;
  const hipError_t e = ensure_lds_attribute<kern, SM::BYTES>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(tiles), dim3(256), SM::BYTES, s, d);
  return hipGetLastError();
}

// ---- few output tiles, long contraction: the wavefronts of a workgroup split K ------------------
// A micro-batch of a few hundred tokens gives the products of a layer 30 to 250 tiles of 64 x 64 or less, so a launch
// is one round whose time is the serial walk through K (K = 4096: 64 slices at 0.4 us, a workgroup barrier and a
// load round trip each), while most matrix pipes idle.  Here every wavefront of a workgroup works on the SAME
// tile, 32 x 32 with eight wavefronts or 64 x 64 with four, and takes every NW-th slice through a ring of two
// buffers of its own, with no barrier before the end, so all their loads are in flight side by side; the partial
// tiles are summed through LDS in wavefront order (deterministic).  Bound by the vector L1 (64 bytes per clock:
// 4 us of a 128 x 1024 x 4096 launch) and the latency of the few round trips left.  See choose_split for figures.
template <int ROWS>
struct WvK {                       // K-contiguous operand: ROWS x 64, the placement of PlK, copied by one wavefront
  static constexpr int NLOAD = ROWS / 8;
  static constexpr int BYTES = ROWS * BK * 2;
  __device__ static __forceinline__ int chunk(int i) {
    const int l = threadIdx.x & 63;
    return (l & 7) ^ ((4 * i + (l >> 4)) & 7);
  }
  __device__ static __forceinline__ void load_offsets(unsigned (&off)[NLOAD], long ld, int row0, int row_lim) {
    const int l = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const int row = min(row0 + i * 8 + (l >> 3), row_lim - 1) - row0;
      off[i] = (unsigned)((long)row * ld * 2 + (chunk(i) << 4));
    }
  }
  __device__ static __forceinline__ void mask_tail(unsigned (&off)[NLOAD], int rem) {
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) off[i] = chunk(i) * 8 < rem ? off[i] : kBufOutside;
  }
  __device__ static __forceinline__ bf16x8 frag(unsigned lds_base, int blk, int ks) {
    const int l = threadIdx.x & 63;
    return *(lds_bf16x8_ptr)(lds_base + (blk * 32 + (l & 31)) * (BK * 2) + (((2 * ks + (l >> 5)) ^ ((l >> 1) & 7)) << 4));
  }
};
template <int ROWS>
struct WvMN {                      // row-contiguous operand: 64 k-rows x ROWS, the placement of PlMN
  static constexpr int NLOAD = ROWS / 8;
  static constexpr int BYTES = ROWS * BK * 2;
  static constexpr int CPR = ROWS / 8;
  static_assert(ROWS == 32 || ROWS == 64, "");
  // rows of 64 bytes: four consecutive k-rows fill the bank line by themselves; rows of 128: see PlMN
  __device__ static __forceinline__ int swz(int k) { return ROWS == 64 ? 4 * ((k >> 1) & 1) : 0; }
  __device__ static __forceinline__ int krow(int i) { return (i * 64 + ((int)threadIdx.x & 63)) / CPR; }
  __device__ static __forceinline__ void load_offsets(unsigned (&off)[NLOAD], long ld, int row0, int row_lim) {
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
      const int p = (threadIdx.x & 63) % CPR, kr = krow(i);
      const int col = min(row0 + ((p ^ swz(kr)) << 3), row_lim - 8) - row0;
      off[i] = (unsigned)((long)kr * ld * 2 + col * 2);
    }
  }
  __device__ static __forceinline__ void mask_tail(unsigned (&off)[NLOAD], int rem) {
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) off[i] = krow(i) < rem ? off[i] : kBufOutside;
  }
  __device__ static __forceinline__ bf16x8 frag(unsigned lds_base, int blk, int ks) {
    const int l = threadIdx.x & 63, i = l & 15;
    const int k = ks * 16 + (l >> 5) * 8 + (i >> 2), col = blk * 32 + ((l >> 4) & 1) * 16 + (i & 3) * 4;
    const unsigned a = lds_base + k * ROWS * 2 + (((col >> 3) ^ swz(k)) << 4) + (col & 7) * 2;
    union { short4_t s4[2]; bf16x8 b; } u;
    u.s4[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(a));
    u.s4[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(a + 4 * ROWS * 2));   // k + 4: the same swizzle
    return u.b;
  }
};

// operands the epilogue of one 8-output chunk reads from memory
template <int EPI>
struct ChunkOperands {
  bf16x8 bias, pre;
  __device__ __forceinline__ void fetch(const GemmDesc& d, int m, int n) {
    if (m >= d.M || n >= d.N) return;
    if (EPI == EPI_BIAS || EPI == EPI_BIAS_RES || is_gelu(EPI)) bias = *(const bf16x8*)((const bf16_t*)d.bias + n);
    if (EPI == EPI_BIAS_RES || EPI == EPI_RES) pre = *(const bf16x8*)((const bf16_t*)d.res + (long)m * d.N + n);
    if (EPI == EPI_MUL) pre = *(const bf16x8*)((const bf16_t*)d.aux_in + (long)m * d.N + n);
  }
};

template <int T32, int NW, bool B_K, int EPI>
struct SmemSplit {
  static constexpr int TILE = 32 * T32;
  static constexpr int STAGE = 2 * TILE * BK * 2;              // bytes of one slice of A and B
  static constexpr int LD = TILE + 4;                           // floats per row of a partial tile
  static constexpr int RING = NW * 2 * STAGE, PART = NW * TILE * LD * 4;
  static constexpr int TABLE_OFF = RING > PART ? RING : PART;
  static constexpr int BYTES = TABLE_OFF + (is_gelu(EPI) ? kGeluBytes : 0);
};

template <int T32, int NW, bool B_K, int EPI>
__global__ __launch_bounds__(64 * NW) void gemm_mfma_split_kernel(GemmDesc d) {
  typedef SmemSplit<T32, NW, B_K, EPI> SM;
  constexpr int TILE = SM::TILE, LD = SM::LD;
  typedef WvK<TILE> OpA;
  typedef typename std::conditional<B_K, WvK<TILE>, WvMN<TILE>>::type OpB;
  constexpr int NL = OpA::NLOAD + OpB::NLOAD;
  constexpr int CH = TILE / 8, CHUNKS = TILE * CH;              // 8-output chunks: per row, per tile
  constexpr int PER = (CHUNKS + 64 * NW - 1) / (64 * NW);       // per thread
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int tiles_m = (d.M + TILE - 1) / TILE, tiles_n = (d.N + TILE - 1) / TILE;
  int tm, tn;
  tile_walk(xcd_range(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, &tm, &tn);
  const int m0 = tm * TILE, n0 = tn * TILE;
  const unsigned lds0 = (unsigned)(uintptr_t)(lds_void_ptr)smem_raw;
  const unsigned ring = lds0 + wave * 2 * SM::STAGE;

  // everything the epilogue reads is requested first: older than the slice loads, hence covered by their waits
  ChunkOperands<EPI> ops[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int idx = threadIdx.x + q * 64 * NW;
    if (CHUNKS >= 64 * NW || idx < CHUNKS) ops[q].fetch(d, m0 + idx / CH, n0 + (idx % CH) * 8);
  }
  if (is_gelu(EPI)) {
    for (int c0 = wave * 64; c0 < kGeluBytes / 16; c0 += 64 * NW)
      gload_lds16((unsigned)(lane << 4), (const char*)g_gelu_table + (long)c0 * 16, lds0 + SM::TABLE_OFF + c0 * 16);
  }
  BAMBOO_SCHED_FENCE();

  unsigned offA[OpA::NLOAD], offB[OpB::NLOAD];
  OpA::load_offsets(offA, d.a_sm, m0, d.M);
  const long ldb = B_K ? d.b_sn : d.b_sk;
  OpB::load_offsets(offB, ldb, n0, d.N);
  const long stepA = BK * 2, stepB = B_K ? BK * 2 : BK * ldb * 2;
  buf_rsrc rA = make_rsrc((const char*)((const bf16_t*)d.A + (long)m0 * d.a_sm) + wave * stepA);
  buf_rsrc rB = make_rsrc((const char*)((const bf16_t*)d.B + (B_K ? (long)n0 * ldb : (long)n0)) + wave * stepB);
  int rem = d.K - wave * BK;                                    // contraction left from this wavefront's next slice on
  const int mine = rem <= 0 ? 0 : (rem + NW * BK - 1) / (NW * BK);
  auto issue = [&](unsigned stage) __attribute__((always_inline)) {
    if (rem < BK) {
      OpA::mask_tail(offA, rem);
      OpB::mask_tail(offB, rem);
    }
    rem -= NW * BK;
#pragma unroll
    for (int i = 0; i < OpA::NLOAD; ++i) bload_lds16(offA[i], rA, ring + stage + i * 1024);
#pragma unroll
    for (int i = 0; i < OpB::NLOAD; ++i) bload_lds16(offB[i], rB, ring + stage + OpA::BYTES + i * 1024);
    bump_rsrc(rA, NW * stepA);
    bump_rsrc(rB, NW * stepB);
  };
  f32x16 acc[T32][T32];
#pragma unroll
  for (int i = 0; i < T32; ++i)
#pragma unroll
    for (int j = 0; j < T32; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  if (mine > 0) issue(0);
  if (mine > 1) issue(SM::STAGE);
  for (int s = 0; s < mine; ++s) {
    const unsigned st = (s & 1) * SM::STAGE;
    if (s + 1 < mine) wait_loads_and_lds<NL>();                 // the slice after this one may be in flight
    else wait_loads_and_lds<0>();
    asm volatile("" ::: "memory");
    bf16x8 fa[4][T32], fb[4][T32];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
      for (int i = 0; i < T32; ++i) fa[ks][i] = OpA::frag(ring + st, i, ks);
#pragma unroll
      for (int j = 0; j < T32; ++j) fb[ks][j] = OpB::frag(ring + st + OpA::BYTES, j, ks);
    }
    if (s + 2 < mine) {
      __builtin_amdgcn_s_waitcnt(0xc07f);                       // the reads have returned: the buffer is free
      BAMBOO_SCHED_FENCE();
      issue(st);
    }
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < T32; ++i)
#pragma unroll
        for (int j = 0; j < T32; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][i], fb[ks][j], acc[i][j], 0, 0, 0);
  }
  __builtin_amdgcn_s_waitcnt(0x0070);                           // vmcnt(0) lgkmcnt(0): also where a wavefront had no slice
  __syncthreads();
  float* part = (float*)smem_raw + wave * TILE * LD;
#pragma unroll
  for (int i = 0; i < T32; ++i)
#pragma unroll
    for (int j = 0; j < T32; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        part[(i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)) * LD + j * 32 + (lane & 31)] = acc[i][j][r];
  __syncthreads();
  constexpr bool SUMS = EPI == EPI_MUL;
  float cs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int idx = threadIdx.x + q * 64 * NW;
    const int row = idx / CH, c = (idx % CH) * 8, m = m0 + row, n = n0 + c;
    if ((CHUNKS >= 64 * NW || idx < CHUNKS) && m < d.M && n < d.N) {
      float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < NW; ++w) {                            // partial tiles in wavefront order
        const float* p = (const float*)smem_raw + (w * TILE + row) * LD + c;
        const f32x4 lo = *(const f32x4*)p, hi = *(const f32x4*)(p + 4);
#pragma unroll
        for (int j = 0; j < 4; ++j) { v[j] += lo[j]; v[4 + j] += hi[j]; }
      }
      float st8[8];
      epilogue8<EPI>(d, m, n, v, ops[q].pre, ops[q].bias, lds0 + SM::TABLE_OFF, SUMS ? st8 : nullptr);
      if (SUMS) {
#pragma unroll
        for (int j = 0; j < 8; ++j) cs[j] += st8[j];
      }
    }
  }
  if (SUMS && d.tile_colsum != nullptr) {                       // uniform: column sums of the stored outputs
    // lanes of a wavefront that share the 8 columns, then the wavefronts that hold rows of the tile, in order
#pragma unroll
    for (int o = CH; o < 64; o <<= 1)
#pragma unroll
      for (int j = 0; j < 8; ++j) cs[j] += __shfl_xor(cs[j], o, 64);
    constexpr int WAVES = CHUNKS >= 64 * NW ? NW : CHUNKS / 64; // wavefronts that stored something
    __syncthreads();
    float* x = (float*)smem_raw;
    if (wave < WAVES && lane < CH)
#pragma unroll
      for (int j = 0; j < 8; ++j) x[wave * TILE + lane * 8 + j] = cs[j];
    __syncthreads();
    if (threadIdx.x < TILE && n0 + (int)threadIdx.x < d.N) {
      float t = x[threadIdx.x];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) t += x[w * TILE + threadIdx.x];
      d.tile_colsum[(long)tm * d.N + n0 + threadIdx.x] = t;
    }
  }
}

template <int T32, int NW, bool B_K, int EPI>
static hipError_t launch_split(hipStream_t s, const GemmDesc& d) {
  typedef SmemSplit<T32, NW, B_K, EPI> SM;
  constexpr auto kern = gemm_mfma_split_kernel<T32, NW, B_K, EPI>;
  const hipError_t e = ensure_lds_attribute<kern, SM::BYTES>();
  if (e != hipSuccess) return e;
  const int tiles_m = (d.M + SM::TILE - 1) / SM::TILE, tiles_n = (d.N + SM::TILE - 1) / SM::TILE;
  if (EPI == EPI_MUL && d.tile_colsum != nullptr && d.tile_colsum_parts != nullptr) *d.tile_colsum_parts = tiles_m;
  hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(64 * NW), SM::BYTES, s, d);
  return hipGetLastError();
}

static std::atomic<int> g_forced_stages{0};      // test / tuning knob, process-wide
int set_gemm_stages(int n) { return g_forced_stages.exchange(n); }

template <int WM, int WN, bool A_K, bool B_K, int EPI>
static hipError_t launch_cfg(hipStream_t s, const GemmDesc& d, int ns) {
  const int tiles = ((d.M + 64 * WM - 1) / (64 * WM)) * ((d.N + 64 * WN - 1) / (64 * WN));
  const int nk = k_slices(d.K);
  if (g_forced_stages) ns = g_forced_stages;
  if (ns > nk) ns = nk >= 3 ? 3 : 2;     // no ring deeper than the contraction
  constexpr bool G = is_gelu(EPI);
  if constexpr (SmemPl<WM, WN, 4, G>::BYTES <= 160 * 1024) {
    if (ns == 4) return launch_pl<WM, WN, A_K, B_K, EPI, 4>(s, d, tiles);
  }
  if constexpr (SmemPl<WM, WN, 3, G>::BYTES <= 160 * 1024) {
    if (ns >= 3) return launch_pl<WM, WN, A_K, B_K, EPI, 3>(s, d, tiles);
  }
  return launch_pl<WM, WN, A_K, B_K, EPI, 2>(s, d, tiles);
}

static std::atomic<int> g_forced_tile{0};        // test / tuning knob, process-wide
bool gemm_tile_code_valid(int code) {
  return code == 0 || code == 44 || code == 43 || code == 42 || code == 24 || code == 22 || code == 11;
}
int set_gemm_tile(int code) { return g_forced_tile.exchange(code); }

// Tile and pipeline-depth choice.  Each candidate's run time is estimated as
//   rounds * (a + b * slices) + c   [microseconds]
// where slices = K / 64, a is the per-tile fill and epilogue cost, b the time of one 64-deep slice, c a launch
// constant, and rounds = tiles / (256 CUs * workgroups that fit a CU), a partial last round of a fraction f of the
// CUs counting 0.75 + 0.25 f (with fewer matrix cores busy the clock is higher: a 256 x 256 slice takes 1.03 us on
// 64 CUs and 1.4 us on 256).  The coefficients are fits to timings of 29 shapes (1024 to 12000 rows, N and K 512 to
// 50304: the BERT-large-, GPT-2- and large-layer-shaped products, the LM head and generic ones) on an MI355X with
// operands that are not cache-resident, as inside a training iteration; the candidate they pick is on average 0.6 %
// and at most 6 % slower than the best one (2048 x 12288 x 49152: 256 x 256 tiles 2056 us, 128 x 256 2440 us).
struct TileCost { int code, ns; float a, b, c; };
static const TileCost kCostStore[] = {     // bf16 output (forward and input-gradient forms)
    {11, 2, 0.02f, 0.452f, 2.72f}, {11, 4, 0.35f, 0.457f, 1.55f}, {22, 2, 2.58f, 1.057f, 0.25f},
    {22, 3, 2.05f, 0.578f, 2.21f}, {24, 3, 4.69f, 0.918f, 1.96f}, {42, 3, 4.05f, 0.934f, 2.45f},
    {44, 2, 10.33f, 1.370f, 0.f},
    // 256 x 192 (offered for the bias-only forward form: N = 3 H of the QKV projection is 16 x 192 when
    // H = 1024, i.e. with 4096 tokens exactly 256 tiles)
    {43, 2, 4.41f, 1.370f, 3.69f}};
static const TileCost kCostAcc[] = {       // fp32 read-modify-write output (weight-gradient form)
    {11, 2, 0.69f, 0.444f, 6.39f}, {11, 4, 1.88f, 0.438f, 2.32f}, {22, 2, 12.15f, 0.935f, 0.f},
    {22, 3, 5.78f, 0.564f, 3.32f}, {24, 3, 9.21f, 0.981f, 3.42f}, {42, 3, 9.66f, 0.958f, 3.31f},
    {44, 2, 28.80f, 1.223f, 0.f}};
// The same for the four products of a layer in one launch (launch_gemm_group_mfma), whose tiles share the rounds: fits to
// timings of 18 groups.  Timed again with the present epilogue (accumulate4), microseconds:
//   tokens  layer         128 x 128, three deep   128 x 128, two deep, two per CU   256 x 256   128 x 256   256 x 128
//   128      768 x 3072    14.8                    14.3                              20.6        14.6        16.2
//   128     1024 x 4096    22.3                    22.4                              27.9        27.7        28.6
//   768     1024 x 4096    35.7                    38.1                              39.9        41.2        42.6
//   2048    1024 x 4096    63.8                    67.7                              63.6        73.3        72.0
//   4096    1024 x 4096   113.1                   126.0                             101.7       127.9       122.7
//   128     1600 x 6400    49.9                    48.0                              59.3        51.9        55.2
//   1024    1600 x 6400   102.5                    90.5                              96.2       100.0       111.5
//   4096    1600 x 6400   317.8                   283.4                             284.3       282.6       311.5
//   4096    1280 x 5120   205.2                   202.7                             202.7       202.4       197.1
// Two workgroups on a CU overlap one's gradient reads and writes, which are most of a short product's time, with the other's
// loop.  Over 65 groups (layers of 512 x 2048 to 2048 x 8192, 64 to 4096 tokens) the choice by these coefficients takes 0.4 %
// more than the best of the five tiles, at most 6.7 % (768 tokens of 1024 x 4096); a least-squares fit to all of them 1.2 % and
// 21 %.  128 x 256 and 256 x 128 are not offered: the best in two of the 65, by 0.3 and 2.5 %.
static const TileCost kCostGroup[] = {
    {22, 3, 5.3f, 0.51f, 4.0f}, {22, 2, 9.6f, 0.84f, 1.1f}, {44, 2, 29.5f, 1.30f, 0.f}};
static float rounds_of(long tiles, long slots) {
  const long full = tiles / slots, rest = tiles % slots;
  return (float)full + (rest > 0 ? 0.75f + 0.25f * (float)rest / (float)slots : 0.f);
}

// *code = 0: no tile's loads reach that far
static float choose_tile(const GemmDesc& d, bool acc_form, long extra_lds, bool by_work, int* code, int* ns,
                         bool offer_43 = false) {
  const int nk = k_slices(d.K);
  const TileCost* tab = acc_form ? kCostAcc : kCostStore;
  const int ntab = acc_form ? (int)(sizeof(kCostAcc) / sizeof(kCostAcc[0])) : (int)(sizeof(kCostStore) / sizeof(kCostStore[0]));
  float best = 0.f;
  bool found = false;
  *code = 0;
  *ns = 2;
  for (int i = 0; i < ntab; ++i) {
    const TileCost& t = tab[i];
    if (t.ns > nk && t.ns > 2) continue;
    if (t.code == 43 && !offer_43) continue;
    const int wm = t.code / 10, wn = t.code % 10;
    if (!tile_in_reach(d, 64 * wm, 64 * wn)) continue;
    const long tiles = (long)((d.M + 64 * wm - 1) / (64 * wm)) * ((d.N + 64 * wn - 1) / (64 * wn));
    const long stage = (long)(wm + wn) * 64 * BK * 2, epi = 4L * 32 * (32 * wn + 4) * 4;
    const long lds = (t.ns * stage > epi ? t.ns * stage : epi) + extra_lds;
    if (lds > 160 * 1024) continue;
    const long slots = 256 * (2 * lds <= 160 * 1024 ? 2 : 1);
    // alone on the chip: rounds of tiles.  Beside another stream's kernels: CU time summed over the tiles, but
    // no shape that leaves fewer than 128 tiles where another offers more -- the launch still has to finish
    // (measured: with 64-tile launches on the second lane that lane becomes the critical path).
    const float cost = by_work ? (float)(tiles < 128 ? 4 * 256 : tiles) * (t.a + t.b * nk) : rounds_of(tiles, slots) * (t.a + t.b * nk) + t.c;
    if (!found || cost < best) {
      found = true;
      best = cost;
      *code = t.code;
      *ns = t.ns;
    }
  }
  return best;
}

// Whether the wavefronts of a workgroup should split K (gemm_mfma_split_kernel): 0 no, 1 with 32 x 32, 2 with
// 64 x 64 tiles.  Estimated like the tiles above, rounds * (a + b * slices), one workgroup per CU; fitted to
// timings of 54 shapes (16 to 2048 rows, N 256 to 4096, K 1024 to 6400; microseconds, forward / input gradient):
//     rows  N     K      tiles        split 32        split 64
//     128   1024  1024    6.6 /  6.5    4.1 /  4.1      6.4 /  6.3
//     128   1024  4096   31.0 / 31.2   11.9 /  8.4     16.0 / 13.7
//     512   1024  4096   31.7 / 31.7   19.3 / 14.9     15.2 / 14.7
//     1000  1024  4096   31.8 / 31.8   35.0 / 27.1     16.5 / 16.0
//     1536  1024  4096   32.7 / 32.5   50.8 / 39.3     28.9 / 27.9
//     512   3072  1024   11.0 / 10.8   22.9 / 18.4     12.9 / 12.1
// i.e. splitting pays where one round of small tiles covers the output, and more the longer K is.  The choice depends
// on the shape alone (not on the stream, nor on a forced tile; a forced ring depth rules the split out): the sums are
// taken in another order than the tiles'.
// row_sums: the kernel may be asked for column sums, one row per tile row: not with more of them than the buffers hold.
static int choose_split(const GemmDesc& d, bool b_k, long extra_lds, bool row_sums) {
  int code, ns;
  float best = choose_tile(d, false, extra_lds, false, &code, &ns);
  const int nk = k_slices(d.K);
  int pick = 0;
  for (int t = 1; t <= 2; ++t) {
    const long tiles = (long)((d.M + 32 * t - 1) / (32 * t)) * ((d.N + 32 * t - 1) / (32 * t));
    const long rounds = (tiles + 255) / 256;
    if (!tile_in_reach(d, 32 * t, 32 * t)) continue;
    if (row_sums && (size_t)((d.M + 32 * t - 1) / (32 * t)) > reduce_max_partials()) continue;
    const float cost = rounds * (t == 1 ? (b_k ? 2.7f + 0.09f * nk : 1.5f + 0.16f * nk) : 4.0f + 0.18f * nk);
    if (cost < best || (code == 0 && pick == 0)) {
      best = cost;
      pick = t;
    }
  }
  return pick;
}

template <bool A_K, bool B_K, int EPI>
static hipError_t launch_form(hipStream_t s, GemmDesc d) {
  if (is_gelu(EPI)) {
    const hipError_t e = ensure_gelu_table(s);
    if (e != hipSuccess) return e;
  }
  if constexpr (EPI != EPI_ACC_F32) {
    // a forced ring depth is one of the tiled kernel's
    switch (d.tiled_only || g_forced_stages ? 0 : choose_split(d, B_K, is_gelu(EPI) ? kGeluBytes : 0, EPI == EPI_MUL)) {
      case 1: return launch_split<1, 8, B_K, EPI>(s, d);
      case 2: return launch_split<2, 4, B_K, EPI>(s, d);
      default: break;
    }
  }
  int pick, ns;
  constexpr bool HAS_43 = A_K && !B_K && EPI == EPI_BIAS;
  choose_tile(d, EPI == EPI_ACC_F32, is_gelu(EPI) ? kGeluBytes : 0, d.shared_chip != 0, &pick, &ns, HAS_43 && !g_forced_stages);
  const int forced = g_forced_tile == 43 && !HAS_43 ? 44 : (int)g_forced_tile;   // 256 x 192 where this form has it
  if (forced && tile_in_reach(d, 64 * (forced / 10), 64 * (forced % 10))) {
    pick = forced;
    ns = 2;
  }
  if (pick == 0) return hipErrorNotSupported;
  if (EPI == EPI_MUL && d.tile_colsum != nullptr && d.tile_colsum_parts != nullptr) {
    const int rows = (d.M + 64 * (pick / 10) - 1) / (64 * (pick / 10));         // one row of column sums per tile row
    if ((size_t)rows <= reduce_max_partials()) *d.tile_colsum_parts = rows;
    else d.tile_colsum = nullptr;                                               // left to launch_gemm
  }
  if constexpr (HAS_43) {
    if (pick == 43) {
      const int tiles = ((d.M + 255) / 256) * ((d.N + 191) / 192);
      return launch_pl<4, 3, A_K, B_K, EPI, 2>(s, d, tiles);
    }
  }
  switch (pick) {
    case 44: return launch_cfg<4, 4, A_K, B_K, EPI>(s, d, ns);
    case 42: return launch_cfg<4, 2, A_K, B_K, EPI>(s, d, ns);
    case 24: return launch_cfg<2, 4, A_K, B_K, EPI>(s, d, ns);
    case 22: return launch_cfg<2, 2, A_K, B_K, EPI>(s, d, ns);
    case 11: return launch_cfg<1, 1, A_K, B_K, EPI>(s, d, ns);
    default: return hipErrorInvalidValue;
  }
}

// How a launch of 256 x 256 tiles covers an M x N output: tm x tn of them, and strips half as wide along an edge whose
// remainder needs no more.
static int edge_strips(int M, int N, int* tm, int* tn) {
  const bool low = M > 256 && M % 256 > 0 && M % 256 <= 128, right = N > 256 && N % 256 > 0 && N % 256 <= 128;
  *tm = low ? M / 256 : (M + 255) / 256;
  *tn = right ? N / 256 : (N + 255) / 256;
  return (low ? (N + 255) / 256 : 0) + (right ? *tm : 0);
}
// What a strip of a launch of 256 x 256 tiles takes of a tile's time: 0.67 at 64 slices (from the coefficients above)
static float strip_share(float slices) { return (9.5f + 0.97f * slices) / (28.8f + 1.223f * slices); }

template <int WM, int WN, int NS>
static hipError_t launch_group_cfg(hipStream_t s, GemmGroup& g) {
  typedef SmemPl<WM, WN, NS, false> SM;
  constexpr bool STRIPS = WM == 4 && WN == 4;
  constexpr int BYTES = STRIPS && SmemPl<2, 4, 3>::BYTES > SM::BYTES ? SmemPl<2, 4, 3>::BYTES : SM::BYTES;
  static_assert(!STRIPS || (SmemPl<4, 2, 3>::BYTES <= BYTES && BYTES <= 160 * 1024), "");
  constexpr auto kern = gemm_mfma_pl_group_kernel<WM, WN, NS, (2 * BYTES <= 160 * 1024 ? 2 : 1)>;
  const hipError_t e = ensure_lds_attribute<kern, BYTES>();
  if (e != hipSuccess) return e;
  int total = 0, strips = 0;
  long slices = 0;
  for (int i = 0; i < g.n; ++i) {
    g.first[i] = total;
    g.strip0[i] = strips;
    if (STRIPS) {
      strips += edge_strips(g.d[i].M, g.d[i].N, &g.tiles_m[i], &g.tiles_n[i]);
    } else {
      g.tiles_m[i] = (g.d[i].M + 64 * WM - 1) / (64 * WM);
      g.tiles_n[i] = (g.d[i].N + 64 * WN - 1) / (64 * WN);
    }
    total += g.tiles_m[i] * g.tiles_n[i];
    slices += k_slices(g.d[i].K);
  }
  for (int i = g.n; i <= GemmGroup::MAX; ++i) {
    g.first[i] = total;
    g.strip0[i] = strips;
  }
  // As many strips in a row as fit the rounds of the launch (three in two rounds), started first: the CUs that take
  // them finish with the others, where strips left for the end would have added a round of their own.
  const float share = strip_share((float)slices / g.n);
  const float rounds = ceilf(((float)total + share * (float)strips) / 256.f);
  g.chain = strips > 0 ? std::max(1, (int)(rounds / share + 0.05f)) : 1;
  g.chains = (strips + g.chain - 1) / g.chain;
  // One round of tiles: XCD ranges over the whole launch halve what the L2s fetch (measured at the
  // BERT-large-shaped stage: 231 instead of 440 MiB per launch, 1.3 x the operands) at the same run time.
  // Over several rounds the per-problem ranges are faster (GPT-2-shaped stage: 288 against 302 us), so
  // they stay there.
  g.whole_launch_ranges = total <= 256 * (2 * BYTES <= 160 * 1024 ? 2 : 1) ? 1 : 0;
  static_assert(BYTES >= kReduceLdsFloats * 4, "the tail workgroups use the front of the tile ring");
  total += g.chains + grad_reduce_blocks(g.tail);
  hipLaunchKernelGGL(kern, dim3(total), dim3(256), BYTES, s, g);
  return hipGetLastError();
}

static bool wgrad_form_ok(const GemmDesc& d) {
  if (d.epi != EPI_ACC_F32 || d.a_sk == 1 || d.b_sk == 1 || d.a_sm != 1 || d.b_sn != 1) return false;
  if (d.M % 8 || d.N % 8 || d.a_sk % 8 || d.b_sk % 8) return false;
  if (((uintptr_t)d.A | (uintptr_t)d.B | (uintptr_t)d.C) & 15) return false;
  return d.M > 0 && d.N > 0;
}

// n <= GemmGroup::MAX weight-gradient GEMMs (dW += X^T dY) as one launch where the pipelined MFMA kernel
// covers all of them with one tile shape; hipErrorNotSupported otherwise (the caller launches them singly).
hipError_t launch_gemm_group_mfma(hipStream_t s, const GemmDesc* d, int n, const GradReduceBatch* tail) {
  if (n < 1 || n > GemmGroup::MAX) return hipErrorNotSupported;
  GemmGroup g;
  memset(&g, 0, sizeof(g));
  g.n = n;
  if (tail != nullptr) g.tail = *tail;
  for (int i = 0; i < n; ++i) {
    if (!wgrad_form_ok(d[i])) return hipErrorNotSupported;
    g.d[i] = d[i];
  }
  // Tile shape for the whole group: the cheapest by the cost model, with all tiles of the group sharing the rounds.
  int pick = 0, depth = 0;
  float best = 0.f;
  for (const TileCost& t : kCostGroup) {
    const int wm = t.code / 10, wn = t.code % 10;
    bool reached = true;
    for (int i = 0; i < n; ++i) reached = reached && tile_in_reach(d[i], 64 * wm, 64 * wn);
    if (!reached) continue;
    long tiles = 0;
    double slices = 0;
    for (int i = 0; i < n; ++i) {
      long ti = (long)((d[i].M + 64 * wm - 1) / (64 * wm)) * ((d[i].N + 64 * wn - 1) / (64 * wn));
      if (t.code == 44) {
        int tm, tn;
        const int strips = edge_strips(d[i].M, d[i].N, &tm, &tn);
        ti = (long)tm * tn + (long)ceilf(strips * strip_share((float)k_slices(d[i].K)));
      }
      tiles += ti;
      slices += (double)ti * k_slices(d[i].K);
    }
    const bool pairs = t.code == 22 && t.ns == 2;            // two workgroups to a CU
    const float cost = rounds_of(tiles, pairs ? 512 : 256) * (t.a + t.b * (float)(slices / tiles)) + t.c;
    if (pick == 0 || cost < best) {
      pick = t.code;
      depth = t.ns;
      best = cost;
    }
  }
  if (pick == 0) return hipErrorNotSupported;
  if (g_forced_tile == 22 || g_forced_tile == 44) {
    for (int i = 0; i < n; ++i)
      if (!tile_in_reach(d[i], 64 * (g_forced_tile / 10), 64 * (g_forced_tile % 10))) return hipErrorNotSupported;
    pick = g_forced_tile;
    depth = g_forced_stages == 2 ? 2 : 3;          // of the 128 x 128 tile; the others have one
  } else if (g_forced_tile || g_forced_stages) {
    return hipErrorNotSupported;   // a forced shape this launch does not offer
  }
  if (pick == 44) return launch_group_cfg<4, 4, 2>(s, g);
  return depth == 2 ? launch_group_cfg<2, 2, 2>(s, g) : launch_group_cfg<2, 2, 3>(s, g);
}

hipError_t launch_gemm_mfma(hipStream_t s, const GemmDesc& d) {
  const bool a_k = d.a_sk == 1, b_k = d.b_sk == 1;
  if (!a_k && d.a_sm != 1) return hipErrorNotSupported;
  if (!b_k && d.b_sn != 1) return hipErrorNotSupported;
  // 16-byte accesses everywhere: the contiguous dimension of each operand and of the output, and the leading
  // dimensions, in multiples of 8 (the rows of A and C and a contraction index that is strided in both operands
  // may have any length)
  const long lda = a_k ? d.a_sm : d.a_sk, ldb = b_k ? d.b_sn : d.b_sk;
  if (d.N % 8 || lda % 8 || ldb % 8 || (a_k || b_k ? d.K % 8 != 0 : false) || (!a_k && d.M % 8)) return hipErrorNotSupported;
  auto misaligned = [](const void* p) { return p != nullptr && ((uintptr_t)p & 15) != 0; };
  if (misaligned(d.A) || misaligned(d.B) || misaligned(d.C) || misaligned(d.bias) || misaligned(d.res) ||
      misaligned(d.aux_in) || misaligned(d.aux_out))
    return hipErrorNotSupported;
  if (a_k && !b_k) {           // forward
    switch (d.epi) {
      case EPI_STORE: return launch_form<true, false, EPI_STORE>(s, d);   // the LM head has no bias
      case EPI_BIAS: return launch_form<true, false, EPI_BIAS>(s, d);
      case EPI_BIAS_RES: return launch_form<true, false, EPI_BIAS_RES>(s, d);
      case EPI_BIAS_GELU:
        return d.M % 8 ? launch_form<true, false, EPI_BIAS_GELU_FINE>(s, d) : launch_form<true, false, EPI_BIAS_GELU>(s, d);
      default: return hipErrorNotSupported;
    }
  }
  if (a_k && b_k) {            // input gradient
    switch (d.epi) {
      case EPI_STORE: return launch_form<true, true, EPI_STORE>(s, d);
      case EPI_RES: return launch_form<true, true, EPI_RES>(s, d);
      case EPI_MUL: return launch_form<true, true, EPI_MUL>(s, d);
      default: return hipErrorNotSupported;
    }
  }
  if (!a_k && !b_k && d.epi == EPI_ACC_F32) return launch_form<false, false, EPI_ACC_F32>(s, d);
  return hipErrorNotSupported;
}

}  // namespace bamboo
