// Tiled softmax attention on the gfx950 matrix cores (bf16 in, fp32 softmax and
// accumulation), head size 64 or 128, any sequence length.
//
// Forward: a wavefront owns 32 queries and streams 64-key tiles through LDS.  It
// computes the TRANSPOSED score tile S^T = K Q^T, so a lane owns one query and
// its registers run over keys: the row maximum and row sum of the online
// softmax are then plain per-lane reductions (one exchange with the other
// half-wave), and the rescaling of the running output is a per-lane scalar.
// The probabilities never leave registers: in the MFMA accumulator layout a
// lane's 16 values of a 32x32 tile are 16 keys of its query, which is exactly an
// operand fragment of O^T = V^T P^T once V is read from LDS with the transposing
// load (ds_read_b64_tr_b16) in the matching key order.  Only the per-row
// log-sum-exp is kept for the backward.
//
// Backward recomputes the probabilities from the log-sum-exp and uses no
// atomics: one kernel owns query rows (dQ), one owns key rows (dK, dV), so the
// result is bitwise reproducible.
#include "common.h"

namespace bamboo {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short short4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kMasked = -1.0e30f;
constexpr int TILE = 64;   // rows streamed through LDS per step

// Workgroup -> (row block, batch*head).  The grid is one-dimensional and ordered by row block
// first, all (batch, head) pairs of a row block being consecutive; with a causal mask the row
// blocks with the most key tiles to visit come first (HEAVY_LAST: the highest row block is the
// heaviest, as for query owners; otherwise the lowest, as for key owners), so the dispatcher
// hands out long workgroups first and the short ones fill the tail of the launch.
template <bool CAUSAL, bool HEAVY_LAST>
__device__ __forceinline__ void block_of(int wg, int nblk, int nbh, int* blk, int* bh) {
  const int i = wg / nbh;
  *bh = wg % nbh;
  *blk = (CAUSAL && HEAVY_LAST) ? nblk - 1 - i : i;
}

// ---- cooperative copy of 64 rows x D (bf16) global -> LDS ---------------------------
// The tiles go straight to LDS (global_load_lds_dwordx4: 16 bytes per lane to consecutive addresses behind a
// wavefront-uniform base), so nothing waits in registers and no LDS store is issued.  Rows are not padded; the 16-byte
// chunk ch of row r sits at position ch ^ swz(r) of its row, which every lane applies to the chunk that it FETCHES.  The
// placement serves both ways a tile is read: 16 consecutive rows of one chunk (frag_k) and 4 rows x 64 bytes (frag_tr)
// each cover the 64 banks once.  With the rows padded to D + 8 (D + 16 for the values of the forward pass) and staged
// through registers the second kind, half of the backward's reads, met its own banks twice.  Backward in us, before and now
// (samples x tokens x heads x size; the forward: see fwd_launch):
//   8 x 512 x 16 x 64   45.0 / 42.6     4 x 1024 x 25 x 64 causal   81.3 / 79.8     1 x 2048 x 96 x 128 causal  613 / 512
//   4 x 512 x 16 x 64   23.7 / 22.8     2 x 2048 x 25 x 64 causal  129.9 / 129.2    2 x 512 x 24 x 128        52.9 / 50.1
//   3 x 333 x 16 x 64   17.3 / 16.7     1 x 8192 x 16 x 64 causal  517 / 492        1 x 1500 x 20 x 128 causal 136.5 / 124.6
// What bounds both passes is still a wavefront's own chain of matrix and vector instructions, at two wavefronts per SIMD.
// Rows at or beyond row_lim are read from row row_lim - 1 (finite values that the consumers' masks turn
// into exact zeros), so no load sits behind a branch.  A thread's byte offsets inside a tile and their
// upper limits (the same chunk in the last valid row) are computed once; per tile and chunk an add and a
// min remain.  Offsets are 32-bit: the launcher checks that a sequence stays below 4 GiB.
// The loads are inline assembly, which the compiler's wait counts do not see: wait_tiles() before the barrier that
// publishes a tile.
template <int D>
__device__ __forceinline__ int swz(int r) {
  return D == 64 ? ((r & 2) << 1) | ((r >> 2) & 3)       // rows of 128 bytes: two to a line of the 64 banks
                 : ((r & 3) << 2) | ((r >> 2) & 3);      // rows of 256 bytes
}
typedef __attribute__((address_space(3))) void* lds_void_ptr;
__device__ __forceinline__ unsigned lds_address(const void* p) { return (unsigned)(uintptr_t)(lds_void_ptr)p; }
template <int D>
struct TileCopy {
  static constexpr int N = TILE * D / 8 / 256;   // 16-byte chunks per thread
  static constexpr int BYTES = TILE * D * 2;
  unsigned ofs[N], last[N];
  unsigned tile_bytes;                           // 64 rows
  unsigned wave_lds;
  __device__ __forceinline__ void init(long row_stride, int row_lim) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int c = threadIdx.x + i * 256, r = c / (D / 8);
      const unsigned col = (unsigned)(((c % (D / 8)) ^ swz<D>(r)) * 8) * 2u;
      ofs[i] = (unsigned)r * (unsigned)row_stride * 2u + col;
      last[i] = (unsigned)(row_lim - 1) * (unsigned)row_stride * 2u + col;
    }
    tile_bytes = (unsigned)TILE * (unsigned)row_stride * 2u;
    wave_lds = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 1024;
  }
  // tile: index of the 64-row tile counted from g; lds: where it goes (all uniform)
  __device__ __forceinline__ void issue(const bf16_t* g, int tile, unsigned lds) const {
    const unsigned t0 = (unsigned)tile * tile_bytes;
#pragma unroll
    for (int i = 0; i < N; ++i)
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                   :
                   : "v"(min(t0 + ofs[i], last[i])), "s"(g), "s"(lds + wave_lds + i * 4096)
                   : "memory", "m0");
  }
};
// at most the N youngest of this wavefront's loads are still on their way
template <int N>
__device__ __forceinline__ void wait_tiles() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// The same placement through registers: requested (fetch) ahead of a step, put into LDS (stash) behind it.
template <int D>
struct RegCopy {
  static constexpr int N = TileCopy<D>::N;
  bf16x8 v[N];
  __device__ __forceinline__ void fetch(const TileCopy<D>& c, const bf16_t* g, int tile) {
    const unsigned t0 = (unsigned)tile * c.tile_bytes;
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = *(const bf16x8*)((const char*)g + min(t0 + c.ofs[i], c.last[i]));
  }
  __device__ __forceinline__ void stash(unsigned lds) const {
    typedef __attribute__((address_space(3))) bf16x8* lds_ptr;
#pragma unroll
    for (int i = 0; i < N; ++i) *(lds_ptr)(lds + i * 4096) = v[i];
  }
};

// Addresses of the operand fragments.  Tiles are 256-byte aligned and the placement moves bits 4 to 7 only, so a fragment's
// address is the slot's + (row 0, this lane's chunk ^ chunk) + an immediate offset for the tile in the slot and the row.
// HELD: one register per chunk, and with slots that are constants (for_each_tile) no address arithmetic in a step: the
// forward 0.94 to 0.98 of the time with addresses formed in each.  The backward passes, where registers are short, form
// them from chunk 0, once for both tiles of a slot (held there: 1.02 to 1.08 of the time, from other schedules and spills).
template <int D, bool HELD>
struct FragAddr {
  unsigned k[HELD ? D / 16 : 1];       // frag_k at row 0
  unsigned tr[HELD ? D / 32 : 1][2];   // frag_tr at row 0: its two halves
  __device__ __forceinline__ void init(unsigned ring) {
    const int l = threadIdx.x & 63, i = l & 15, q = 4 * (l >> 5) + (i >> 2);
    const int ch = ((l >> 4) & 1) * 2 + ((i & 3) >> 1);
#pragma unroll
    for (int ks = 0; ks < (HELD ? D / 16 : 1); ++ks)
      k[ks] = ring + (l & 31) * D * 2 + ((((l >> 5) ^ swz<D>(l & 31)) ^ (2 * ks)) << 4);
#pragma unroll
    for (int dt = 0; dt < (HELD ? D / 32 : 1); ++dt)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        tr[dt][h] = ring + (q + 8 * h) * D * 2 + (((ch ^ swz<D>(q + 8 * h)) ^ (4 * dt)) << 4) + (i & 1) * 8;
  }
  // Operand fragment with the contraction index contiguous in LDS: lane l holds
  // row row_base + l%32, contraction elements 16*ks + 8*(l/32) .. +7.
  __device__ __forceinline__ bf16x8 frag_k(unsigned slot, unsigned tile, int row_base, int ks) const {
    typedef __attribute__((address_space(3))) const bf16x8* lds_ptr;
    const unsigned at = HELD ? k[HELD ? ks : 0] + slot : (k[0] + slot) ^ (ks << 5);
    return *(lds_ptr)(at + (tile + row_base * D * 2));
  }
  // Operand fragment with the contraction index running over LDS rows (transposing
  // load): lane l holds column 32*dt + l%32; its 8 contraction slots are rows
  // kbase + 4*(l/32) + {0..3} and kbase + 8 + 4*(l/32) + {0..3} -- the order in
  // which a 32x32 accumulator tile hands 8 of a lane's 16 values to the next MFMA.
  __device__ __forceinline__ bf16x8 frag_tr(unsigned slot, unsigned tile, int dt, int kbase) const {
    typedef __attribute__((address_space(3))) short4_t* lds_ptr;
    union { short4_t s4[2]; bf16x8 b; } u;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const unsigned at = HELD ? tr[HELD ? dt : 0][h] + slot : (tr[0][h] + slot) ^ (dt << 6);
      u.s4[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(at + (tile + kbase * D * 2)));
    }
    return u.b;
  }
};
// step(t, slot) for t = 0 .. nt - 1, slot = t mod 2 as a constant
template <typename STEP>
__device__ __forceinline__ void for_each_tile(int nt, STEP step) {
  for (int t = 0; t < nt; t += 2) {
    step(t, 0);
    if (t + 1 < nt) step(t + 1, 1);
  }
}
// registers 8*half .. 8*half+7 of an accumulator tile as a bf16 operand fragment
__device__ __forceinline__ bf16x8 pack8(const f32x16& t, int half) {
  bf16x8 o;
#pragma unroll
  for (int j = 0; j < 8; ++j) o[j] = (bf16_t)t[8 * half + j];
  return o;
}
// the value the lane 32 places away holds (v_permlane32_swap: no trip through LDS)
__device__ __forceinline__ float other_half(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  // r[0]: lanes 0..31 keep theirs, lanes 32..63 receive the lower half's; r[1]: the other way round
  const unsigned lo = r[0], hi = r[1];
  return __builtin_bit_cast(float, (threadIdx.x & 32) ? lo : hi);
}
// row index inside a 32x32 accumulator tile of register r for this lane
__device__ __forceinline__ int acc_row(int r) { return 8 * (r >> 2) + 4 * ((threadIdx.x & 63) >> 5) + (r & 3); }

// Per-lane operand fragments of 32 rows taken straight from global memory
// (lane l: row row0 + l%32, elements 16*ks + 8*(l/32) .. +7), zero beyond row_lim.
template <int D>
__device__ __forceinline__ void load_row_frags(bf16x8 (&f)[D / 16], const bf16_t* g, long row_stride, int row0,
                                               int row_lim) {
  const int l = threadIdx.x & 63;
  const int row = row0 + (l & 31);
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) {
    bf16x8 t = {};
    if (row < row_lim) t = *(const bf16x8*)(g + (long)row * row_stride + ks * 16 + (l >> 5) * 8);
    f[ks] = t;
  }
}

// Write a wavefront's transposed result (lane = output row, accumulator rows =
// feature index) through its private LDS area to global rows of D features.
// cs (optional): the lane's running sums of the 8 columns it stores (every pass meets the same 8, as 64 is a
// multiple of the chunks per row), over the rows it stores.
template <int D, bool SUM>
__device__ __forceinline__ void store_rows_impl(const f32x16 (&acc)[D / 32], float mul, bf16_t* stage, bf16_t* g,
                                                long row_stride, int row0, int row_lim, float (&cs)[8]) {
  constexpr int LD = D + 8;
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      bf16x4 o;
#pragma unroll
      for (int c = 0; c < 4; ++c) o[c] = (bf16_t)(acc[dt][4 * a + c] * mul);
      *(bf16x4*)(stage + (l & 31) * LD + dt * 32 + 8 * a + 4 * (l >> 5)) = o;
    }
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int it = 0; it < 32 * (D / 8) / 64; ++it) {
    const int idx = l + it * 64;
    const int row = idx / (D / 8), ch = (idx % (D / 8)) * 8;
    const bf16x8 t = *(const bf16x8*)(stage + row * LD + ch);
    if (row0 + row < row_lim) {
      *(bf16x8*)(g + (long)(row0 + row) * row_stride + ch) = t;
      if (SUM) {
#pragma unroll
        for (int j = 0; j < 8; ++j) cs[j] += (float)t[j];
      }
    }
  }
  __builtin_amdgcn_wave_barrier();
}

template <int D>
__device__ __forceinline__ void store_rows(const f32x16 (&acc)[D / 32], float mul, bf16_t* stage, bf16_t* g,
                                           long row_stride, int row0, int row_lim) {
  float unused[8];
  store_rows_impl<D, false>(acc, mul, stage, g, row_stride, row0, row_lim, unused);
}
template <int D>
__device__ __forceinline__ void store_rows_sum(const f32x16 (&acc)[D / 32], float mul, bf16_t* stage, bf16_t* g,
                                               long row_stride, int row0, int row_lim, float (&cs)[8]) {
  store_rows_impl<D, true>(acc, mul, stage, g, row_stride, row0, row_lim, cs);
}

// Column sums of what the workgroup's four wavefronts stored with store_rows (D columns, 128 rows): lanes that
// share a chunk first, then the wavefronts, both in a fixed order; written to dst[0..D).  xch: 4 * D floats of
// LDS that nobody else uses between the two barriers.  Must be reached by the whole workgroup.
template <int D>
__device__ __forceinline__ void block_colsum_write(float (&cs)[8], float* xch, float* dst) {
  constexpr int CH = D / 8;
  static_assert(64 % CH == 0, "a lane must keep its columns across passes");
  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63;
#pragma unroll
  for (int o = CH; o < 64; o <<= 1)
#pragma unroll
    for (int j = 0; j < 8; ++j) cs[j] += __shfl_xor(cs[j], o, 64);
  __syncthreads();
  if (l < CH)
#pragma unroll
    for (int j = 0; j < 8; ++j) xch[wave * D + l * 8 + j] = cs[j];
  __syncthreads();
  if (wave == 0 && l < CH)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int c = l * 8 + j;
      dst[c] = ((xch[c] + xch[D + c]) + xch[2 * D + c]) + xch[3 * D + c];
    }
}

// =============================================================== forward
// REGS: the tiles pass through registers (see fwd_launch)
template <int D, bool CAUSAL, bool REGS>
__global__ __launch_bounds__(256, D == 64 ? 3 : 2) void attn_fwd_mfma_kernel(AttnDesc a) {
  constexpr unsigned TB = TileCopy<D>::BYTES;
  extern __shared__ __attribute__((aligned(256))) unsigned char smem_raw[];
  // both slots requested ahead of the first step: 2-3 % at head size 64, nothing or -1 % in the other forms
  constexpr bool BOTH = !REGS && D == 64 && !CAUSAL;
  const unsigned ring = lds_address(smem_raw);    // [2][keys, values]
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 5;
  const int H = a.heads * D, S = a.S;
  int qblk, bh;
  block_of<CAUSAL, true>(blockIdx.x, (S + 127) / 128, a.B * a.heads, &qblk, &bh);
  const int b = bh / a.heads, h = bh % a.heads;
  const int q0 = qblk * 128, qw0 = q0 + wave * 32;
  const long rs = 3L * H;
  const bf16_t* base = (const bf16_t*)a.qkv + (long)b * S * rs + h * D;
  const float c = rsqrtf((float)D) * kLog2e;

  bf16x8 qf[D / 16];
  load_row_frags<D>(qf, base, rs, qw0, S);
  f32x16 o[D / 32];
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
  float m_i = kMasked, l_i = 0.f;
  const int query = qw0 + (lane & 31);

  const int kend = CAUSAL ? min(S, q0 + 128) : S;
  const int nt = (kend + TILE - 1) / TILE;
  TileCopy<D> copy;
  copy.init(rs, S);
  FragAddr<D, true> fr;
  fr.init(ring);
  RegCopy<D> kr, vr;
  const unsigned put = ring + threadIdx.x * 16;
  if constexpr (REGS) {
    kr.fetch(copy, base + H, 0);
    vr.fetch(copy, base + 2 * H, 0);
    kr.stash(put);
    vr.stash(put + TB);
    __syncthreads();
  } else {
    copy.issue(base + H, 0, ring);
    copy.issue(base + 2 * H, 0, ring + TB);
    if (BOTH && nt > 1) {
      copy.issue(base + H, 1, ring + 2 * TB);
      copy.issue(base + 2 * H, 1, ring + 3 * TB);
    }
  }
  for_each_tile(nt, [&](int t, int slot) __attribute__((always_inline)) {
    const unsigned at = slot * 2 * TB;
    if constexpr (REGS) {
      if (t + 1 < nt) {
        kr.fetch(copy, base + H, t + 1);
        vr.fetch(copy, base + 2 * H, t + 1);
      }
    } else {
      if (BOTH && t == 0 && nt > 1) wait_tiles<2 * TileCopy<D>::N>();        // tile t has landed
      else wait_tiles<0>();
      __syncthreads();                            // everywhere, and tile t - 1 has been read everywhere
      if ((!BOTH || t > 0) && t + 1 < nt) {
        // formed here: captured, it moves the register allocation of the other form, 3 % of its time at head size 128
        const unsigned ring = lds_address(smem_raw);
        copy.issue(base + H, t + 1, ring + (slot ^ 1) * 2 * TB);
        copy.issue(base + 2 * H, t + 1, ring + (slot ^ 1) * 2 * TB + TB);
      }
    }
    const int k0 = t * TILE;
    if (!CAUSAL || k0 <= qw0 + 31) {              // wave-uniform: tile not entirely above the diagonal
      f32x16 s[2];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[u][r] = 0.f;
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
        for (int u = 0; u < 2; ++u)
          s[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.frag_k(at, 0, u * 32, ks), qf[ks], s[u], 0, 0, 0);
      // Online softmax in the log2 domain.  The running maximum m_i is only raised when some row's
      // maximum has grown by more than 8 (a factor 256, harmless in fp32 and bf16): softmax is
      // invariant to the shift, and the rescaling of the running output then happens on a few
      // tiles instead of on every one.  Tiles that need no masking take a path without the
      // per-element index arithmetic (the choice is uniform over the wavefront).
      const bool need_mask = (k0 + TILE > S) || (CAUSAL && k0 + TILE - 1 > qw0);
      float mx = kMasked;
      if (need_mask) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = k0 + u * 32 + acc_row(r);
            const float v = (key >= S || (CAUSAL && key > query)) ? kMasked : s[u][r] * c;
            s[u][r] = v;
            mx = fmaxf(mx, v);
          }
      } else {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[u][r]);
        mx *= c;
      }
      mx = fmaxf(mx, other_half(mx));
      const bool grow = mx > m_i + 8.f;
      if (__builtin_amdgcn_ballot_w64(grow) != 0) {
        const float m_new = grow ? mx : m_i;
        const float alpha = __builtin_amdgcn_exp2f(m_i - m_new);
        l_i *= alpha;
        m_i = m_new;
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
      }
      if (need_mask) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int r = 0; r < 16; ++r) s[u][r] = __builtin_amdgcn_exp2f(s[u][r] - m_i);
      } else {
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int r = 0; r < 16; ++r) s[u][r] = __builtin_amdgcn_exp2f(fmaf(s[u][r], c, -m_i));
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bf16x8 pb = pack8(s[u >> 1], u & 1);
#pragma unroll
        for (int j = 0; j < 8; ++j) l_i += s[u >> 1][8 * (u & 1) + j];
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.frag_tr(at, TB, dt, 16 * u), pb, o[dt], 0, 0, 0);
      }
    }
    if constexpr (REGS) {
      if (t + 1 < nt) {
        kr.stash(put + (slot ^ 1) * 2 * TB);
        vr.stash(put + (slot ^ 1) * 2 * TB + TB);
      }
      __syncthreads();
    }
  });
  if constexpr (!REGS) __syncthreads();                     // the tiles' place takes the results
  const float l_tot = l_i + __shfl_xor(l_i, 32, 64);
  const float inv = 1.f / l_tot;
  bf16_t* stage = (bf16_t*)smem_raw + wave * 32 * (D + 8);
  store_rows<D>(o, inv, stage, (bf16_t*)a.ctx + (long)b * S * H + h * D, H, qw0, S);
  if (g == 0 && query < S) a.lse[((long)b * a.heads + h) * S + query] = (m_i + __builtin_amdgcn_logf(l_tot)) * kLn2;
}

// =============================================================== backward
// Two passes, by one kernel template: PASS_DQ and PASS_DKV are launched one after the other; with PASS_BOTH the first
// n workgroups own key rows (the longer pass) and the others query rows, side by side.
enum BwdPass { PASS_DQ, PASS_DKV, PASS_BOTH };
// At head size 128 the dQ pass fits two wavefronts per SIMD since its tiles no longer pass through registers, with 12 to 24
// bytes spilled (1 x 2048 x 96 x 128 causal, when this was chosen: backward 570 us with one, 531 with two; 512 now); the
// other pass holds 72 to 81 registers more.
template <int D, bool CAUSAL, int PASS>
__global__ __launch_bounds__(256, (D == 64 || PASS == PASS_DQ) ? 2 : 1) void attn_bwd_mfma_kernel(AttnDesc a, int n) {
  constexpr unsigned TB = TileCopy<D>::BYTES;
  constexpr bool OWN_DELTA = PASS == PASS_BOTH;
  extern __shared__ __attribute__((aligned(256))) unsigned char smem_raw[];
  const unsigned ring = lds_address(smem_raw);      // [2][two tiles]
  FragAddr<D, false> fr;
  fr.init(0);
  // dQ: a wavefront owns 32 queries (lane = query) and streams 64-key tiles.
  if (PASS == PASS_DQ || (PASS == PASS_BOTH && (int)blockIdx.x >= n)) {
    const int wg = PASS == PASS_BOTH ? (int)blockIdx.x - n : (int)blockIdx.x;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int H = a.heads * D, S = a.S;
    int qblk, bh;
    block_of<CAUSAL, true>(wg, (S + 127) / 128, a.B * a.heads, &qblk, &bh);
    const int b = bh / a.heads, h = bh % a.heads;
    const int q0 = qblk * 128, qw0 = q0 + wave * 32;
    const long rs = 3L * H;
    const bf16_t* base = (const bf16_t*)a.qkv + (long)b * S * rs + h * D;
    const bf16_t* dbase = (const bf16_t*)a.dctx + (long)b * S * H + h * D;
    const float scale = rsqrtf((float)D), c = scale * kLog2e;

    bf16x8 qf[D / 16], dof[D / 16];
    load_row_frags<D>(qf, base, rs, qw0, S);
    load_row_frags<D>(dof, dbase, H, qw0, S);
    const int query = qw0 + (lane & 31);
    const long sidx = ((long)b * a.heads + h) * S + min(query, S - 1);
    const float lse2 = a.lse[sidx] * kLog2e;
    // delta[q] = sum over the head's features of ctx * dctx: the two lanes of a query hold the two halves of
    // every 16-feature group of dctx already; the same pieces of ctx are read once.  The dK/dV kernel, where it
    // runs after this one, takes delta from memory.
    float delta = 0.f;
    {
      bf16x8 of[D / 16];
      load_row_frags<D>(of, (const bf16_t*)a.ctx + (long)b * S * H + h * D, H, qw0, S);
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
        for (int j = 0; j < 8; ++j) delta += (float)of[ks][j] * (float)dof[ks][j];
      delta += __shfl_xor(delta, 32, 64);
      if (lane < 32 && query < S) a.delta[sidx] = delta;
    }
    f32x16 dq[D / 32];
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) dq[dt][r] = 0.f;
    // the dP MFMAs start from -delta (a per-lane constant here: a lane owns a query), so their accumulator
    // comes out as dP - delta
    f32x16 neg_delta, zero16;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      neg_delta[r] = -delta;
      zero16[r] = 0.f;
    }

    const int kend = CAUSAL ? min(S, q0 + 128) : S;
    const int nt = (kend + TILE - 1) / TILE;
    TileCopy<D> copy;
    copy.init(rs, S);
    copy.issue(base + H, 0, ring);
    copy.issue(base + 2 * H, 0, ring + TB);
    wait_tiles<0>();
    __syncthreads();
    for (int t = 0; t < nt; ++t) {
      const int slot = t & 1;
      const unsigned at = ring + slot * 2 * TB;
      const int k0 = t * TILE;
      if (t + 1 < nt) {
        copy.issue(base + H, t + 1, ring + (slot ^ 1) * 2 * TB);
        copy.issue(base + 2 * H, t + 1, ring + (slot ^ 1) * 2 * TB + TB);
      }
      if (!CAUSAL || k0 <= qw0 + 31) {
        f32x16 s[2], dp[2];
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            s[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.frag_k(at, 0, u * 32, ks), qf[ks], ks == 0 ? zero16 : s[u], 0, 0, 0);
            dp[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.frag_k(at, TB, u * 32, ks), dof[ks], ks == 0 ? neg_delta : dp[u], 0,
                                                            0, 0);
          }
        const bool need_mask = (k0 + TILE > S) || (CAUSAL && k0 + TILE - 1 > qw0);
        if (need_mask) {                            // uniform over the wavefront
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              float p = __builtin_amdgcn_exp2f(fmaf(s[u][r], c, -lse2));
              const int key = k0 + u * 32 + acc_row(r);
              if (key >= S || (CAUSAL && key > query)) p = 0.f;
              s[u][r] = p * dp[u][r];               // dS^T
            }
        } else {
#pragma unroll
          for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[u][r] = __builtin_amdgcn_exp2f(fmaf(s[u][r], c, -lse2)) * dp[u][r];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const bf16x8 dsb = pack8(s[u >> 1], u & 1);
#pragma unroll
          for (int dt = 0; dt < D / 32; ++dt)
            dq[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.frag_tr(at, 0, dt, 16 * u), dsb, dq[dt], 0, 0, 0);
        }
      }
      wait_tiles<0>();
      __syncthreads();
    }
    bf16_t* stage = (bf16_t*)smem_raw + wave * 32 * (D + 8);
    float* xch = (float*)((bf16_t*)smem_raw + 4 * 32 * (D + 8));     // behind the four staging areas
    if (a.dqkv_colsum != nullptr) {                                  // uniform over the grid
      float cs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      store_rows_sum<D>(dq, scale, stage, (bf16_t*)a.dqkv + (long)b * S * rs + h * D, rs, qw0, S, cs);
      float* part = a.dqkv_colsum + ((long)b * ((S + 127) / 128) + qblk) * rs;
      block_colsum_write<D>(cs, xch, part + h * D);
    } else {
      store_rows<D>(dq, scale, stage, (bf16_t*)a.dqkv + (long)b * S * rs + h * D, rs, qw0, S);
    }
    return;
  }
  if constexpr (PASS != PASS_DQ) {
    // dK, dV: a wavefront owns 32 keys (lane = key) and streams 64-query tiles.
    // OWN_DELTA: delta of the sample's and head's queries is formed here, ahead of the tiles, into LDS behind the rest
    // (S floats), in the order of the additions of the dQ pass; otherwise it comes from memory.
    const int wg = blockIdx.x;
    float* lse_s = (float*)(smem_raw + 4 * TB);     // [2][64]  (log2 domain), behind the tiles
    float* del_s = lse_s + 2 * TILE;                // [2][64]
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 5;
    const int H = a.heads * D, S = a.S;
    int kblk, bh;
    block_of<CAUSAL, false>(wg, (S + 127) / 128, a.B * a.heads, &kblk, &bh);
    const int b = bh / a.heads, h = bh % a.heads;
    const int kb0 = kblk * 128, kw0 = kb0 + wave * 32;
    const long rs = 3L * H;
    const bf16_t* base = (const bf16_t*)a.qkv + (long)b * S * rs + h * D;
    const bf16_t* dbase = (const bf16_t*)a.dctx + (long)b * S * H + h * D;
    const float* lse_g = a.lse + ((long)b * a.heads + h) * S;
    const float* del_g = a.delta + ((long)b * a.heads + h) * S;
    const float scale = rsqrtf((float)D), c = scale * kLog2e;

    bf16x8 kf[D / 16], vf[D / 16];
    load_row_frags<D>(kf, base + H, rs, kw0, S);
    load_row_frags<D>(vf, base + 2 * H, rs, kw0, S);
    const int key = kw0 + (lane & 31);
    f32x16 dk[D / 32], dv[D / 32];
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) { dk[dt][r] = 0.f; dv[dt][r] = 0.f; }

    const int qbeg = CAUSAL ? (kb0 / TILE) * TILE : 0;
    const int nt = (S - qbeg + TILE - 1) / TILE;
    float* own_delta = del_s + 2 * TILE;             // [S]
    if (OWN_DELTA) {
      // two threads a query, as the two lanes of a query share its features in the dQ pass
      const bf16_t* cbase = (const bf16_t*)a.ctx + (long)b * S * H + h * D + (threadIdx.x & 1) * 8;
      const bf16_t* gbase = dbase + (threadIdx.x & 1) * 8;
      for (int q = qbeg + (threadIdx.x >> 1); q - (int)(threadIdx.x >> 1) < S; q += 128) {
        const long row = (long)min(q, S - 1) * H;
        bf16x8 of[D / 16], gf[D / 16];
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
          of[ks] = *(const bf16x8*)(cbase + row + ks * 16);
          gf[ks] = *(const bf16x8*)(gbase + row + ks * 16);
        }
        float d = 0.f;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
          for (int j = 0; j < 8; ++j) d += (float)of[ks][j] * (float)gf[ks][j];
        d += __shfl_xor(d, 1, 64);
        if ((threadIdx.x & 1) == 0 && q < S) own_delta[q] = d;
      }
      __syncthreads();
    }
    float lse_r = 0.f, del_r = 0.f;
    auto fetch_stats = [&](int q0t) {
      if (threadIdx.x < TILE) {
        const int q = q0t + threadIdx.x;
        lse_r = q < S ? lse_g[q] * kLog2e : 0.f;
        if (OWN_DELTA) del_r = q < S ? -own_delta[q] : 0.f;
        else del_r = q < S ? -del_g[q] : 0.f;        // negated: the dP accumulators start from it
      }
    };
    auto stash_stats = [&](int buf) {
      if (threadIdx.x < TILE) {
        lse_s[buf * TILE + threadIdx.x] = lse_r;
        del_s[buf * TILE + threadIdx.x] = del_r;
      }
    };
    TileCopy<D> copy_q, copy_do;
    copy_q.init(rs, S);
    copy_do.init(H, S);
    copy_q.issue(base, qbeg / TILE, ring);
    copy_do.issue(dbase, qbeg / TILE, ring + TB);
    fetch_stats(qbeg);
    stash_stats(0);
    wait_tiles<0>();
    __syncthreads();
    for (int t = 0; t < nt; ++t) {
      const int buf = t & 1;
      const unsigned at = ring + buf * 2 * TB;
      const int q0t = qbeg + t * TILE;
      if (t + 1 < nt) {
        fetch_stats(q0t + TILE);
        copy_q.issue(base, qbeg / TILE + t + 1, ring + (buf ^ 1) * 2 * TB);
        copy_do.issue(dbase, qbeg / TILE + t + 1, ring + (buf ^ 1) * 2 * TB + TB);
      }
      if (!CAUSAL || q0t + TILE - 1 >= kw0) {       // wave-uniform: some query at or after the wave's first key
        // the queries' -delta runs along the accumulator registers here and comes from LDS with the tile: the
        // dP accumulators start from it and come out as dP - delta
        f32x16 s[2], dp[2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int a4 = 0; a4 < 4; ++a4) {
            const f32x4 d4 = *(const f32x4*)(del_s + buf * TILE + u * 32 + 8 * a4 + 4 * g);
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) dp[u][4 * a4 + cc] = d4[cc];
          }
        const f32x16 zero16 = {};
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            s[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.frag_k(at, 0, u * 32, ks), kf[ks], ks == 0 ? zero16 : s[u], 0, 0, 0);
            dp[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.frag_k(at, TB, u * 32, ks), vf[ks], dp[u], 0, 0, 0);
          }
        const bool need_mask = (q0t + TILE > S) || (kw0 + 32 > S) || (CAUSAL && q0t < kw0 + 31);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int a4 = 0; a4 < 4; ++a4) {
            const int row = u * 32 + 8 * a4 + 4 * g;   // first of 4 consecutive query rows of this lane
            const f32x4 l4 = *(const f32x4*)(lse_s + buf * TILE + row);
            if (need_mask) {                        // uniform over the wavefront
#pragma unroll
              for (int cc = 0; cc < 4; ++cc) {
                const int r = 4 * a4 + cc;
                float p = __builtin_amdgcn_exp2f(fmaf(s[u][r], c, -l4[cc]));
                const int query = q0t + row + cc;
                if (query >= S || key >= S || (CAUSAL && key > query)) p = 0.f;
                s[u][r] = p;
                dp[u][r] *= p;                      // dS
              }
            } else {
#pragma unroll
              for (int cc = 0; cc < 4; ++cc) {
                const int r = 4 * a4 + cc;
                const float p = __builtin_amdgcn_exp2f(fmaf(s[u][r], c, -l4[cc]));
                s[u][r] = p;
                dp[u][r] *= p;                      // dS
              }
            }
          }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const bf16x8 pb = pack8(s[u >> 1], u & 1);
          const bf16x8 dsb = pack8(dp[u >> 1], u & 1);
#pragma unroll
          for (int dt = 0; dt < D / 32; ++dt) {
            dv[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.frag_tr(at, TB, dt, 16 * u), pb, dv[dt], 0, 0, 0);
            dk[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.frag_tr(at, 0, dt, 16 * u), dsb, dk[dt], 0, 0, 0);
          }
        }
      }
      if (t + 1 < nt) stash_stats(buf ^ 1);
      wait_tiles<0>();
      __syncthreads();
    }
    bf16_t* stage = (bf16_t*)smem_raw + wave * 32 * (D + 8);
    bf16_t* out = (bf16_t*)a.dqkv + (long)b * S * rs + h * D;
    float* xch = (float*)((bf16_t*)smem_raw + 4 * 32 * (D + 8));     // behind the four staging areas
    if (a.dqkv_colsum != nullptr) {                                  // uniform over the grid
      float* part = a.dqkv_colsum + ((long)b * ((S + 127) / 128) + kblk) * rs;
      float cs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      store_rows_sum<D>(dk, scale, stage, out + H, rs, kw0, S, cs);
      block_colsum_write<D>(cs, xch, part + H + h * D);
      float cv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      store_rows_sum<D>(dv, 1.f, stage, out + 2 * H, rs, kw0, S, cv);
      block_colsum_write<D>(cv, xch, part + 2 * H + h * D);
    } else {
      store_rows<D>(dk, scale, stage, out + H, rs, kw0, S);
      store_rows<D>(dv, 1.f, stage, out + 2 * H, rs, kw0, S);
    }
  }
}

// ------------------------------------------------------------------ launchers
static bool covered(const AttnDesc& a) {
  if (a.d != 64 && a.d != 128) return false;
  // 32-bit byte offsets inside one sequence, the rows of a last, partial tile included (they are clamped after the add)
  if ((long)(a.S + TILE) * 3 * a.heads * a.d * 2 >= (1L << 32)) return false;
  auto misaligned = [](const void* p) { return p != nullptr && ((uintptr_t)p & 15) != 0; };
  return !(misaligned(a.qkv) || misaligned(a.ctx) || misaligned(a.dctx) || misaligned(a.dqkv));
}

template <int D, bool CAUSAL, bool REGS>
static hipError_t fwd_launch_form(hipStream_t s, const AttnDesc& a, unsigned grid) {
  constexpr int BYTES = 2 * 2 * TileCopy<D>::BYTES;
  static_assert(BYTES >= 4 * 32 * (D + 8) * 2, "the four staging areas");
  constexpr auto kern = attn_fwd_mfma_kernel<D, CAUSAL, REGS>;
  const hipError_t e = ensure_lds_attribute<kern, BYTES>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), BYTES, s, a);
  return hipGetLastError();
}
// Tiles go straight to LDS, or through registers where that is the faster way.  Loads to LDS that miss the chiplet's 4 MB of
// L2 return later (428 clocks a request on average against 353, with the same misses, at 1 x 1536 x 20 x 128 causal), and
// workgroups of different lengths, alone on their SIMDs at the end, wait for them.  Workgroup i runs on chiplet i mod 8 and
// reads the keys and values of pair i mod (samples x heads): `met` bytes in all.  So with a causal mask, at head size 64:
// registers beyond 1.75 MB, except for half a workgroup per CU or less, and where many row blocks of a pair meet on a chiplet
// and share what is fetched and later workgroups fill the gaps.  At head size 128 a CU holds two workgroups and the lines lie where both were measured to meet:
// straight to LDS up to half a workgroup per CU and from a round and a half on; short sequences, with few steps to wait in,
// through registers.  Without a mask hardly ever.  Forward in us: before (padded rows, through registers) / straight to
// LDS / through registers, the form chosen marked *:
//   8 x 512 x 16 x 64          15.3 / 14.1* / 15.6      1 x 4096 x 20 x 64 causal   69.2 / 72.7 / 66.4*
//   3 x 333 x 16 x 64           8.7 /  7.7* /  8.4      2 x 2048 x 25 x 64 causal   42.4 / 43.3 / 41.7*
//   4 x 1024 x 25 x 64         47.0 / 42.4* / 45.5      4 x 1024 x 25 x 64 causal   26.4 / 25.7 / 25.1*
//   1 x 2048 x 16 x 64 causal  31.9 / 30.6* / 31.2      1 x 3072 x 10 x 64 causal   45.8 / 52.7 / 44.8*
//   2 x 4096 x 16 x 64 causal  92.2 / 85.2* / 90.2      4 x 2048 x 5 x 64 causal: 1.08 / 0.97* of before
//   1 x 2048 x 96 x 128         226 /  212* /  223      1 x 1536 x 20 x 128         36.1 / 36.9 / 36.1*
//   1 x 4096 x 4 x 128 causal  86.0 / 83.5* / 85.8      1 x 1500 x 20 x 128 causal  36.1 / 40.9 / 36.1*
//   1 x 8192 x 16 x 128 causal  302 /  265* /  300      1 x 8192 x 4 x 128 causal    168 /  195 /  166*
//   3 x 2048 x 20 x 128 causal 85.0 / 78.6* / 84.4      48 x 256 x 12 x 128 causal  33.2 / 35.3 / 33.1*
// Over 187 shapes 0.946 of the time before (at most 1.02) and 0.941 of that of a ring of three straight to LDS in every launch
// at head size 64 and up to 256 workgroups at 128.
template <int D, bool CAUSAL>
static hipError_t fwd_launch(hipStream_t s, const AttnDesc& a) {
  const unsigned grid = (unsigned)(((a.S + 127) / 128) * a.B * a.heads);
  const int pairs = a.B * a.heads, shared = pairs % 8 == 0 ? 8 : pairs % 4 == 0 ? 4 : pairs % 2 == 0 ? 2 : 1;
  const double met = (double)(pairs / shared) * a.S * D * 4;
  const int blocks = (a.S + 127) / 128;
  bool regs;
  if (D == 64) regs = CAUSAL && a.S > 256 && grid > 128 && met > 1.75e6 && (grid < 1000 || blocks * shared < 128);
  else if (CAUSAL) regs = grid > 128 && (a.S <= 680 || grid < (a.S > 2048 ? 800u : 768u));
  else regs = met > 3e6 && (a.S > 1024 ? grid <= 256 : a.S <= 300 && grid > 512);
  return regs ? fwd_launch_form<D, CAUSAL, true>(s, a, grid) : fwd_launch_form<D, CAUSAL, false>(s, a, grid);
}

// Both backward passes as one launch: the second need not wait for the first, whose last workgroups leave most CUs idle, and
// a launch is saved; it costs the key owners their own delta.  With a causal mask the passes' workgroups differ in length
// and fill each other's gaps, so it pays to more workgroups.  The chip holds 512 at head size 64 and 256 at 128, where the
// kernel of both passes leaves room for one wavefront per SIMD and the dQ pass by itself for two.  The limits are where
// the two were measured to meet.  Backward in us, two launches / one (samples x tokens x heads, workgroups of both passes):
//   head size 64                                            causal
//   1 x 1024 x 4   (64)    43.0 / 31.7   6 x 512 x 16 (768)  36.6 / 34.5    4 x 512 x 16 (512)   29.8 / 22.5
//   4 x 512 x 16  (512)    27.1 / 22.8   7 x 512 x 16 (896)  43.5 / 44.0    8 x 512 x 16 (1024)  37.0 / 33.8
//   5 x 512 x 16  (640)    36.0 / 29.3   8 x 512 x 16 (1024) 43.4 / 46.7   12 x 512 x 16 (1536)  54.3 / 51.1
//   3 x 1024 x 16 (768)    61.0 / 59.7   9 x 512 x 16 (1152) 61.9 / 52.5   16 x 512 x 16 (2048)  69.3 / 70.7
//   head size 128
//   1 x 1024 x 8  (128)    81.7 / 60.3   1 x 1024 x 22 (352) 88.1 / 98.5    1 x 1024 x 32 (512)  87.6 / 66.6
//   2 x 512 x 20  (320)    49.4 / 41.5   2 x 512 x 24 (384)  50.2 / 53.0    8 x 256 x 16 (512)   37.1 / 33.5
//   5 x 256 x 16  (320)    31.6 / 26.8   1 x 1024 x 32 (512) 88.5 / 98.4    3 x 1024 x 16 (768)  94.3 / 101
// Up to two row blocks a sequence the causal workgroups hardly differ: 16 x 256 x 16 x 64 (1024) 27.6 / 29.4.
// Longer sequences keep two launches: the deltas of a sequence are held in LDS, 4 KB of it here (few heads of more
// tokens were not measured).
constexpr int kBothMaxSeq = 1024;
template <int D, bool CAUSAL>
static bool side_by_side(const AttnDesc& a, unsigned wgs) {
  const unsigned most = D == 64 ? (CAUSAL && a.S > 256 ? 1536u : 768u) : (CAUSAL ? 512u : 320u);
  return a.S <= kBothMaxSeq && 2 * wgs <= most;
}

template <int D, bool CAUSAL>
static hipError_t bwd_launch(hipStream_t s, const AttnDesc& a) {
  constexpr int BYTES_DQ = 4 * TileCopy<D>::BYTES;
  constexpr int BYTES_DKV = 4 * TileCopy<D>::BYTES + 4 * TILE * 4;
  static_assert(BYTES_DQ >= 4 * 32 * (D + 8) * 2 + 4 * D * 4, "the four staging areas and the column sums behind them");
  constexpr auto kq = attn_bwd_mfma_kernel<D, CAUSAL, PASS_DQ>;
  constexpr auto kkv = attn_bwd_mfma_kernel<D, CAUSAL, PASS_DKV>;
  hipError_t e = ensure_lds_attribute<kq, BYTES_DQ>();
  if (e == hipSuccess) e = ensure_lds_attribute<kkv, BYTES_DKV>();
  if (e != hipSuccess) return e;
  dim3 grid(((a.S + 127) / 128) * a.B * a.heads);
  if (side_by_side<D, CAUSAL>(a, grid.x)) {
    constexpr int BYTES_BOTH = BYTES_DKV + kBothMaxSeq * 4;
    constexpr auto kboth = attn_bwd_mfma_kernel<D, CAUSAL, PASS_BOTH>;
    e = ensure_lds_attribute<kboth, BYTES_BOTH>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kboth, dim3(2 * grid.x), dim3(256), BYTES_DKV + a.S * 4, s, a, (int)grid.x);
    if (a.dqkv_colsum != nullptr && a.dqkv_colsum_parts != nullptr) *a.dqkv_colsum_parts = a.B * ((a.S + 127) / 128);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(kq, grid, dim3(256), BYTES_DQ, s, a, 0);
  hipLaunchKernelGGL(kkv, grid, dim3(256), BYTES_DKV, s, a, 0);
  if (a.dqkv_colsum != nullptr && a.dqkv_colsum_parts != nullptr) *a.dqkv_colsum_parts = a.B * ((a.S + 127) / 128);
  return hipGetLastError();
}

hipError_t launch_attention_fwd_mfma(hipStream_t s, const AttnDesc& a) {
  if (!covered(a)) return hipErrorNotSupported;
  if (a.d == 64) return a.causal ? fwd_launch<64, true>(s, a) : fwd_launch<64, false>(s, a);
  return a.causal ? fwd_launch<128, true>(s, a) : fwd_launch<128, false>(s, a);
}

hipError_t launch_attention_bwd_mfma(hipStream_t s, const AttnDesc& a) {
  if (!covered(a)) return hipErrorNotSupported;
  if (a.d == 64) return a.causal ? bwd_launch<64, true>(s, a) : bwd_launch<64, false>(s, a);
  return a.causal ? bwd_launch<128, true>(s, a) : bwd_launch<128, false>(s, a);
}

}  // namespace bamboo
