// fp16 x fp16 -> fp32 GEMM on the gfx950 matrix cores, C[M,N] = A[M,K] . W[N,K]^T, with the
// epilogues the decoder needs fused in.  (Weights are the caller's bf16 values held in fp16, which
// represents them exactly; activations are fp16, whose 11 significant bits keep the logits within
// the parity bound where bf16 activations do not.)  Both operands are K-block major (see kblk_off), so a
// block's tile is one contiguous run in memory and every MFMA operand fragment is one 16-byte LDS read.
// A block of WM x WN waves owns a BM x BN tile; each wave a (BM/WM) x (BN/WN) sub-tile built from 16x16x32
// MFMAs.  A and W tiles of depth 64 go from global memory straight into LDS (16-byte chunks, XOR-swizzled by
// row so that fragment reads spread over all banks).  Three main loops share the epilogues and the matrix instruction,
// which walks K front to back in all of them: gemm_f16_kernel (two stages, one barrier per K step; a K that is not a
// multiple of 64 takes its older path through registers, which can zero-fill the tail), gemm_big_kernel (256x256 on four
// waves, for launches that fill the chip) and gemm_ring_kernel (a ring of stages, for launches that do not).
#include "kernels.h"
#include <algorithm>
#include <type_traits>

namespace {

constexpr int BK = 64;            // fp16 elements of K per LDS stage (128 bytes per row)
#ifndef SWZ_SHIFT
#define SWZ_SHIFT 1
#endif
// LDS rows are 8 chunks of 16 bytes; chunk c of row r is stored at chunk position c ^ swz(r).  The LDS of
// gfx950 has 64 banks of 4 bytes: 16 lanes of a 128-bit read are served per cycle, and rows r, r + 1 sit in
// opposite halves of the banks, so the swizzle steps every second row (measured: SQ_LDS_BANK_CONFLICT = 0).
__device__ __forceinline__ int swz(int r) { return (r >> SWZ_SHIFT) & 7; }

// Blocks are handed to the 8 XCDs round-robin by the hardware.  Renumber them so that each XCD
// (one L2) works on a contiguous range of logical tile ids, then walk tiles M-fastest inside groups
// of 8 M-tiles: the blocks that share a weight tile run on the same L2 at the same time.
// With split-K the `splits` blocks of one tile are neighbours in that order.
__device__ __forceinline__ void tile_of_block(int tiles_m, int tiles_n, int splits, int& tm, int& tn, int& split) {
  const int nb = gridDim.x, bid = blockIdx.x;
  const int per = (nb + 7) >> 3;
  const int full = (nb & 7) == 0 ? 8 : (nb & 7);
  const int xcd = bid & 7, slot = bid >> 3;
  int logical = xcd < full ? xcd * per + slot : full * per + (xcd - full) * (per - 1) + slot;
  split = logical % splits;
  logical /= splits;
  constexpr int GROUP_M = 8;
  const int per_group = GROUP_M * tiles_n;
  const int group = logical / per_group;
  const int first_m = group * GROUP_M;
  const int gsz = min(tiles_m - first_m, GROUP_M);
  const int in_group = logical - group * per_group;
  tm = first_m + in_group % gsz;
  tn = in_group / gsz;
}

// gelu(v) = v/2 (1 + erf(v / sqrt 2)) = v/2 + |v|/2 erf(|v| / sqrt 2), with erf by the rational-exponential form of Abramowitz &
// Stegun 7.1.26 (absolute error < 1.5e-7, far below the 16-bit rounding of the result).  The epilogue of the widest layer is
// bound by this arithmetic: 17 instructions and two transcendentals a value, sqrt 2 and log2 e folded into the constants, the
// hardware's reciprocal (1 ulp) corrected once.  Against 64 bits on [-4, 4] at most 3.8e-7 off, and 1.2e-7 in the mean square.
__device__ __forceinline__ float gelu_erf(float v) {
  const float b = fmaf(0.3275911f * 0.70710678118654752f, fabsf(v), 1.0f);
  const float t0 = __builtin_amdgcn_rcpf(b), t = fmaf(fmaf(-b, t0, 1.0f), t0, t0);
  const float poly = t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
  const float z = v * 0.84932180028801907f;                   // sqrt(log2(e) / 2) v
  const float r = fmaf(-poly, __builtin_amdgcn_exp2f(-z * z), 1.0f);
  const float h = 0.5f * v;
  return fmaf(fabsf(h), r, h);
}
// v / (1 + exp(-v)), the division by a reciprocal with its residual folded back in; an eighth of both keeps the reciprocal in
// fp32's normal range, and the fix-up sets what the residual cannot (infinite operands).  The values are those of a true division
// (four million random arguments on [-90, 90]): at most 3.5e-7 from 64 bits on [-4, 4], where the bare reciprocal is up to 4.9e-7
// off.  Over that one it costs 0.5 % of a generate call at the 8B shape, the true division 0.8 %.
__device__ __forceinline__ float silu(float v) {
  const float w = 0.125f * v, b = fmaf(__expf(-v), 0.125f, 0.125f);
  const float y = __builtin_amdgcn_rcpf(b), q = w * y;
  return __builtin_amdgcn_div_fixupf(fmaf(fmaf(-q, b, w), y, q), b, w);
}
// v / t for one divisor t >= 2^-60 and its reciprocal: the quotient with its residual folded back in (equal to v / t on a million
// random pairs; 3 instructions where a division takes 11).  An infinite quotient would turn into NaN there; INF: kept below
// infinity until the residual is added, which then restores it.
template <bool INF>
__device__ __forceinline__ float div_by(float v, float t, float inv_t) {
  const float q = INF ? __builtin_amdgcn_fmed3f(v * inv_t, -3.402823466e38f, 3.402823466e38f) : v * inv_t;
  return fmaf(fmaf(-q, t, v), inv_t, q);
}
// Temperatures below are divided by as they stand, in kernels of their own (EPI_LMHEAD_EXACT).  Above, the logits of the default
// formats (at most 65504^2 x 8192 < 2^46) have finite quotients; those of precise mode, whose operands have fp32's range, may
// overflow (a test of every value costs the default formats 3 % of the sampling stage: 64 rows at 2.8B width 75.6 -> 78.1 us).
constexpr float MIN_FAST_TEMPERATURE = 0x1p-60f;

template <int N>
__device__ __forceinline__ void wait_loads_then_barrier() {
  // all but the N most recent vector-memory loads of this wave have landed; then every wave of the block is here
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
}

// nothing may be scheduled across this point
#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// What becomes of a wave's accumulators.  The products were issued as W_tile . A_tile^T, so acc[i][j][r] is C[m][n] with
// m = 16 i + lane % 16 and n = 16 j + 4 (lane / 16) + r: every lane holds runs of four consecutive columns of one row,
// which makes outputs, bias and residual 16-byte accesses and turns the row-wise softmax statistics of the LM head into
// in-register reductions.  (wrow0, wcol0): the wave's first row and column.  FULL: every row and column of the wave exists
// and rows start on 16-byte boundaries, so that no access needs a condition of its own (a wave that runs alone on its SIMD
// waits out every branch: the epilogue of a whole 256x256 tile is a third shorter without them).  STAGED: a QKV projection
// of the prompt pass only (the kernel has no code for a decode step's cache writes).
template <int TM, int TN, int EPI, bool PR, bool FULL, bool STAGED>
__device__ __forceinline__ void gemm_epilogue_as(const GemmArgs& g, const f32x4 (&acc)[TM][TN], int wrow0, int wcol0, int lane, int split) {
  const int frow = lane & 15, fq = lane >> 4;
  if constexpr (EPI == EPI_LMHEAD || EPI == EPI_LMHEAD_EXACT) {
    // per row and per 64-column group: max and sum of exp of the tempered logits; optional capture
    // of the target column's tempered logit.  Nothing of size [M, N] is written.
    static_assert(TN % 4 == 0, "a wave must own whole 64-column groups");
    const int ngroups = (g.N + 63) >> 6;
    constexpr bool EXACT = EPI == EPI_LMHEAD_EXACT;
    constexpr bool INF = EXACT || PR || !FULL;           // logits, and then whole groups of them, may be -inf
    const float inv_t = 1.0f / g.temperature;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = wrow0 + i * 16 + frow;
      const int tgt = (g.target != nullptr && (FULL || row < g.M)) ? g.target[row] : -1;
#pragma unroll
      for (int gi = 0; gi < TN / 4; ++gi) {
        const int group = (wcol0 >> 6) + gi;
        float l[16];
        float mx = -INFINITY;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int col = wcol0 + (4 * gi + jj) * 16 + 4 * fq + r;
            const float a = acc[i][4 * gi + jj][r];
            const float v = !FULL && col >= g.N ? -INFINITY : EXACT ? a / g.temperature : div_by<PR>(a, g.temperature, inv_t);
            l[jj * 4 + r] = v;
            mx = fmaxf(mx, v);
            if (col == tgt) g.target_logit[row] = v;
          }
        mx = fmaxf(mx, __shfl_xor(mx, 16, WAVE));
        mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) sum += (INF && l[e] == -INFINITY) ? 0.f : __expf(l[e] - mx);
        sum += __shfl_xor(sum, 16, WAVE);
        sum += __shfl_xor(sum, 32, WAVE);
        if (fq == 0 && (FULL || (row < g.M && group < ngroups))) g.partial[(size_t)row * ngroups + group] = make_float2(mx, sum);
      }
    }
  } else if constexpr (EPI == EPI_QKV) {
    // What depends on the row (angles, place in the cache) is found before anything is stored, what depends on the column
    // (head, rotary pair, destination) once per column tile, and the next tile's bias and angles are requested in front of
    // this one's stores: loads and stores return in order, so that a load behind a store waits for the store (a 256x256 tile
    // of the prompt pass on four waves: 53 us with, 18 us without such waits).  A column tile of which no column is rotated
    // is stored in 8-byte pieces.
    const QkvEpi& e = g.qe;
    [[maybe_unused]] bool sat = false;
    const bool staged = STAGED || e.kvstage != nullptr;
    auto live = [&](int i) { return FULL || wrow0 + i * 16 + frow < g.M; };
    uint32_t rope[TM];       // byte offset of the row's angles: at most 2^20 positions of 128 pairs
    // a row's place in the cache: its stream's super-block, and the key's row and place in the two kinds of value units
    [[maybe_unused]] long long kv_at[STAGED ? 1 : TM];
    [[maybe_unused]] int per_head[STAGED ? 1 : TM];                              // elements between kv heads
    [[maybe_unused]] int slot[STAGED ? 1 : TM];
    {
      int pos[TM];
      [[maybe_unused]] int seq[TM], sub[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = FULL ? wrow0 + i * 16 + frow : min(wrow0 + i * 16 + frow, g.M - 1);
        pos[i] = e.pos[row] + e.pos_add;
        if (!staged) {
          seq[i] = e.dst_seq[row];
          sub[i] = e.slot_sub ? e.slot_sub[row] : 0;
        }
      }
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        rope[i] = (uint32_t)pos[i] * (uint32_t)(e.r >> 1) * 8u;
        if constexpr (!STAGED) {
          if (!staged) {
            const long long base = e.lay.seq_base(e.kv_off[seq[i]]);
            per_head[i] = 2 * e.kv_cap[seq[i]] * e.h;
            slot[i] = (pos[i] - sub[i]) & 31;
            kv_at[i] = base + (long long)((pos[i] - sub[i]) >> 5) * 64 * e.h;
          }
        }
      }
    }
    struct Col { int head, p0; bool isq, rot; };
    auto column = [&](int j) {
      Col c;
      const int col = FULL ? wcol0 + j * 16 + 4 * fq : min(wcol0 + j * 16 + 4 * fq, g.N - 4);
      c.head = (int)(((float)col + 0.5f) * e.inv_h);
      c.p0 = col - c.head * e.h;
      c.isq = c.head < e.Hq;
      c.rot = c.head < e.Hq + e.Hkv && c.p0 < e.r;
      return c;
    };
    f32x4 bias_n = f32x4{0.f, 0.f, 0.f, 0.f}, cs_n[TM];
    auto fetch = [&](int j) {
      const Col c = column(j);
      if (g.bias) bias_n = *(const f32x4*)(g.bias + (c.head * e.h + c.p0));
      if (__ballot(c.rot) != 0) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          cs_n[i] = f32x4{1.f, 0.f, 1.f, 0.f};
          if (c.rot) cs_n[i] = *(const f32x4*)((const char*)e.table + (rope[i] + (uint32_t)(c.p0 >> 1) * 8u));
        }
      }
    };
    fetch(0);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const Col c = column(j);
      const bool in_n = FULL || wcol0 + j * 16 + 4 * fq < g.N;
      const bool any_rot = __ballot(c.rot) != 0;
      // head dims of the lane's four columns: a rotary group holds the pairs (d0, d0 + r/2) and (d0 + 1, d0 + 1 + r/2) as
      // (v0, v2) and (v1, v3); any other group holds four consecutive dims.  d0, d1: dims of (v0, v1) and of (v2, v3)
      const int d0 = c.rot ? c.p0 >> 1 : c.p0, d1 = c.rot ? d0 + (e.r >> 1) : c.p0 + 2;
      f32x4 v[TM];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        v[i] = acc[i][j] + bias_n;
        if (any_rot) {
          const f32x4 cs = cs_n[i];
          // (as fmaf: left to the compiler, which of the two products is rounded first could differ between tile shapes)
          const float lo0 = fmaf(v[i][0], cs[0], -(v[i][2] * cs[1])), hi0 = fmaf(v[i][2], cs[0], v[i][0] * cs[1]);
          const float lo1 = fmaf(v[i][1], cs[2], -(v[i][3] * cs[3])), hi1 = fmaf(v[i][3], cs[2], v[i][1] * cs[3]);
          v[i][0] = lo0; v[i][1] = lo1; v[i][2] = hi0; v[i][3] = hi1;
        }
      }
      if (j + 1 < TN) fetch(j + 1);
      SCHED_FENCE();
      // 16-bit outputs in rows: q, or staged k | v (precise: q rows are fp32, addressed apart)
      const int ld = c.isq ? e.Hq * e.h : 2 * e.Hkv * e.h;
      uint16_t* out = (c.isq ? e.q : e.kvstage) + (size_t)(wrow0 + frow) * ld + (c.isq ? c.head : c.head - e.Hq) * e.h;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        if (!live(i) || !in_n) continue;
        uint16_t* p = out + (size_t)i * 16 * ld;
        uint32_t w01, w23;
        [[maybe_unused]] u32x2 wl;
        if constexpr (PR) {
          SPLIT_BF16X2(v[i][0], v[i][1], w01, wl[0]);
          SPLIT_BF16X2(v[i][2], v[i][3], w23, wl[1]);
          if (c.isq) {
            float* qp = (float*)e.q + (size_t)(wrow0 + i * 16 + frow) * ld + c.head * e.h;
            *(float2*)(qp + d0) = make_float2(v[i][0], v[i][1]);
            *(float2*)(qp + d1) = make_float2(v[i][2], v[i][3]);
            continue;
          }
        } else {
          // q is fp16; cached keys and values are bf16 but enter the attention products as fp16
#pragma unroll
          for (int r = 0; r < 4; ++r) sat |= f16_out_of_range(v[i][r]);
          w01 = c.isq ? pack_f16x2(v[i][0], v[i][1]) : pack_bf16x2(v[i][0], v[i][1]);
          w23 = c.isq ? pack_f16x2(v[i][2], v[i][3]) : pack_bf16x2(v[i][2], v[i][3]);
        }
        if (staged || c.isq) {
          if constexpr (PR) {
            *(uint32_t*)(p + e.stage_lo_off + d0) = wl[0];
            *(uint32_t*)(p + e.stage_lo_off + d1) = wl[1];
          }
          if (any_rot) {
            *(uint32_t*)(p + d0) = w01;
            *(uint32_t*)(p + d1) = w23;
          } else {
            u32x2 w;
            w[0] = w01; w[1] = w23;
            *(u32x2*)(p + d0) = w;
          }
        } else if constexpr (!STAGED) {
          uint16_t* st = e.kv + kv_at[i];
          if (c.head < e.Hq + e.Hkv) {
            st += (long long)(c.head - e.Hq) * per_head[i] + ((slot[i] >> 2) & 1) * 16 * e.h;
            const int r = e.lay.k_row(slot[i]);
            uint16_t* s0 = st + e.lay.k_dim(d0) + r * e.lay.k_width(d0);
            uint16_t* s1 = st + e.lay.k_dim(d1) + r * e.lay.k_width(d1);
            if (any_rot) {
              *(uint32_t*)s0 = w01;
              *(uint32_t*)s1 = w23;
              if constexpr (PR) {
                *(uint32_t*)(s0 + e.kv_lo_off) = wl[0];
                *(uint32_t*)(s1 + e.kv_lo_off) = wl[1];
              }
            } else {
              *(u32x2*)s0 = u32x2{w01, w23};
              if constexpr (PR) *(u32x2*)(s0 + e.kv_lo_off) = wl;
            }
          } else {
            st += (long long)(c.head - e.Hq - e.Hkv) * per_head[i];
            if (e.lay.v_grouped(c.p0)) {
              st += e.lay.v_key_grouped(slot[i]) + e.lay.v_dim_grouped(c.p0);
              *(u32x2*)st = u32x2{w01, w23};
              if constexpr (PR) *(u32x2*)(st + e.kv_lo_off) = wl;
            } else {
              st += e.lay.v_key_rest(slot[i]) + e.lay.v_dim_rest(c.p0);
              st[0] = (uint16_t)w01; st[8] = (uint16_t)(w01 >> 16); st[16] = (uint16_t)w23; st[24] = (uint16_t)(w23 >> 16);
              if constexpr (PR) {
                st += e.kv_lo_off;
                st[0] = (uint16_t)wl[0]; st[8] = (uint16_t)(wl[0] >> 16); st[16] = (uint16_t)wl[1]; st[24] = (uint16_t)(wl[1] >> 16);
              }
            }
          }
        }
      }
      SCHED_FENCE();
    }
    if constexpr (!PR) flag_f16_range(sat, g.status);
  } else {
    // The place of (i, j) is a distance common to the wave plus one 32-bit distance of the lane: a scalar base and one
    // register address every access (the rows of plain fp32 outputs are as long as a vocabulary: 64 bits there).  Column
    // tiles outside, so that a bias is read once.
    [[maybe_unused]] bool sat = false;
    constexpr bool F32OUT = EPI == EPI_F32 || EPI == EPI_RESID || EPI == EPI_PARTIAL;
    const int ld = EPI == EPI_PARTIAL ? g.N : g.ldo;
    using lane_t = std::conditional_t<EPI == EPI_F32, size_t, uint32_t>;
    const lane_t lane_off = F32OUT ? ((lane_t)frow * ld + 4 * fq) * 4 : (lane_t)(frow * 64 + 4 * fq) * 2;
    auto place = [&](int i, int j) -> char* {
      const size_t row = wrow0 + i * 16;
      // first output column of the tile (SwiGLU: weight rows come in blocks of 32, gates and then the matching ups)
      const int col = EPI == EPI_SWIGLU_F16 ? (wcol0 >> 1) + (j >> 2) * 32 + (j & 1) * 16 : wcol0 + j * 16;
      if constexpr (EPI == EPI_PARTIAL) return (char*)(g.ws + ((size_t)split * g.M + row) * g.N + col);
      else if constexpr (F32OUT) return (char*)((float*)g.out + row * g.ldo + col);
      else return (char*)((uint16_t*)g.out + ((size_t)(col >> 6) * g.M + row) * 64 + (col & 63));
    };
    auto live = [&](int i) { return FULL || wrow0 + i * 16 + frow < g.M; };
    // only plain fp32 outputs (logits of any vocabulary) have widths or rows that break up the groups of four
    auto whole = [&](int j) { return FULL || EPI != EPI_F32 || (wcol0 + j * 16 + 4 * fq + 3 < g.N && (ld & 3) == 0); };
    // Bias and residual travel one column tile ahead, in front of the stores: loads and stores return in order, so that a
    // load behind a store waits for the store, and with one wave per SIMD nothing else covers that.
    [[maybe_unused]] f32x4 old[TM];
    f32x4 bias_n = f32x4{0.f, 0.f, 0.f, 0.f};
    auto fetch = [&](int j) {
      const int col4 = wcol0 + j * 16 + 4 * fq;
      if (!FULL && col4 >= g.N) return;
      if (EPI != EPI_PARTIAL && g.bias) {
        if (whole(j)) bias_n = *(const f32x4*)((const char*)(g.bias + wcol0 + j * 16) + (uint32_t)(fq * 16));
        else
          for (int r = 0; r < 4; ++r) bias_n[r] = col4 + r < g.N ? g.bias[col4 + r] : 0.f;
      }
      if constexpr (EPI == EPI_RESID) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
          if (live(i)) old[i] = *(const f32x4*)(place(i, j) + lane_off);
      }
    };
    fetch(0);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if (EPI == EPI_SWIGLU_F16 && (j & 2)) continue;       // the ups, taken along with their gates
      const int col4 = wcol0 + j * 16 + 4 * fq;             // first of the lane's four columns
      if (!FULL && col4 >= g.N) continue;
      const bool four = whole(j);
      const f32x4 bias = bias_n;
      auto at = [&](int i) -> char* { return place(i, j); };
      f32x4 v[TM];
      if constexpr (EPI == EPI_RESID) {
#pragma unroll
        for (int i = 0; i < TM; ++i) v[i] = old[i];
      }
      // column tile whose turn is next (SwiGLU: gates only, 0, 1, 4, 5, ...)
      const int jn = EPI == EPI_SWIGLU_F16 && (j & 1) ? j + 3 : j + 1;
      if (jn < TN) fetch(jn);
      SCHED_FENCE();
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        if (!live(i)) continue;
        if constexpr (EPI == EPI_PARTIAL) v[i] = acc[i][j];
        else if constexpr (EPI == EPI_F32) v[i] = acc[i][j] + bias;
        else if constexpr (EPI == EPI_RESID) v[i] += acc[i][j] + bias;
        else {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if constexpr (EPI == EPI_GELU_F16) v[i][r] = gelu_erf(acc[i][j][r] + bias[r]);
            else v[i][r] = silu(acc[i][j][r] + bias[r]) * acc[i][(j + 2) % TN][r];
            if constexpr (!PR) sat |= f16_out_of_range(v[i][r]);
          }
        }
        if constexpr (F32OUT) {
          if (four) *(f32x4*)(at(i) + lane_off) = v[i];
          else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (col4 + r < g.N) ((float*)(at(i) + lane_off))[r] = v[i][r];
          }
        } else {
          u32x2 w;
          if constexpr (PR) {
            u32x2 wl;
            SPLIT_BF16X2(v[i][0], v[i][1], w[0], wl[0]);
            SPLIT_BF16X2(v[i][2], v[i][3], w[1], wl[1]);
            *(u32x2*)(at(i) + g.out_lo_off * 2 + lane_off) = wl;
          } else {
            w[0] = pack_f16x2(v[i][0], v[i][1]);
            w[1] = pack_f16x2(v[i][2], v[i][3]);
          }
          *(u32x2*)(at(i) + lane_off) = w;
        }
      }
      SCHED_FENCE();
    }
    if constexpr ((EPI == EPI_GELU_F16 || EPI == EPI_SWIGLU_F16) && !PR) flag_f16_range(sat, g.status);
  }
}
// EPI_QKV_UP: tile columns behind the QKV product's belong to the second one, which takes the first one's place in the arguments
template <int EPI, int BN>
__device__ __forceinline__ bool take_second(GemmArgs& g, int& tile_n) {
  if constexpr (EPI != EPI_QKV_UP) return false;
  const int first = (g.N + BN - 1) / BN;
  if (tile_n < first) return false;
  tile_n -= first;
  g.A = g.A2; g.W = g.W2; g.N = g.N2; g.bias = g.bias2;
  return true;
}
// tile columns of a launch
template <int EPI, int BN>
__host__ __device__ __forceinline__ int tile_cols(const GemmArgs& g) {
  return (g.N + BN - 1) / BN + (EPI == EPI_QKV_UP ? (g.N2 + BN - 1) / BN : 0);
}
template <int TM, int TN, int EPI, bool PR, bool STAGED = false>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& g, const f32x4 (&acc)[TM][TN], int wrow0, int wcol0, int lane, int split, bool second = false) {
  if constexpr (EPI == EPI_QKV_UP) {
    if (second) gemm_epilogue<TM, TN, EPI_GELU_F16, PR>(g, acc, wrow0, wcol0, lane, split);
    else gemm_epilogue<TM, TN, EPI_QKV, PR, STAGED>(g, acc, wrow0, wcol0, lane, split);
    return;
  }
  const bool fits = wrow0 + TM * 16 <= g.M && wcol0 + TN * 16 <= g.N && (EPI != EPI_F32 || (g.ldo & 3) == 0);
  if (fits) gemm_epilogue_as<TM, TN, EPI, PR, true, STAGED>(g, acc, wrow0, wcol0, lane, split);
  else gemm_epilogue_as<TM, TN, EPI, PR, false, STAGED>(g, acc, wrow0, wcol0, lane, split);
}

// One 16x16x32 matrix instruction on 16-bit fragments: fp16, or bf16 in precise mode.  (The 32x32x16 form reads half the
// operand bits per product and yet costs more power: on random operands the chip sustains 1960 TFLOP/s with this one and
// 1700 with that one, at 1.92 and 1.62 GHz.)
template <bool PR>
__device__ __forceinline__ f32x4 mfma16(f16x8 b, f16x8 a, f32x4 c) {
  if constexpr (PR) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b), __builtin_bit_cast(bf16x8, a), c, 0, 0, 0);
  else return __builtin_amdgcn_mfma_f32_16x16x32_f16(b, a, c, 0, 0, 0);
}

// Two LDS stages.  NS = 0: tiles travel global -> registers -> LDS.  NS = 2: by direct global -> LDS loads, issued one K step
// ahead (needs K % 64 == 0).
// PR: precise mode (see GemmArgs): bf16 operands, A as hi/lo pairs; every K block of W meets the hi and then the lo
// block of A in two consecutive steps of the K loop.
template <int BM, int BN, int WM, int WN, int EPI, bool KTAIL, int NS = 0, bool PR = false>
__global__ __launch_bounds__(WM * WN * 64) void gemm_f16_kernel(GemmArgs g) {
  constexpr int NT = WM * WN * 64;               // threads
  constexpr int TM = BM / WM / 16, TN = BN / WN / 16;   // 16x16 MFMA tiles per wave in each direction
  constexpr int RPP = NT / 8;                    // rows covered by one pass of 16-byte loads
  constexpr int PA = BM / RPP, PB = BN / RPP;
  static_assert(PA >= 1 && PB >= 1 && TM >= 1 && TN >= 1, "tile too small for the thread count");
  static_assert(NS == 0 || (NS == 2 && !KTAIL), "direct loads need whole K tiles");
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];   // max(2, NS) x (BM + BN) x BK
  // GEMM waves issue ahead of whatever shares their SIMD: in a decode step that is the other half's attention, whose
  // waves mostly wait for memory (measured: the GEMMs' time in that company -10 %, the decode phase -0.8 %)
  __builtin_amdgcn_s_setprio(3);
  constexpr int STAGE = (BM + BN) * BK;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = tile_cols<EPI, BN>(g);
  int tile_m, tile_n, split;
  const int splits = EPI == EPI_PARTIAL ? g.splits : 1;
  tile_of_block(tiles_m, tiles_n, splits, tile_m, tile_n, split);
  const bool second = take_second<EPI, BN>(g, tile_n);
  const int row0 = tile_m * BM, col0 = tile_n * BN;

  // ---- global -> register staging: thread t covers chunk (t % 8) of rows (t / 8) + RPP i
  const int ld_chunk = tid & 7, ld_row = tid >> 3;
  const uint16_t* __restrict__ A = (const uint16_t*)g.A;
  const uint16_t* __restrict__ W = (const uint16_t*)g.W;
  // operands are K-block major: K tile kt of rows r0.. is the contiguous run starting at (kt * rows + r0) * 64,
  // and thread t reads bytes [16 t, 16 t + 16) of it (rows past the end repeat the last row)
  u32x4 ra[PA], rb[PB];
  const uint16_t* pa[PA];
  const uint16_t* pb[PB];
#pragma unroll
  for (int i = 0; i < PA; ++i) {
    int r = min(row0 + ld_row + RPP * i, g.M - 1);
    pa[i] = A + (size_t)r * 64 + ld_chunk * 8;
  }
#pragma unroll
  for (int i = 0; i < PB; ++i) {
    int r = min(col0 + ld_row + RPP * i, g.N - 1);
    pb[i] = W + (size_t)r * 64 + ld_chunk * 8;
  }
  const size_t ka = (size_t)g.M * 64, kw = (size_t)g.N * 64;    // elements between K tiles
  const int nkb = (g.K + BK - 1) / BK;                          // K blocks of W (and of each half of a hi/lo A)
  // K tile kt of the loop reads block ak(kt) of A and block wk(kt) of W.  Precise mode takes the hi and the lo block of A
  // against the same block of W in consecutive steps (A holds its nkb hi blocks, then its nkb lo blocks): the second
  // request for the W block finds it in L2, so the weights cross HBM once
  auto wk = [&](int kt) { return PR ? kt >> 1 : kt; };
  auto ak = [&](int kt) { return PR ? (kt >> 1) + (kt & 1) * nkb : kt; };
  auto load_global = [&](int kt) {
    if constexpr (KTAIL) {     // K is not a multiple of BK: chunks beyond K read as zero
      const bool ok = wk(kt) * BK + ld_chunk * 8 < g.K;
#pragma unroll
      for (int i = 0; i < PA; ++i) ra[i] = ok ? *(const u32x4*)(pa[i] + ak(kt) * ka) : u32x4{0, 0, 0, 0};
#pragma unroll
      for (int i = 0; i < PB; ++i) rb[i] = ok ? *(const u32x4*)(pb[i] + wk(kt) * kw) : u32x4{0, 0, 0, 0};
    } else {
#pragma unroll
      for (int i = 0; i < PA; ++i) ra[i] = *(const u32x4*)(pa[i] + ak(kt) * ka);
#pragma unroll
      for (int i = 0; i < PB; ++i) rb[i] = *(const u32x4*)(pb[i] + wk(kt) * kw);
    }
  };
  auto store_lds = [&](int buf) {
    uint16_t* la = lds + buf * STAGE;
    uint16_t* lb = la + BM * BK;
#pragma unroll
    for (int i = 0; i < PA; ++i) {
      int r = ld_row + RPP * i;
      *(u32x4*)(la + r * BK + ((ld_chunk ^ swz(r)) * 8)) = ra[i];
    }
#pragma unroll
    for (int i = 0; i < PB; ++i) {
      int r = ld_row + RPP * i;
      *(u32x4*)(lb + r * BK + ((ld_chunk ^ swz(r)) * 8)) = rb[i];
    }
  };

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nk_all = PR ? 2 * nkb : nkb;
  const int kt0 = (int)((long long)split * nk_all / splits);          // this block's share of the K tiles
  const int nk = (int)((long long)(split + 1) * nk_all / splits);
  const int frow = lane & 15, fq = lane >> 4;
  // one K step on the LDS stage `buf`; `mid` runs between the last two MFMA groups
  auto k_step = [&](int buf, auto&& mid) {
    const uint16_t* la = lds + buf * STAGE + (wm * (BM / WM)) * BK;
    const uint16_t* lb = lds + buf * STAGE + BM * BK + (wn * (BN / WN)) * BK;
    // fragments of step kk + 1 are fetched from LDS while the MFMAs of step kk run
    f16x8 fa[2][TM], fb[2][TN];
    auto load_frags = [&](int kk, int slot) {
      const int chunk = kk * 4 + fq;
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        int r = i * 16 + frow;
        fa[slot][i] = *(const f16x8*)(la + r * BK + ((chunk ^ swz(r)) * 8));
      }
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        int r = j * 16 + frow;
        fb[slot][j] = *(const f16x8*)(lb + r * BK + ((chunk ^ swz(r)) * 8));
      }
    };
    load_frags(0, 0);
#pragma unroll
    for (int kk = 0; kk < BK / 32; ++kk) {
      if (kk + 1 < BK / 32) load_frags(kk + 1, (kk + 1) & 1);
      if (kk == BK / 32 - 2) mid();
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = mfma16<PR>(fb[kk & 1][j], fa[kk & 1][i], acc[i][j]);
    }
  };

  if constexpr (NS == 0) {
    load_global(kt0);
    store_lds(kt0 & 1);
    __syncthreads();
    for (int kt = kt0; kt < nk; ++kt) {
      const int cur = kt & 1;
      if (kt + 1 < nk) load_global(kt + 1);
      // the next tile moves from registers to the other LDS buffer under the last MFMAs of this one
      k_step(cur, [&] { if (kt + 1 < nk) store_lds(cur ^ 1); });
      __syncthreads();
    }
  } else {
    // Direct loads: a wave instruction moves 64 16-byte chunks = 8 tile rows into 1 KB of LDS in lane order, so
    // the XOR swizzle is applied on the source side: the lane that fills chunk position p of row r fetches chunk
    // p ^ swz(r).  Rows advance by a multiple of 16 per pass, which leaves swz(r) unchanged.
    static_assert(RPP % 16 == 0, "the swizzle must not depend on the pass");
    const int wave_u = __builtin_amdgcn_readfirstlane(wave);
    const int lrow = wave_u * 8 + (lane >> 3);
    const int schunk = (lane & 7) ^ swz(lrow);
    const uint16_t* qa[PA];
    const uint16_t* qb[PB];
#pragma unroll
    for (int i = 0; i < PA; ++i) qa[i] = A + (size_t)min(row0 + lrow + RPP * i, g.M - 1) * 64 + schunk * 8;
#pragma unroll
    for (int i = 0; i < PB; ++i) qb[i] = W + (size_t)min(col0 + lrow + RPP * i, g.N - 1) * 64 + schunk * 8;
    typedef const __attribute__((address_space(1))) void* gptr_t;
    typedef __attribute__((address_space(3))) void* lptr_t;
    auto issue = [&](int kt, int buf) {
      uint16_t* la = lds + buf * STAGE + wave_u * 8 * BK;
#pragma unroll
      for (int i = 0; i < PA; ++i)
        __builtin_amdgcn_global_load_lds((gptr_t)(qa[i] + ak(kt) * ka), (lptr_t)(la + i * RPP * BK), 16, 0, 0);
#pragma unroll
      for (int i = 0; i < PB; ++i)
        __builtin_amdgcn_global_load_lds((gptr_t)(qb[i] + wk(kt) * kw), (lptr_t)(la + (BM + i * RPP) * BK), 16, 0, 0);
    };
    {
      // Skewed by less than half a K step: the wait for the next stage and the barrier sit behind the first products of the
      // second of a stage's two MFMA groups (one per K slice of 32), whose fragments are in registers by then.  Behind the
      // barrier nobody reads this stage's LDS any more, so its buffer is refilled at once, and the first fragments of the
      // next stage are fetched while the rest of the group runs: the matrix pipe does not drain at the stage boundary.
      f16x8 fa[2][TM], fb[2][TN];
      auto frags = [&](int buf, int kk, int slot) {
        const uint16_t* la = lds + buf * STAGE + (wm * (BM / WM)) * BK;
        const uint16_t* lb = lds + buf * STAGE + BM * BK + (wn * (BN / WN)) * BK;
        const int chunk = kk * 4 + fq;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          int r = i * 16 + frow;
          fa[slot][i] = *(const f16x8*)(la + r * BK + ((chunk ^ swz(r)) * 8));
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          int r = j * 16 + frow;
          fb[slot][j] = *(const f16x8*)(lb + r * BK + ((chunk ^ swz(r)) * 8));
        }
      };
      constexpr int HEAD = TM * TN >= 16 ? 4 : 2;
      auto mma = [&](int slot, int lo, int hi) {     // MFMAs lo .. hi - 1 of the group, row-major over the wave's tiles
#pragma unroll
        for (int t = 0; t < TM * TN; ++t)
          if (t >= lo && t < hi)
            acc[t / TN][t % TN] = mfma16<PR>(fb[slot][t % TN], fa[slot][t / TN], acc[t / TN][t % TN]);
      };
      issue(kt0, 0);
      wait_loads_then_barrier<0>();
      if (kt0 + 1 < nk) issue(kt0 + 1, 1);
      frags(0, 0, 0);
      // Per MFMA group: the first MFMAs, then the LDS reads of the next group's fragments, then the rest, in exactly
      // this order (the fences stop the compiler from sinking the reads behind the MFMAs, where the wait for them
      // would sit directly in front of their first use).  `req` / `more`: is stage kt + 2 requested, does stage kt + 1
      // follow; the loop proper has no conditions inside, since a branch costs a wave as much as an MFMA.
      auto stage = [&](int kt, auto req, auto more) {
        const int buf = (kt - kt0) & 1;
        mma(0, 0, HEAD);
        SCHED_FENCE();
        frags(buf, 1, 1);
        SCHED_FENCE();
        mma(0, HEAD, TM * TN);
        SCHED_FENCE();
        mma(1, 0, HEAD);
        SCHED_FENCE();
        if constexpr (decltype(more)::value) {
          // stage kt + 1 has landed, and every wave holds its last fragments of stage kt in registers
          asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
          if constexpr (decltype(req)::value) issue(kt + 2, buf);
          frags(buf ^ 1, 0, 0);
          SCHED_FENCE();
        }
        mma(1, HEAD, TM * TN);
        SCHED_FENCE();
      };
      int kt = kt0;
#pragma unroll 1
      for (; kt + 2 < nk; ++kt) stage(kt, std::true_type{}, std::true_type{});
      if (kt + 1 < nk) {
        stage(kt, std::false_type{}, std::true_type{});
        ++kt;
      }
      stage(kt, std::false_type{}, std::false_type{});
    }
  }

  gemm_epilogue<TM, TN, EPI, PR>(g, acc, row0 + wm * (BM / WM), col0 + wn * (BN / WN), lane, split, second);
}

// The 256x256 tile: four waves of 128x128, one per SIMD, K >= 128 (two K steps).  Every wave is its SIMD's only one, so the
// main loop is laid out by hand: between any two products there is at most one LDS read or one request, and no branch.
// A K step is four phases of 32 products, one for each pair of row half and column half; a half tile (128 rows of 64 K
// values, 16 KB) is read from LDS into registers one phase before its first use and never again, so its place in LDS is
// free two phases later and takes the same half of the K step after next: five to six half tiles (80 - 96 KB) are in flight
// all the time, which covers the 1.3 us that the operand stream takes from HBM and the other XCDs' L2 under load.  One
// barrier per phase: the half needed next has landed, and everybody has read the half that is about to be overwritten.
// Measured (M = 32768, random operands, bursts of ten): N = 2560, K = 10240 1.28 PFLOP/s where the two-stage loop on eight
// waves gave 1.01, N = 10240, K = 2560 with GELU 1.19 (0.90), N = 7680, K = 2560 1.16 (0.95; 1.04 in a whole prompt pass).  The
// loop is bound by power: 2420 clocks per K step (2048 of them matrix products) at 1.65 GHz; on zeros the clock stays at 2.4 GHz.
// The other products raise their waves' priority for the decode step's sake; this one need not (the LM head is all of a decode
// step it takes: generate of 2.8B width on two streams 371.1 ms without, 370.3 with, 1B 137.3 and 137.4).
template <int EPI, bool PR>
__global__ __launch_bounds__(256, 1) void gemm_big_kernel(GemmArgs g) {
  constexpr int TM = 8, TN = 8;                  // 16x16 tiles of a wave: 128 x 128
  constexpr int HALF = 128 * BK;                 // elements of a half tile: 128 rows of one K step
  constexpr int STAGE = 4 * HALF;                // A0, A1, B0, B1
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];   // two stages
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int tiles_m = (g.M + 255) >> 8, tiles_n = tile_cols<EPI, 256>(g);
  int tile_m, tile_n, split;
  tile_of_block(tiles_m, tiles_n, 1, tile_m, tile_n, split);
  const bool second = take_second<EPI, 256>(g, tile_n);
  const int row0 = tile_m << 8, col0 = tile_n << 8;

  const int nkb = g.K / BK;                      // K blocks of W (and of each half of a hi/lo A)
  const int nk = PR ? 2 * nkb : nkb;
  const size_t ka = (size_t)g.M * 128, kw = (size_t)g.N * 128;    // bytes between K blocks
  // A wave instruction moves 64 16-byte chunks = 8 rows into 1 KB of LDS in lane order; a wave fills 32 of a half tile's
  // 128 rows.  Row r of half h is row 128 (r / 64) + 64 h + r % 64 of the tile: 64 rows for each of the two waves that
  // share the operand.  The XOR swizzle is applied on the source side.  The tile's first row is part of the 64-bit base, so that
  // the 32-bit distances stay inside the tile (a matrix of 2^24 rows has 2 GiB to a K block).
  const char* const a0 = (const char*)g.A + (size_t)row0 * 128;
  const char* const w0 = (const char*)g.W + (size_t)col0 * 128;
  uint32_t va[2][4], vb[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = wave * 32 + i * 8 + (lane >> 3);
      const int chunk = (lane & 7) ^ swz(r);
      const int t = (r >> 6) * 128 + h * 64 + (r & 63);
      va[h][i] = (uint32_t)min(t, g.M - 1 - row0) * 128 + chunk * 16;
      vb[h][i] = (uint32_t)min(t, g.N - 1 - col0) * 128 + chunk * 16;
    }
  typedef __attribute__((address_space(3))) void* lptr_t;
  // request i (of 4) of half h of K step kt
  auto load_a = [&](int kt, int h, int i) {
    const char* base = a0 + (size_t)(PR ? (kt >> 1) + (kt & 1) * nkb : kt) * ka;
    uint16_t* dst = lds + (kt & 1) * STAGE + h * HALF + wave * 32 * BK + i * 8 * BK;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, 0x00027000), (lptr_t)dst, 16, va[h][i], 0, 0, 0);
  };
  auto load_b = [&](int kt, int h, int i) {
    const char* base = w0 + (size_t)(PR ? kt >> 1 : kt) * kw;
    uint16_t* dst = lds + (kt & 1) * STAGE + (2 + h) * HALF + wave * 32 * BK + i * 8 * BK;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, 0x00027000), (lptr_t)dst, 16, vb[h][i], 0, 0, 0);
  };
  const int frow = lane & 15, fq = lane >> 4;
  const int sw = swz(frow);
  int oa[2], ob[2];                       // LDS element offsets of this lane's fragments, by K slice of 32
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int c = ((4 * ks + fq) ^ sw) * 8;
    oa[ks] = (wm * 64 + frow) * BK + c;
    ob[ks] = 2 * HALF + (wn * 64 + frow) * BK + c;
  }
  f16x8 fa[2][4][2], fb[2][4][2];         // [half][16-row tile][K slice]
  // fragment n (of 8) of half h in buffer buf: tile n % 4, K slice n / 4
  auto read_a = [&](int buf, int h, int n) { fa[h][n & 3][n >> 2] = *(const f16x8*)(lds + buf * STAGE + h * HALF + (n & 3) * 16 * BK + oa[n >> 2]); };
  auto read_b = [&](int buf, int h, int n) { fb[h][n & 3][n >> 2] = *(const f16x8*)(lds + buf * STAGE + h * HALF + (n & 3) * 16 * BK + ob[n >> 2]); };
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#define BIG_BAR(N, L) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(%1)\n\ts_barrier" ::"n"(N), "n"(L) : "memory")
  // the 32 products of row half mh and column half nh; behind the n-th, rd(n) fetches fragments and ld(0..3) requests
  auto phase = [&](int mh, int nh, auto&& rd, auto&& ld) {
#pragma unroll
    for (int n = 0; n < 32; ++n) {
      const int ks = n >> 4, i = (n >> 2) & 3, j = n & 3;
      acc[4 * mh + i][4 * nh + j] = mfma16<PR>(fb[nh][j][ks], fa[mh][i][ks], acc[4 * mh + i][4 * nh + j]);
      SCHED_FENCE();
      rd(n);
      if (n % 4 == 1 && n < 16) ld(n / 4);
      SCHED_FENCE();
    }
  };
  // T: 0 in the loop, 1 in the last K step but one, 2 in the last (nothing is requested any more)
  auto step = [&](int kt, auto tail) {
    constexpr int T = decltype(tail)::value;
    const int buf = kt & 1;
    phase(0, 0, [&](int n) { if (n % 2 == 0 && n < 16) read_b(buf, 1, n / 2); }, [&](int n) { if (T == 0) load_a(kt + 2, 0, n); });
    BIG_BAR(T == 0 ? 20 : T == 1 ? 16 : 0, T == 0 ? 8 : 0);
    SCHED_FENCE();
    phase(0, 1, [&](int n) { if (n % 2 == 0 && n < 16) read_a(buf, 1, n / 2); }, [&](int n) { if (T == 0) load_b(kt + 2, 0, n); });
    BIG_BAR(T == 0 ? 20 : T == 1 ? 12 : 0, T == 0 ? 8 : 0);
    SCHED_FENCE();
    phase(1, 1, [&](int n) { if (T < 2 && n % 2 == 0 && n < 16) read_a(buf ^ 1, 0, n / 2); }, [&](int n) { if (T == 0) load_b(kt + 2, 1, n); });
    BIG_BAR(T == 0 ? 20 : T == 1 ? 8 : 0, T == 0 ? 8 : 0);
    SCHED_FENCE();
    // the next K step's B0 takes the registers of this one's as they are used up
    phase(1, 0, [&](int n) {
      if (T < 2 && n >= 16 && n < 20) read_b(buf ^ 1, 0, n - 16);
      if (T < 2 && n >= 28) read_b(buf ^ 1, 0, 4 + n - 28);
    }, [&](int n) { if (T == 0) load_a(kt + 2, 1, n); });
    if constexpr (T < 2) BIG_BAR(T == 0 ? 20 : 4, T == 0 ? 8 : 0);
    SCHED_FENCE();
  };
#pragma unroll
  for (int s = 0; s < 2; ++s) {
#pragma unroll
    for (int i = 0; i < 4; ++i) load_a(s, 0, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_b(s, 0, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_b(s, 1, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_a(s, 1, i);
  }
  BIG_BAR(24, 0);
#pragma unroll
  for (int n = 0; n < 8; ++n) { read_a(0, 0, n); read_b(0, 0, n); }
  BIG_BAR(20, 0);
  int kt = 0;
#pragma unroll 1
  for (; kt < nk - 2; ++kt) step(kt, std::integral_constant<int, 0>{});
  step(kt, std::integral_constant<int, 1>{});
  step(kt + 1, std::integral_constant<int, 2>{});
  gemm_epilogue<TM, TN, EPI, PR, true>(g, acc, row0 + wm * 128, col0 + wn * 128, lane, 0, second);
}
#undef BIG_BAR

// Tiles for launches with few blocks to a CU (decode steps, short prompt passes): a ring of NS stages of 64 K values, requested
// NS - 1 stages ahead, and fragments one K slice of 32 ahead of the products, across the stage boundary too.  The wait for
// the next stage and the only barrier of a K step sit between its two slices, where every wave holds fragments for the
// second; behind the barrier nobody reads the stage before any more, whose slot is requested anew.  No branch in the loop.
// What bounds these launches is the latency of the weights (1 us from another XCD's side of the chip, 1.8 us from HBM) over
// the bytes a CU has in flight, and the number of CUs that have a block, so the shapes go from 32x32 (several blocks to a CU) to
// 256x128 (most of LDS).  Measured with weights from HBM (us): 32x32, 16 rows, N x K = 3072 x 1024 4.8, 6144 x 2048 7.1, 6144 x
// 4096 11.3 (64x64 6.8, 10.5, 18.9); 32x64, 64 rows, 6144 x 2048 9.5 (64x64 11.8); 64x64, 128 rows, 4096 x 1024 7.4 and as the 8
// parts of a K split 1024 x 5120 6.6; 64x96 (64x128), 256 rows, 6144 x 4096 25.4 (28.4); 128x64, 256 rows, 8192 x 2048 16.4 (17.1);
// 32x128, 16 rows, 28672 x 4096 38.2 (128x128 42.0); 256x128, 1024 rows, 7680 x 2560 43.9 (two-stage loop 48.8).  K divided
// among the waves of a block instead, operands straight to registers: 16 rows, 6144 x 2048 8.3, 2048 x 10240 21.2 (64x64 in 8
// parts 9.5), 128 rows, 4096 x 1024 8.6: such operands are 64-byte pieces of sixteen rows, which a CU takes in at a third of the
// rate of the kilobytes that go to LDS.
template <int BM, int BN, int WM, int WN, int NS, int EPI, bool PR = false>
__global__ __launch_bounds__(WM * WN * 64) void gemm_ring_kernel(GemmArgs g) {
  constexpr int NW = WM * WN;                            // waves
  constexpr int TM = BM / WM / 16, TN = BN / WN / 16;    // 16x16 tiles of a wave
  constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW, L = LA + LB;     // requests per wave and stage, 8 rows each
  constexpr int STAGE = (BM + BN) * BK;
  static_assert(NS >= 3 && (NS - 2) * L < 64 && BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "whole requests, as many as a wait can count");
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];   // NS stages
  __builtin_amdgcn_s_setprio(3);       // ahead of the other half's attention (see gemm_f16_kernel)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = tile_cols<EPI, BN>(g);
  int tile_m, tile_n, split;
  const int splits = EPI == EPI_PARTIAL ? g.splits : 1;
  tile_of_block(tiles_m, tiles_n, splits, tile_m, tile_n, split);
  const bool second = take_second<EPI, BN>(g, tile_n);
  const int row0 = tile_m * BM, col0 = tile_n * BN;
  const int nkb = g.K / BK;
  const int nk_all = PR ? 2 * nkb : nkb;
  const int kt0 = (int)((long long)split * nk_all / splits);
  const int nk = (int)((long long)(split + 1) * nk_all / splits) - kt0;       // this block's K steps
  const size_t ka = (size_t)g.M * 128, kw = (size_t)g.N * 128;
  const char* const a0 = (const char*)g.A + (size_t)row0 * 128;      // 32-bit distances stay inside the tile
  const char* const w0 = (const char*)g.W + (size_t)col0 * 128;
  uint32_t va[LA], vb[LB];
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    const int r = (wave * LA + i) * 8 + (lane >> 3);
    va[i] = (uint32_t)min(r, g.M - 1 - row0) * 128 + ((lane & 7) ^ swz(r)) * 16;
  }
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    const int r = (wave * LB + i) * 8 + (lane >> 3);
    vb[i] = (uint32_t)min(r, g.N - 1 - col0) * 128 + ((lane & 7) ^ swz(r)) * 16;
  }
  typedef __attribute__((address_space(3))) void* lptr_t;
  // request n of stage kt (counted from kt0) into slot s: first the rows of A, then those of W
  auto request = [&](int kt, int s, int n) {
    kt += kt0;
    const bool is_a = n < LA;
    const char* base = is_a ? a0 + (size_t)(PR ? (kt >> 1) + (kt & 1) * nkb : kt) * ka : w0 + (size_t)(PR ? kt >> 1 : kt) * kw;
    uint16_t* dst = lds + s * STAGE + (is_a ? wave * LA + n : BM / 8 + wave * LB + n - LA) * 8 * BK;
    const uint32_t off = is_a ? va[is_a ? n : 0] : vb[is_a ? 0 : n - LA];
    __builtin_amdgcn_raw_ptr_buffer_load_lds(__builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, 0x00027000), (lptr_t)dst, 16, off, 0, 0, 0);
  };
  const int frow = lane & 15, fq = lane >> 4;
  int oa[2], ob[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int c = ((4 * ks + fq) ^ swz(frow)) * 8;
    oa[ks] = (wm * (BM / WM) + frow) * BK + c;
    ob[ks] = (BM + wn * (BN / WN) + frow) * BK + c;
  }
  f16x8 fa[2][TM], fb[2][TN];
  auto read = [&](int s, int ks, int n) {      // fragment n of K slice ks of the stage in slot s
    const uint16_t* st = lds + s * STAGE;
    if (n < TN) fb[ks][n < TN ? n : 0] = *(const f16x8*)(st + ob[ks] + n * 16 * BK);
    else fa[ks][n < TN ? 0 : n - TN] = *(const f16x8*)(st + oa[ks] + (n - TN) * 16 * BK);
  };
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int T = TM * TN, R = TM + TN;
  auto slice = [&](int ks, auto&& rd, auto&& rq) {
#pragma unroll
    for (int n = 0; n < T; ++n) {
      acc[n / TN][n % TN] = mfma16<PR>(fb[ks][n % TN], fa[ks][n / TN], acc[n / TN][n % TN]);
      SCHED_FENCE();
#pragma unroll
      for (int r = n * R / T; r < (n + 1) * R / T; ++r) rd(r);
#pragma unroll
      for (int l = n * L / T; l < (n + 1) * L / T; ++l) rq(l);
      SCHED_FENCE();
    }
  };
#define RING_WAIT(N) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory")
  auto wait_younger = [&](int stages) {     // all but the `stages` youngest stages of this wave have landed; then everybody is here
    if (stages >= NS - 2) RING_WAIT((NS - 2) * L);
    else if (NS > 6 && stages >= 4) RING_WAIT(4 * L);
    else if (stages == 3) RING_WAIT(3 * L);
    else if (stages == 2) RING_WAIT(2 * L);
    else if (stages == 1) RING_WAIT(L);
    else RING_WAIT(0);
  };
#pragma unroll
  for (int s = 0; s < NS - 1; ++s)
    if (s < nk) {
#pragma unroll
      for (int n = 0; n < L; ++n) request(s, s, n);
    }
  wait_younger(min(nk, NS - 1) - 1);
#pragma unroll
  for (int n = 0; n < R; ++n) read(0, 0, n);
  int kt = 0, s = 0;
  auto next = [](int x) { return x + 1 == NS ? 0 : x + 1; };
#pragma unroll 1
  for (; kt + NS - 1 < nk; ++kt) {
    const int s1 = next(s), sp = s == 0 ? NS - 1 : s - 1;
    slice(0, [&](int n) { read(s, 1, n); }, [](int) {});
    RING_WAIT((NS - 3) * L);
    SCHED_FENCE();
    slice(1, [&](int n) { read(s1, 0, n); }, [&](int n) { request(kt + NS - 1, sp, n); });
    s = s1;
  }
#pragma unroll 1
  for (; kt + 1 < nk; ++kt) {
    const int s1 = next(s);
    slice(0, [&](int n) { read(s, 1, n); }, [](int) {});
    wait_younger(nk - 2 - kt);
    SCHED_FENCE();
    slice(1, [&](int n) { read(s1, 0, n); }, [](int) {});
    s = s1;
  }
  if (nk > 0) {
    slice(0, [&](int n) { read(s, 1, n); }, [](int) {});
    slice(1, [](int) {}, [](int) {});
  }
  gemm_epilogue<TM, TN, EPI, PR>(g, acc, row0 + wm * (BM / WM), col0 + wn * (BN / WN), lane, split, second);
}
#undef RING_WAIT

// Second half of a split-K product: sums the partial results in split order (so the result does not depend
// on scheduling) and applies the epilogue.
template <int EPI>
__global__ void splitk_epilogue_kernel(GemmArgs g) {
  const size_t n = (size_t)g.M * g.N;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int row = (int)(i / g.N), col = (int)(i % g.N);
  float v = 0.f;
  for (int sp = 0; sp < g.splits; ++sp) v += g.ws[(size_t)sp * n + i];
  if (g.bias) v += g.bias[col];
  if constexpr (EPI == EPI_F32) {
    ((float*)g.out)[(size_t)row * g.ldo + col] = v;
  } else if constexpr (EPI == EPI_RESID) {
    float* p = (float*)g.out + (size_t)row * g.ldo + col;
    *p = *p + v;
  } else if constexpr (EPI == EPI_GELU_F16) {
    v = gelu_erf(v);
    uint16_t* p = (uint16_t*)g.out + kblk_off(row, col, g.M);
    if (g.precise) {
      split_bf16(v, p[0], p[g.out_lo_off]);
    } else {
      flag_f16_range(f16_out_of_range(v), g.status);
      *p = f32_to_f16_bits(v);
    }
  }
}

template <int BM, int BN, int WM, int WN, int EPI, bool KTAIL, int NS = 0, bool PR = false>
hipError_t launch_k(const GemmArgs& g, hipStream_t s) {
  constexpr size_t lds_bytes = (NS ? NS : 2) * (size_t)(BM + BN) * BK * sizeof(uint16_t);
  static_assert(lds_bytes <= 160 * 1024, "LDS of one CU");
  // once per device and instantiation (a repeated call is harmless, so no lock)
  static bool configured_on[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  bool& configured = configured_on[dev];
  if (!configured) {
    if (lds_bytes > 65536) {
      hipError_t e = hipFuncSetAttribute((const void*)gemm_f16_kernel<BM, BN, WM, WN, EPI, KTAIL, NS, PR>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
      if (e != hipSuccess) return e;
    }
    configured = true;
  }
  const int tiles = ((g.M + BM - 1) / BM) * tile_cols<EPI, BN>(g) * (EPI == EPI_PARTIAL ? g.splits : 1);
  hipLaunchKernelGGL((gemm_f16_kernel<BM, BN, WM, WN, EPI, KTAIL, NS, PR>), dim3(tiles), dim3(WM * WN * 64), lds_bytes, s, g);
  return hipGetLastError();
}

// the 256x256 tile; a K of less than two steps or with a ragged end goes through registers
template <int EPI, bool PR>
hipError_t launch_big(const GemmArgs& g, hipStream_t s) {
  if (g.K % BK != 0 || (!PR && g.K < 2 * BK)) return launch_k<256, 256, 4, 2, EPI, true, 0, PR>(g, s);
  constexpr int lds_bytes = 2 * 512 * BK * (int)sizeof(uint16_t);
  static bool configured_on[64] = {};       // once per device (a repeated call is harmless, so no lock)
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (!configured_on[dev]) {
    hipError_t e = hipFuncSetAttribute((const void*)gemm_big_kernel<EPI, PR>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (e != hipSuccess) return e;
    configured_on[dev] = true;
  }
  const int tiles = ((g.M + 255) / 256) * tile_cols<EPI, 256>(g);
  hipLaunchKernelGGL((gemm_big_kernel<EPI, PR>), dim3(tiles), dim3(256), lds_bytes, s, g);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int NS, int EPI, bool PR = false>
hipError_t launch_ring(const GemmArgs& g, hipStream_t s) {
  constexpr int lds_bytes = NS * (BM + BN) * BK * (int)sizeof(uint16_t);
  static_assert(lds_bytes <= 160 * 1024, "LDS of one CU");
  static bool configured_on[64] = {};       // once per device (a repeated call is harmless, so no lock)
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (lds_bytes > 65536 && !configured_on[dev]) {
    hipError_t e = hipFuncSetAttribute((const void*)gemm_ring_kernel<BM, BN, WM, WN, NS, EPI, PR>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (e != hipSuccess) return e;
    configured_on[dev] = true;
  }
  const int tiles = ((g.M + BM - 1) / BM) * tile_cols<EPI, BN>(g) * (EPI == EPI_PARTIAL ? g.splits : 1);
  hipLaunchKernelGGL((gemm_ring_kernel<BM, BN, WM, WN, NS, EPI, PR>), dim3(tiles), dim3(WM * WN * 64), lds_bytes, s, g);
  return hipGetLastError();
}

// Whole K tiles take the direct-load pipeline with two LDS stages, which leave room for a second block on a CU (launches with fewer
// blocks take the ring); a ragged K falls back to register staging, which can zero-fill the tail.
template <int BM, int BN, int WM, int WN, int EPI, int NS = 2, bool PR = false>
hipError_t launch(const GemmArgs& g, hipStream_t s) {
  return g.K % BK == 0 ? launch_k<BM, BN, WM, WN, EPI, false, NS, PR>(g, s) : launch_k<BM, BN, WM, WN, EPI, true, 0, PR>(g, s);
}

// precise mode is compiled for four of the tile shapes (128x128, 256x256, 256x128 with 8 waves, 64x128)
template <int EPI>
hipError_t launch_variant_precise(const GemmArgs& g, int variant, hipStream_t s) {
  switch (variant) {
    case 0: return launch<128, 128, 2, 2, EPI, 2, true>(g, s);
    case 3:
      if (EPI == EPI_PARTIAL || (EPI == EPI_QKV && !g.qe.kvstage)) return launch<256, 128, 4, 2, EPI, 2, true>(g, s);
      if constexpr (EPI != EPI_PARTIAL) return launch_big<EPI, true>(g, s);
      break;
    case 5: return launch<256, 128, 4, 2, EPI, 2, true>(g, s);
    case 7:
      if constexpr (EPI != EPI_SWIGLU_F16 && EPI != EPI_LMHEAD) return launch<64, 128, 1, 4, EPI, 2, true>(g, s);
      else return hipErrorInvalidValue;
  }
  return hipErrorInvalidValue;
}

// the tile shapes by number; a K that is not whole K tiles takes the register-staged form of the same or the nearest tile
template <int EPI>
hipError_t launch_variant(const GemmArgs& g, int variant, hipStream_t s) {
  if constexpr (EPI == EPI_QKV_UP) {
    if (g.precise) return hipErrorInvalidValue;
  } else {
    if (g.precise) return launch_variant_precise<EPI>(g, variant, s);
  }
  constexpr bool WIDE = EPI == EPI_SWIGLU_F16 || EPI == EPI_LMHEAD;      // a wave must own 64 columns
  const bool whole = g.K % BK == 0;
  switch (variant) {
    case 0: return launch<128, 128, 2, 2, EPI>(g, s);
    case 2: return whole ? launch_ring<128, 128, 4, 2, 4, EPI>(g, s) : launch_k<128, 128, 2, 2, EPI, true, 0>(g, s);
    case 3:
      // (a K split is for shapes with few tiles: partial sums come from 256x128 at most, and so do a decode step's cache writes)
      if (EPI == EPI_PARTIAL || ((EPI == EPI_QKV || EPI == EPI_QKV_UP) && !g.qe.kvstage)) return launch<256, 128, 4, 2, EPI>(g, s);
      if constexpr (EPI != EPI_PARTIAL) return launch_big<EPI, false>(g, s);
      break;
    case 5: return launch<256, 128, 4, 2, EPI>(g, s);
    case 10: return whole ? launch_ring<256, 128, 4, 2, 3, EPI>(g, s) : launch_k<256, 128, 4, 2, EPI, true, 0>(g, s);
  }
  if constexpr (WIDE) {
    if (!whole) return launch_k<128, 128, 2, 2, EPI, true, 0>(g, s);
    switch (variant) {
      case 1: return launch_ring<32, 128, 2, 2, 7, EPI>(g, s);
      case 4: return launch_ring<64, 128, 2, 2, 6, EPI>(g, s);
    }
  } else {
    if (!whole) return launch_k<64, 128, 1, 4, EPI, true, 0>(g, s);
    switch (variant) {
      case 1: return launch_ring<32, 32, 2, 2, 8, EPI>(g, s);
      case 4: return launch_ring<32, 64, 2, 2, 6, EPI>(g, s);
      case 6: return launch_ring<64, 64, 2, 2, 5, EPI>(g, s);
      case 7: return launch_ring<128, 64, 4, 2, 6, EPI>(g, s);
      case 8: return launch_ring<64, 96, 2, 2, 7, EPI>(g, s);
      case 9: return launch_ring<64, 128, 2, 4, 6, EPI>(g, s);
      // (two stages leave room for three blocks to a CU, a ring of 64x128 for one: where the tiles make a round and a half to three, us:
      // 1300 rows, 1024 x 5120 in 3 parts 25.8 (rings 27.0 and more), 300 rows, 2560 x 12800 in 5 parts 37.8 (42.1), 10240 x 2560,
      // 420 rows 41.7 (43.7))
      case 11: return launch<64, 128, 1, 4, EPI>(g, s);
    }
  }
  return hipErrorInvalidValue;
}

}  // namespace

static bool valid_qkv(const GemmArgs& g) {
  const QkvEpi& e = g.qe;
  return e.r % 4 == 0 && e.h % 16 == 0 && g.N == (e.Hq + 2 * e.Hkv) * e.h && e.q && e.pos && (e.r == 0 || e.table) &&
         (e.kvstage || (e.kv && e.dst_seq && e.kv_off && e.kv_cap));
}
hipError_t rl_gemm_variant(const GemmArgs& g, int epi, int variant, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (g.K % 8 != 0) return hipErrorInvalidValue;
  // only the plain fp32 and the LM-head epilogue take rows that do not divide into groups of four columns (every other
  // width is a multiple of 16 by the checks on the configuration)
  if (epi != EPI_F32 && epi != EPI_LMHEAD && (g.N % 4 != 0 || (epi == EPI_RESID && g.ldo % 4 != 0))) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_F32: return launch_variant<EPI_F32>(g, variant, s);
    case EPI_RESID: return launch_variant<EPI_RESID>(g, variant, s);
    case EPI_GELU_F16: return launch_variant<EPI_GELU_F16>(g, variant, s);
    case EPI_SWIGLU_F16:
      if (g.N % 64 != 0) return hipErrorInvalidValue;
      return launch_variant<EPI_SWIGLU_F16>(g, variant, s);
    case EPI_LMHEAD:
      if (!(g.temperature >= MIN_FAST_TEMPERATURE))
        return g.precise ? launch<128, 128, 2, 2, EPI_LMHEAD_EXACT, 2, true>(g, s) : launch<128, 128, 2, 2, EPI_LMHEAD_EXACT>(g, s);
      return launch_variant<EPI_LMHEAD>(g, variant, s);
    case EPI_PARTIAL: return launch_variant<EPI_PARTIAL>(g, variant, s);
    case EPI_QKV_UP:
      if (!valid_qkv(g) || !g.A2 || !g.W2 || !g.out || g.N2 <= 0 || g.N2 % 4 != 0) return hipErrorInvalidValue;
      return launch_variant<EPI_QKV_UP>(g, variant, s);
    case EPI_QKV: {
      return valid_qkv(g) ? launch_variant<EPI_QKV>(g, variant, s) : hipErrorInvalidValue;
    }
  }
  return hipErrorInvalidValue;
}

// Split-K: `splits` blocks per tile each take a share of K and write fp32 partial tiles to g.ws
// ([splits, M, N]); a second kernel adds them in order and applies the epilogue.
hipError_t rl_gemm_parts(const GemmArgs& g, int variant, hipStream_t s) {
  // the partial sums must fit, and every part must have a K tile: the two-stage loop takes its last one without asking
  if (g.splits < 2 || !g.ws || (size_t)g.splits * g.M * g.N > g.ws_elems) return hipErrorInvalidValue;
  if (g.splits > (g.K + BK - 1) / BK * (g.precise ? 2 : 1)) return hipErrorInvalidValue;
  return rl_gemm_variant(g, EPI_PARTIAL, variant, s);
}
hipError_t rl_gemm_splitk(const GemmArgs& g, int epi, int variant, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (epi != EPI_F32 && epi != EPI_RESID && epi != EPI_GELU_F16) return hipErrorInvalidValue;
  hipError_t e = rl_gemm_parts(g, variant, s);
  if (e != hipSuccess) return e;
  const size_t n = (size_t)g.M * g.N;
  const dim3 grid((unsigned)((n + 255) / 256)), block(256);
  if (epi == EPI_F32) hipLaunchKernelGGL(splitk_epilogue_kernel<EPI_F32>, grid, block, 0, s, g);
  else if (epi == EPI_RESID) hipLaunchKernelGGL(splitk_epilogue_kernel<EPI_RESID>, grid, block, 0, s, g);
  else hipLaunchKernelGGL(splitk_epilogue_kernel<EPI_GELU_F16>, grid, block, 0, s, g);
  return hipGetLastError();
}

// Tile shape by problem size (measured on MI355X): the largest tile that still gives every CU work.  The K split is
// the caller's (g.splits >= 2 with g.ws set), never chosen here: it fixes the order of the sums.
hipError_t rl_gemm(const GemmArgs& g, int epi, hipStream_t s) {
  const int cols = g.N + (epi == EPI_QKV_UP ? g.N2 : 0);
  auto tiles = [&](int bm, int bn) { return (long long)((g.M + bm - 1) / bm) * ((cols + bn - 1) / bn); };
  const bool wide_only = (epi == EPI_SWIGLU_F16 || epi == EPI_LMHEAD);   // a wave must own 64 columns
  int variant;
  if (tiles(256, 256) >= 160) variant = 3;
  else if (tiles(256, 128) >= 200) variant = 5;
  else if (tiles(128, 128) >= 400 || wide_only) variant = 0;
  else variant = g.precise ? 7 : 9;
  if (g.splits >= 2 && g.ws) return rl_gemm_splitk(g, epi, wide_only ? 0 : g.precise ? 7 : 9, s);
  return rl_gemm_variant(g, epi, variant, s);
}
