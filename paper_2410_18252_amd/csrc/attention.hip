// Softmax attention over the per-sequence bf16 KV cache, for the decode step (one query per
// sequence and query head: the bandwidth-bound part of generation) and for causal prefill.
//
// One wave owns 16 "columns" (queries) and streams one (sequence, kv head) K/V stream in
// super-blocks of 32 keys.  The matrix cores serve as dot-product engines fed straight from global
// memory: the operands never pass through LDS (only what the waves of a shared job add up does), and there is no cross-lane
// reduction over head_dim.
//   S^T[key, col] = sum_d K[key, d] q[col, d]       2 x ceil(h/32) MFMA 16x16x32 per super-block
//   O^T[d, col]  += sum_key V^T[d, key] P^T[key, col]   h/16 MFMA 16x16x32 per super-block
// K and V are stored as bf16 and widened to fp16 in registers (exact for every value in fp16's
// normal range); queries, probabilities and the MFMAs are fp16 with fp32 accumulation.
// The cache is read once and never again within a launch, so its loads are non-temporal (measured:
// +7 % bandwidth), and the next super-block is requested before the current one is consumed.
// The cache layout (see KvLayout) makes every operand fragment one 16-byte load per lane and every
// load instruction one contiguous kilobyte per wave.  The K rows of a super-block are assigned to
// MFMA rows so that the score registers of lane group g (keys 8g..8g+7) are exactly the B-operand
// fragment P^T the second product needs: probabilities never leave registers.
// Decode with one kv head serving G query heads (grouped-query attention) puts the G heads in the
// columns, so K/V are read once per group; with G = 1 the query is replicated over the columns.
// With a shared prompt cache (share_k = K samples per prompt) the K samples sit in the columns as well:
// the prompt's stream is read once for all of them, then each sample's short stream of new tokens.
// Precise mode (PR): every operand is a bf16 hi/lo pair -- the cache holds a second plane with the lo halves, the
// queries arrive as fp32 and are split in registers, the probabilities are split after the softmax -- and each product
// is three bf16 matrix instructions (hi hi + lo hi + hi lo; the lo lo term is below fp32's own rounding).
#include "kernels.h"

#ifndef ATTN_PREFETCH
#define ATTN_PREFETCH 1
#endif
#ifndef ATTN_PREFETCH2
#define ATTN_PREFETCH2 1
#endif
// The prompt pass of contexts whose jobs do not fill the chip, and of precise mode, is not bound by memory but by the latency of a
// wave's serial chain (load, convert, MFMA, softmax, MFMA): it does without the register prefetch of the next super-block, so that
// two or three waves share a SIMD (one at head size 256) and hide each other's L2 latency: with the prefetch 3000 rows, 8 heads of
// size 80, 25.9 us instead of 17.8.
#ifndef ATTN_PROMPT_NOPF
#define ATTN_PROMPT_NOPF 1
#endif
#ifndef ATTN_NT
#define ATTN_NT 1
#endif
#if ATTN_NT
#define ATTN_LOAD(p) __builtin_nontemporal_load(p)
#else
#define ATTN_LOAD(p) (*(p))
#endif

namespace {

// SPLIT > 1: the waves of a block share one job, wave w taking the super-blocks w, w + SPLIT, ... of every segment; their
// maxima, sums and outputs meet in LDS and are added in the order of the waves.  For contexts whose batches cannot give every
// CU several jobs: a wave's walk over its keys is a serial chain of loads and products, 2.8 us a super-block at head size 256.
// QB = query blocks of 16 columns a wave carries through one pass over the keys (prompt pass only: two blocks halve
// the key / value traffic per query; a.jobs then counts blocks of 16 QB tokens).
// Three waves to a SIMD are prescribed where the prompt pass of small contexts would miss them by a few registers (654 tokens, 32 heads
// of size 64 on 8: 16.8 -> 14.5 us; 1300 rows, 8 heads of size 112: 16.4 -> 13.5).
template <int HD, bool DECODE, int QB = 1, bool PR = false, int SPLIT = 1>
__global__ __launch_bounds__(SPLIT > 4 ? SPLIT * 64 : 256, !DECODE && !PR && SPLIT == 4 && (HD == 64 || HD == 112) ? 3 : 1) void attention_kernel(AttnArgs a) {
  static_assert(!DECODE || QB == 1, "decode has one query block");
  static_assert(SPLIT == 1 || SPLIT == 4 || (DECODE && SPLIT == 8), "a job is shared by all waves of a block");
  constexpr int NCH = HD / 8;            // 16-byte chunks per key row
  constexpr int KSTEPS = (HD + 31) / 32; // MFMA steps over head_dim for the scores
  constexpr int VT = HD / 16;            // 16-row tiles of V^T / O^T
  // is the next super-block requested one iteration ahead (precise mode holds two planes per super-block in registers
  // and loads them at the top of the iteration instead)
  constexpr bool PF = (DECODE || !ATTN_PROMPT_NOPF) && !PR;
  constexpr int NP = PR ? 2 : 1;         // cache planes: hi, lo
  // Decode of heads whose wave has a SIMD to itself whatever it holds: values are widened with the keys, off the chain behind the
  // softmax (8 heads, us: size 256, 16 sequences of 1000 keys 36.4 -> 33.3, 40 75.4 -> 73.3; size 112, 64 sequences 46.3 -> 45.1).
  // Elsewhere it costs registers: size 64, eight waves to a job, 64 sequences 25.6 -> 28.1; 128, 24 sequences of 2000 keys 36.8 -> 37.2
  constexpr bool V_EARLY = DECODE && !PR && SPLIT <= 4 && (HD == 112 || HD == 256);
  const int lane = threadIdx.x & 63;
  // A wave number known to be common to the wave makes the job's addresses scalar.  Not for two query blocks to a wave: the compiler
  // then orders their loop worse (precise mode, head size 48, 16 prompts of 500 tokens, 20 heads: 117 -> 123 us)
  const int wave = QB == 1 || SPLIT > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : (int)(threadIdx.x >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int Hkv = a.lay.Hkv, G = a.Hq / Hkv;
  const int job = SPLIT > 1 ? blockIdx.x : blockIdx.x * 4 + wave;
  const int sb0 = SPLIT > 1 ? wave : 0;                 // first super-block of this wave

  // A job streams one or more segments.  Segment i is the stream of cache sequence seg_seq(i) with seg_len(i)
  // keys; column c takes part in it if seg_col(i) < 0 or seg_col(i) == c / G (its sample).
  int kvh, qrow[QB], qhead, qpos[QB], nseg;
  int seq0, len0;           // first segment
  int sfx_seq0 = 0, sfx_len = 0;   // shared-prompt decode: segments 1.. are the samples' own suffix streams
  bool store_col[QB];
  if constexpr (DECODE) {
    const int units = a.share_k ? a.S / a.share_k : a.S;       // prompts or sequences
    if (job >= units * Hkv) return;
    const int slot = job / Hkv;
    kvh = job - slot * Hkv;
    const int u = a.order ? a.order[slot] : slot;     // longest contexts first: the tail of the launch is short jobs
    if (a.share_k) {
      // the K samples of prompt u sit in the MFMA columns (next to the G query heads of the kv head): the
      // prompt's keys and values are read once for all of them, then each sample's own new tokens
      const int j = (c / G) % a.share_k;
      if (a.finished) {           // nothing to do once every sample of the prompt has ended
        bool live = false;
        for (int jj = 0; jj < a.share_k; ++jj) live |= a.finished[u * a.share_k + jj] == 0;
        if (!live) return;
      }
      qrow[0] = u * a.share_k + j;
      seq0 = u;
      len0 = a.ctx_base[u * a.share_k];
      sfx_seq0 = a.sfx_first + u * a.share_k;
      sfx_len = a.ctx_add;
      nseg = 1 + a.share_k;
      store_col[0] = c < G * a.share_k;
    } else {
      if (a.finished && a.finished[u]) return;      // an ended completion's output is never used: do not stream its cache
      qrow[0] = u;
      seq0 = a.cache_seq_of ? a.cache_seq_of[u] : u;       // rows of a compacted batch name their cache sequence
      len0 = a.ctx_base[u] + a.ctx_add;
      nseg = 1;
      store_col[0] = c < G;
    }
    qhead = kvh * G + (c % G);
    qpos[0] = 0x7fffffff;      // a decode query sees every key of its segments
  } else {
    // a.jobs lists blocks of 16 tokens, QB consecutive ones (of one sequence, the first a multiple of QB) per wave
    if (job >= a.njobs / QB * a.Hq) return;
    AttnJob jb = a.jobs[job / a.Hq * QB];
    jb.qblock /= QB;
    qhead = job % a.Hq;
    kvh = qhead / G;
    seq0 = jb.cache_seq;
#pragma unroll
    for (int b = 0; b < QB; ++b) {
      const int tok = (jb.qblock * QB + b) * 16 + c;
      store_col[b] = tok < jb.len;
      qpos[b] = min(tok, jb.len - 1);
      qrow[b] = jb.row0 + qpos[b];
    }
    len0 = min((jb.qblock + 1) * 16 * QB, jb.len);      // keys the last query of the job sees
    nseg = jb.pre_len > 0 ? 2 : 1;                      // a shared prefix is walked first
    sfx_seq0 = jb.pre_seq;
    sfx_len = jb.pre_len;
  }

  // query fragments (B operand): lane (c, g) holds q[col c][32 i + 8 g .. + 7]
  f16x8 qf[QB][KSTEPS];
  [[maybe_unused]] u32x4 qlo[QB][KSTEPS];          // precise mode: qf holds the bf16 hi halves (as bits), qlo the lo halves
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    const uint16_t* qp = a.q + ((size_t)qrow[b] * a.q_ld + qhead * HD) * (PR ? 2 : 1);
#pragma unroll
    for (int i = 0; i < KSTEPS; ++i) {
      const int d0 = 32 * i + 8 * g;
      if constexpr (PR) {
        u32x4 hi = u32x4{0, 0, 0, 0}, lo = u32x4{0, 0, 0, 0};
        if (d0 < HD) {
          const f32x4 x0 = *(const f32x4*)((const float*)qp + d0), x1 = *(const f32x4*)((const float*)qp + d0 + 4);
          SPLIT_BF16X2(x0[0], x0[1], hi[0], lo[0]);
          SPLIT_BF16X2(x0[2], x0[3], hi[1], lo[1]);
          SPLIT_BF16X2(x1[0], x1[1], hi[2], lo[2]);
          SPLIT_BF16X2(x1[2], x1[3], hi[3], lo[3]);
        }
        qf[b][i] = __builtin_bit_cast(f16x8, hi);
        qlo[b][i] = lo;
      } else {
      if (d0 < HD) qf[b][i] = *(const f16x8*)(qp + d0);
      else
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[b][i][e] = (f16_t)0.f;
      }
    }
  }
  // one 16x16x32 matrix instruction on 16-bit fragments: fp16, or bf16 in precise mode
  auto mfma = [](f16x8 x, f16x8 y, f32x4 acc) {
    if constexpr (PR) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), acc, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_f16(x, y, acc, 0, 0, 0);
  };

  // V^T fragment t (16 dims, of which lane c holds one, keys 8 g .. + 7): in a whole group of 64 dims tile 4 q + i has the dims
  // 64 q + 4 c + i, and pair p of its keys sits in unit 4 q + p, dims i in the low or high halves of the words i / 2 and 2 + i / 2
  constexpr int VG = PR ? 0 : HD / 64 * 4;        // tiles in whole groups
  auto value_frag = [](const u32x4 (&raw)[VT], int t) {
    if (t >= VG) return bf16x8_to_f16x8(raw[t]);
    const int i = t & 3;
    f16x8 r;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const uint32_t w0 = raw[(t & ~3) + p][i >> 1], w1 = raw[(t & ~3) + p][2 + (i >> 1)];
      const auto h = i & 1 ? __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w0 & 0xffff0000u), __uint_as_float(w1 & 0xffff0000u))
                           : __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w0 << 16), __uint_as_float(w1 << 16));
      r[2 * p] = (f16_t)h[0];
      r[2 * p + 1] = (f16_t)h[1];
    }
    return r;
  };
  f32x4 o[QB][VT];
  float m[QB], lsum[QB];
#pragma unroll
  for (int b = 0; b < QB; ++b) {
#pragma unroll
    for (int t = 0; t < VT; ++t) o[b][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    m[b] = -INFINITY;
    lsum[b] = 0.f;
  }

  for (int seg = 0; seg < nseg; ++seg) {
    if (seg > 0 && a.finished && a.finished[qrow[0] - (c / G) % a.share_k + seg - 1]) continue;     // ended sample: skip its stream
    // prompt pass with a shared prefix: segment 0 is the prefix (every key visible), segment 1 the sequence itself
    const bool prefix_seg = !DECODE && nseg == 2 && seg == 0;
    const int cache_seq = DECODE ? (seg == 0 ? seq0 : sfx_seq0 + seg - 1) : (prefix_seg ? sfx_seq0 : seq0);
    const int nkeys = DECODE ? (seg == 0 ? len0 : sfx_len) : (prefix_seg ? sfx_len : len0);
    const bool mine = !DECODE || seg == 0 || (c / G) % a.share_k == seg - 1;     // does column c attend to this segment
    const int cap = a.kv_cap[cache_seq];
    const long long off = a.kv_off[cache_seq];
    const uint16_t* __restrict__ st = a.kv + a.lay.stream(off, cap, kvh);
    int klimit[QB];                                                     // last visible key index for this column
#pragma unroll
    for (int b = 0; b < QB; ++b) klimit[b] = !mine ? -1 : prefix_seg ? nkeys - 1 : min(nkeys - 1, qpos[b]);

  const int nsb = (nkeys + 31) >> 5;
  // the whole next super-block (32 keys, 32 values) is requested before the current one is consumed
  auto load_sb = [&](int sb, u32x4 (&kraw)[2][KSTEPS], u32x4 (&vraw)[VT], int plane = 0) {
    const uint16_t* kb = st + (size_t)sb * 64 * HD + (plane ? a.kv_lo_off : 0);      // 32 keys, then the 32 values of the same positions
    const uint16_t* vb = kb + 32 * HD;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < KSTEPS; ++i) {
        const int chunk = 4 * i + g;
        constexpr int LAST = HD % 32 ? HD / 32 : KSTEPS;          // a step of 16 dims
        const int lane_at = PR ? ((4 * i + g) * 16 + c) * 8 : i * 512 + (c * (i == LAST ? 16 : 32) + 8 * g);
        kraw[t][i] = chunk < NCH ? ATTN_LOAD((const u32x4*)(kb + (t * 16 * HD + lane_at))) : u32x4{0, 0, 0, 0};
      }
#pragma unroll
    for (int t = 0; t < VT; ++t) vraw[t] = ATTN_LOAD((const u32x4*)(vb + ((((t * 4 + g) * 16) + c) << 3)));
  };
  u32x4 kraw[2][KSTEPS], vraw[VT];
  [[maybe_unused]] u32x4 kraw_lo[NP - 1 ? 2 : 1][KSTEPS], vraw_lo[VT];
#if ATTN_PREFETCH
  u32x4 knext[2][KSTEPS], vnext[VT];
  if (PF && sb0 < nsb) load_sb(sb0, kraw, vraw);
#endif
#if ATTN_PREFETCH2
  // decode: a second super-block in flight (the kernel is bound by bytes in flight, and registers allow it)
  u32x4 knext2[2][KSTEPS], vnext2[VT];
  // measured: head size 128 gains 4 % from it, head sizes 64 and 80 lose (fewer waves fit), 256 would spill
  constexpr bool P2 = DECODE && HD > 96 && HD <= 128 && !PR;
  if (P2 && sb0 + SPLIT < nsb) load_sb(sb0 + SPLIT, knext, vnext);
#endif
  for (int sb = sb0; sb < nsb; sb += SPLIT) {
#if ATTN_PREFETCH2
    if (P2) {
      if (sb + 2 * SPLIT < nsb) load_sb(sb + 2 * SPLIT, knext2, vnext2);
    } else if (PF) { if (sb + SPLIT < nsb) load_sb(sb + SPLIT, knext, vnext); }
    else {
      load_sb(sb, kraw, vraw);
      if constexpr (PR) load_sb(sb, kraw_lo, vraw_lo, 1);
      // Left to itself the scheduler puts requests back to save registers, for a wave more that cannot come, and the chain waits for
      // each.  A wave of four to a job, with two to a SIMD at most, asks for both planes at once (us a layer: decode of 8 sequences of
      // 600 keys, head size 64 16.6 -> 11.6, 128 27.5 -> 17.6; 300 rows of size 128 15.0 -> 10.1; not two query blocks: 9.0 -> 9.6 at 64)
      if constexpr (PR && SPLIT > 1 && QB == 1) __builtin_amdgcn_sched_barrier(0);
    }
#elif ATTN_PREFETCH
    if (sb + SPLIT < nsb) load_sb(sb + SPLIT, knext, vnext);
#else
    load_sb(sb, kraw, vraw);
#endif

    // the super-block's keys are widened once and serve every query block, and so are its values below
    f16x8 kf[2][KSTEPS];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < KSTEPS; ++i) kf[t][i] = PR ? __builtin_bit_cast(f16x8, kraw[t][i]) : bf16x8_to_f16x8(kraw[t][i]);
    [[maybe_unused]] f16x8 vwide[V_EARLY ? VT : 1];
    if constexpr (V_EARLY) {
#pragma unroll
      for (int t = 0; t < VT; ++t) vwide[t] = value_frag(vraw, t);
    }
    // straight-line code over the query blocks: their chains (MFMA -> softmax -> MFMA) are independent, and the
    // scheduler interleaves them only if no branch separates them
    f32x4 sc[QB][2];
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        sc[b][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < KSTEPS; ++i) {
          sc[b][t] = mfma(kf[t][i], qf[b][i], sc[b][t]);
          if constexpr (PR) {
            sc[b][t] = mfma(__builtin_bit_cast(f16x8, kraw_lo[t][i]), qf[b][i], sc[b][t]);
            sc[b][t] = mfma(kf[t][i], __builtin_bit_cast(f16x8, qlo[b][i]), sc[b][t]);
          }
        }
      }
    // ... and the prompt pass of one query block to a wave has its values on their way before the softmax: in precise mode one wave to
    // a job (24 sequences of 514 tokens, 32 heads of size 128 on 8: 619 -> 520 us a layer, 536 with two waves to a SIMD prescribed;
    // all requests first: 548 and more), else four (654 tokens, 8 heads of size 96 / 128 / 256: 13.5 / 14.5 / 35.4 -> 11.4 / 12.9 / 25.9
    // us, all requests first 12.3 / 17.2 / 22.8; 250 tokens, 32 heads of size 128 on 8: 9.7 -> 8.5, all first 11.6)
    if constexpr (!DECODE && QB == 1 && (!PR || SPLIT == 1)) __builtin_amdgcn_sched_barrier(0);
    // lane (c, g) now holds the scores of keys 32 sb + 8 g + 4 t + j against column c
    float p[QB][8], alpha[QB];
#pragma unroll
    for (int b = 0; b < QB; ++b) {
      float bmax = -INFINITY;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int key = sb * 32 + 8 * g + 4 * t + j;
          const float v = key <= klimit[b] ? sc[b][t][j] * a.scale : -INFINITY;
          p[b][4 * t + j] = v;
          bmax = fmaxf(bmax, v);
        }
      bmax = fmaxf(bmax, __shfl_xor(bmax, 16, WAVE));
      bmax = fmaxf(bmax, __shfl_xor(bmax, 32, WAVE));
      const float mnew = fmaxf(m[b], bmax);
      // a column that has seen no key yet (m and mnew both -inf) keeps alpha = 1 and p = 0
      alpha[b] = mnew == -INFINITY ? 1.f : __expf(m[b] - mnew);
      m[b] = mnew;
      float psum = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[b][e] = mnew == -INFINITY ? 0.f : __expf(p[b][e] - mnew);
        psum += p[b][e];
      }
      lsum[b] = lsum[b] * alpha[b] + psum;
    }
    if constexpr (PR) {
#pragma unroll
      for (int b = 0; b < QB; ++b) {
        u32x4 phi, plo;
#pragma unroll
        for (int e = 0; e < 4; ++e) SPLIT_BF16X2(p[b][2 * e], p[b][2 * e + 1], phi[e], plo[e]);
        const f16x8 pf = __builtin_bit_cast(f16x8, phi);
#pragma unroll
        for (int t = 0; t < VT; ++t) {
          const f16x8 vf = __builtin_bit_cast(f16x8, vraw[t]);
          o[b][t] *= alpha[b];
          o[b][t] = mfma(vf, pf, o[b][t]);
          o[b][t] = mfma(__builtin_bit_cast(f16x8, vraw_lo[t]), pf, o[b][t]);
          o[b][t] = mfma(vf, __builtin_bit_cast(f16x8, plo), o[b][t]);
        }
      }
    } else {
      f16x8 pf[QB];
#pragma unroll
      for (int b = 0; b < QB; ++b)
#pragma unroll
        for (int e = 0; e < 8; ++e) pf[b][e] = (f16_t)p[b][e];
      // (but for V_EARLY the values are widened here, where the keys' registers are free: with it at the top of the super-block the prompt pass of
      // head size 80 needs 202 registers instead of 188, 654 and 1300 rows of 8 heads 14.4 and 14.1 us instead of 14.0 and 13.8)
#pragma unroll
      for (int t = 0; t < VT; ++t) {
        f16x8 vf;
        if constexpr (V_EARLY) vf = vwide[t];
        else vf = value_frag(vraw, t);
#pragma unroll
        for (int b = 0; b < QB; ++b) {
          o[b][t] *= alpha[b];
          o[b][t] = mfma(vf, pf[b], o[b][t]);
        }
      }
    }
#if ATTN_PREFETCH
    if (PF) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < KSTEPS; ++i) kraw[t][i] = knext[t][i];
#pragma unroll
    for (int t = 0; t < VT; ++t) vraw[t] = vnext[t];
    }
#endif
#if ATTN_PREFETCH2
    if (P2) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < KSTEPS; ++i) knext[t][i] = knext2[t][i];
#pragma unroll
      for (int t = 0; t < VT; ++t) vnext[t] = vnext2[t];
    }
#endif
  }
  }   // segments
  // column c's 4 VT values leave for row qrow in runs of four head dims: piece t is tile t, or of a whole group of 64 dims row
  // t % 4 of its four tiles
  auto piece = [&](int b, int t) {
    if (t >= VG) return o[b][t];
    const int q = t & ~3, e = t & 3;
    return f32x4{o[b][q][e], o[b][q + 1][e], o[b][q + 2][e], o[b][q + 3][e]};
  };
  auto store = [&](int b, int t, f32x4 y) {
    u32x2 w;
    uint16_t* dst = a.out + kblk_off(qrow[b], qhead * HD + (t < VG ? 16 * (t & ~3) + 16 * g + 4 * (t & 3) : 16 * t + 4 * g), a.out_rows);
    if constexpr (PR) {
      u32x2 wl;
      SPLIT_BF16X2(y[0], y[1], w[0], wl[0]);
      SPLIT_BF16X2(y[2], y[3], w[1], wl[1]);
      *(u32x2*)(dst + a.out_lo_off) = wl;
    } else {
      w[0] = pack_f16x2(y[0], y[1]);
      w[1] = pack_f16x2(y[2], y[3]);
    }
    *(u32x2*)dst = w;
  };
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    float ls = lsum[b];
    ls += __shfl_xor(ls, 16, WAVE);
    ls += __shfl_xor(ls, 32, WAVE);
    if constexpr (SPLIT > 1) {
      extern __shared__ __attribute__((aligned(16))) unsigned char shared[];
      f32x4 (*part)[VT][64] = (f32x4 (*)[VT][64])shared;                       // [wave][16-dim tile][lane]
      float2 (*ml)[16] = (float2 (*)[16])(shared + (size_t)SPLIT * VT * 64 * 16);   // [wave][column] maximum and sum
      if (g == 0) ml[wave][c] = make_float2(m[b], ls);
      __syncthreads();
      float M = -INFINITY, L = 0.f;
#pragma unroll
      for (int w = 0; w < SPLIT; ++w) M = fmaxf(M, ml[w][c].x);
#pragma unroll
      for (int w = 0; w < SPLIT; ++w) L += ml[w][c].y * __expf(ml[w][c].x - M);
      // a wave without keys has a maximum of -inf and contributes nothing (some wave has keys: M is finite)
      const float mine = __expf(m[b] - M);
#pragma unroll
      for (int t = 0; t < VT; ++t) part[wave][t][lane] = piece(b, t) * mine;
      __syncthreads();
      const float inv = 1.0f / L;
      for (int t = wave; t < VT; t += SPLIT) {
        f32x4 y = part[0][t][lane];
#pragma unroll
        for (int w = 1; w < SPLIT; ++w) y += part[w][t][lane];
        if (store_col[b]) store(b, t, y * inv);
      }
      if (b + 1 < QB) __syncthreads();             // the next query block takes the same place
    } else {
      const float inv = 1.0f / ls;
      if (store_col[b]) {
#pragma unroll
        for (int t = 0; t < VT; ++t) store(b, t, piece(b, t) * inv);
      }
    }
  }
}

// The prompt pass of large contexts: the four waves of a block share every super-block.  Each takes a quarter of it from memory,
// widens it to fp16 and leaves it in LDS as the fragments the products want (a kilobyte each, read back linearly), while the one before
// is consumed; one barrier a super-block.  The waves differ in the query head (groups of four or two heads to a kv head), else in
// the block of 16 queries.  One wave alone streamed everything itself: keys and values crossed L2 four times and were widened
// four times (a layer of 32768 rows, us: head size 256, mean prompt 320 723 -> 235, 128 with four heads to a kv head, 640, 947 ->
// 514, 80, 384, 377 -> 325; 22700 rows of size 64 109 -> 78).  Two query blocks to a wave read LDS half as often and are slower all
// the same: 490 at 80, 897 at 128 (fewer waves, and a completion of 64 tokens leaves half of them idle).
// Masks only where the diagonal is, sums rescaled only where a maximum rose: the values are those of attention_kernel.
template <int HD>
__global__ __launch_bounds__(256) void attention_prompt_kernel(AttnArgs a, int heads_per_block) {
  constexpr int KF = HD / 32, KHALF = HD % 32 ? 1 : 0;      // key steps of 32 dims, and one of 16
  constexpr int KSTEPS = KF + KHALF, VT = HD / 16, NQ = HD / 64, VG = 4 * NQ, VR = VT - VG;
  constexpr int NKF = 2 * KF + KHALF;                        // key fragments: two to a step, the half step's two share one
  constexpr int FRAGS = NKF + VT;
  // What the waves fetch: groups of 64 value dims (four units to a lane, wave w the groups w, w + 4, ...) and single fragments, the
  // latter dealt out so that no wave has more than LEVEL units to a lane unless its groups alone are more
  constexpr int SINGLES = NKF + VR, GW = (NQ + 3) / 4;
  auto room = [](int level, int w) constexpr { const int n = level - 4 * ((NQ - w + 3) / 4); return n > 0 ? n : 0; };
  constexpr int LEVEL = [&room] {
    int level = 1;
    while (room(level, 0) + room(level, 1) + room(level, 2) + room(level, 3) < SINGLES) ++level;
    return level;
  }();
  __shared__ __attribute__((aligned(16))) uint16_t lds[2][FRAGS * 512];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int Hkv = a.lay.Hkv, G = a.Hq / Hkv;
  const int tw = 4 / heads_per_block;                        // waves along the tokens
  const int hgroups = a.Hq / heads_per_block;
  const int job = blockIdx.x / hgroups, hg = blockIdx.x - job * hgroups;
  const int qhead = hg * heads_per_block + wave % heads_per_block, kvh = qhead / G;
  const AttnJob jb = a.jobs[job * tw];
  const int q0 = (jb.qblock + wave / heads_per_block) * 16;  // the wave's first query
  const bool store_col = q0 + c < jb.len;
  const int qpos = min(q0 + c, jb.len - 1), qrow = jb.row0 + qpos;
  const int wave_keys = q0 < jb.len ? min(q0 + 16, jb.len) : 0;
  const int block_keys = min((jb.qblock + tw) * 16, jb.len);
  f16x8 qf[KSTEPS];
  const uint16_t* qp = a.q + (size_t)qrow * a.q_ld + qhead * HD;
#pragma unroll
  for (int i = 0; i < KSTEPS; ++i) {
    const int d0 = 32 * i + 8 * g;
    if (d0 < HD) qf[i] = *(const f16x8*)(qp + d0);
    else
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[i][e] = (f16_t)0.f;
  }
  f32x4 o[VT];
#pragma unroll
  for (int t = 0; t < VT; ++t) o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, lsum = 0.f;
  // this wave's single fragments: their lane offsets in a super-block and their places in LDS
  int first = 0, singles = 0;
  {
    int at = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int n = min(room(LEVEL, w), SINGLES - at);
      if (w == wave) { first = at; singles = n; }
      at += n;
    }
  }
  uint32_t from[LEVEL];
#pragma unroll
  for (int l = 0; l < LEVEL; ++l) {
    const int f = min(first + l, SINGLES - 1);
    if (f < 2 * KF) from[l] = (f >= KF ? 16 * HD + (f - KF) * 512 : f * 512) + c * 32 + 8 * g;
    else if (f < NKF) from[l] = (g >> 1) * 16 * HD + KF * 512 + c * 16 + 8 * (g & 1);
    else from[l] = 32 * HD + NQ * 2048 + (f - NKF) * 512 + lane * 8;
  }
  u32x4 group[GW > 0 ? GW : 1][4], single[LEVEL];
  const int nseg = jb.pre_len > 0 ? 2 : 1;
  int buf = 0;
  for (int seg = 0; seg < nseg; ++seg) {
    const bool prefix = nseg == 2 && seg == 0;               // a shared prompt: every key visible
    const int cache_seq = prefix ? jb.pre_seq : jb.cache_seq, nkeys = prefix ? jb.pre_len : block_keys;
    const int own_keys = prefix ? (wave_keys > 0 ? nkeys : 0) : wave_keys;
    const uint16_t* __restrict__ st = a.kv + a.lay.stream(a.kv_off[cache_seq], a.kv_cap[cache_seq], kvh);
    const int nsb = (nkeys + 31) >> 5;
    auto fetch = [&](int sb) {
      const uint16_t* kb = st + (size_t)sb * 64 * HD;
#pragma unroll
      for (int q = 0; q < GW; ++q)
        if (wave + 4 * q < NQ) {
#pragma unroll
          for (int p = 0; p < 4; ++p) group[q][p] = *(const u32x4*)(kb + (uint32_t)(32 * HD + (wave + 4 * q) * 2048 + p * 512 + lane * 8));
        }
#pragma unroll
      for (int l = 0; l < LEVEL; ++l)
        if (l < singles) single[l] = *(const u32x4*)(kb + from[l]);
    };
    auto put = [&](int to) {
#pragma unroll
      for (int q = 0; q < GW; ++q)
        if (wave + 4 * q < NQ) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            f16x8 r;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
              const uint32_t w0 = group[q][p][i >> 1], w1 = group[q][p][2 + (i >> 1)];
              const auto h = i & 1 ? __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w0 & 0xffff0000u), __uint_as_float(w1 & 0xffff0000u))
                                   : __builtin_amdgcn_cvt_pkrtz(__uint_as_float(w0 << 16), __uint_as_float(w1 << 16));
              r[2 * p] = (f16_t)h[0];
              r[2 * p + 1] = (f16_t)h[1];
            }
            *(f16x8*)(&lds[to][(NKF + 4 * (wave + 4 * q) + i) * 512 + lane * 8]) = r;
          }
        }
#pragma unroll
      for (int l = 0; l < LEVEL; ++l)
        if (l < singles) *(f16x8*)(&lds[to][(first + l < NKF ? first + l : first + l + VG) * 512 + lane * 8]) = bf16x8_to_f16x8(single[l]);
    };
    fetch(0);
    for (int sb = 0; sb < nsb; ++sb) {
      put(buf);
      if (sb + 1 < nsb) fetch(sb + 1);
      // (requests for the next super-block stay on their way across the barrier; behind it nobody reads the other buffer any more)
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      const uint16_t* fr = lds[buf] + lane * 8;
      const uint16_t* half = lds[buf] + 2 * KF * 512 + ((g & 1) * 16 + c) * 8;
      buf ^= 1;
      if (sb * 32 >= own_keys) continue;
      f32x4 sc[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        sc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < KSTEPS; ++i) {
          f16x8 kf = i < KF ? *(const f16x8*)(fr + (t * KF + i) * 512) : *(const f16x8*)(half + t * 256);
          // (lane groups without dims of the half step multiply zeros: a query of zero alone does not cancel an infinity.  32768 rows of
          // head size 80, us a layer: without this 295, zeroed here 296, zeros read from LDS instead 299)
          if (i >= KF && g >= 2) kf = f16x8{};
          sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qf[i], sc[t], 0, 0, 0);
        }
      }
      const int klimit = prefix ? nkeys - 1 : qpos;
      float p[8], bmax = -INFINITY;
#pragma unroll
      for (int e = 0; e < 8; ++e) p[e] = sc[e >> 2][e & 3] * a.scale;
      if (sb * 32 + 31 > (prefix ? nkeys - 1 : q0)) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (sb * 32 + 8 * g + e > klimit) p[e] = -INFINITY;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) bmax = fmaxf(bmax, p[e]);
      bmax = fmaxf(bmax, __shfl_xor(bmax, 16, WAVE));
      bmax = fmaxf(bmax, __shfl_xor(bmax, 32, WAVE));
      const float mnew = fmaxf(m, bmax);
      const bool rose = mnew > m;
      // a column that has seen no key yet (m and mnew both -inf) keeps alpha = 1 and p = 0
      const float alpha = mnew == -INFINITY ? 1.f : __expf(m - mnew);
      m = mnew;
      float psum = 0.f;
      f16x8 pf;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        p[e] = mnew == -INFINITY ? 0.f : __expf(p[e] - mnew);
        psum += p[e];
        pf[e] = (f16_t)p[e];
      }
      lsum = lsum * alpha + psum;
      if (__any(rose)) {
#pragma unroll
        for (int t = 0; t < VT; ++t) o[t] *= alpha;
      }
#pragma unroll
      for (int t = 0; t < VT; ++t) o[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(*(const f16x8*)(fr + (NKF + t) * 512), pf, o[t], 0, 0, 0);
    }
  }
  lsum += __shfl_xor(lsum, 16, WAVE);
  lsum += __shfl_xor(lsum, 32, WAVE);
  const float inv = 1.0f / lsum;
  if (!store_col) return;
#pragma unroll
  for (int t = 0; t < VT; ++t) {
    const int q = t & ~3, e = t & 3;
    const f32x4 y = (t >= VG ? o[t] : f32x4{o[q][e], o[q + 1][e], o[q + 2][e], o[q + 3][e]}) * inv;
    u32x2 w;
    w[0] = pack_f16x2(y[0], y[1]);
    w[1] = pack_f16x2(y[2], y[3]);
    *(u32x2*)(a.out + kblk_off(qrow, qhead * HD + (t < VG ? 16 * q + 16 * g + 4 * e : 16 * t + 4 * g), a.out_rows)) = w;
  }
}

template <int HD, bool DECODE, int QB, bool PR, int SPLIT>
hipError_t launch(const AttnArgs& a, int jobs, hipStream_t s) {
  constexpr int lds_bytes = SPLIT > 1 ? SPLIT * (HD / 16 * 64 * 16 + 16 * (int)sizeof(float2)) : 0;
  if constexpr (lds_bytes > 65536) {
    static bool configured_on[64] = {};       // once per device (a repeated call is harmless, so no lock)
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!configured_on[dev]) {
      hipError_t e = hipFuncSetAttribute((const void*)attention_kernel<HD, DECODE, QB, PR, SPLIT>, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
      if (e != hipSuccess) return e;
      configured_on[dev] = true;
    }
  }
  const dim3 grid(SPLIT > 1 ? jobs : (jobs + 3) / 4), block(SPLIT > 4 ? SPLIT * 64 : 256);
  hipLaunchKernelGGL((attention_kernel<HD, DECODE, QB, PR, SPLIT>), grid, block, lds_bytes, s, a);
  return hipGetLastError();
}
template <int HD, bool DECODE, int QB, bool PR>
hipError_t launch_split(const AttnArgs& a, int jobs, hipStream_t s) {
  if constexpr (DECODE) {
    // (eight waves to a job leave a wave 256 registers: too few for the widest head and for precise mode)
    if (a.split >= 8 && HD <= 128 && !PR) return launch<HD, DECODE, QB, PR, (HD <= 128 && !PR) ? 8 : 4>(a, jobs, s);
  }
  if (a.split >= 4) return launch<HD, DECODE, QB, PR, 4>(a, jobs, s);
  if constexpr (DECODE || PR) return launch<HD, DECODE, QB, PR, 1>(a, jobs, s);
  return hipErrorInvalidValue;
}
template <bool DECODE, int QB>
hipError_t dispatch(const AttnArgs& a, int jobs, hipStream_t s) {
  if (jobs <= 0) return hipSuccess;
  if (a.precise) {
    switch (a.lay.h) {
#define CASE(H) case H: return launch_split<H, DECODE, (QB > 1 && H > 80) ? 1 : QB, true>(a, jobs, s);
      CASE(16) CASE(32) CASE(48) CASE(64) CASE(80) CASE(96) CASE(112) CASE(128)
#undef CASE
      default: return hipErrorInvalidValue;     // head size 256 would not fit the register file with two planes
    }
  }
  switch (a.lay.h) {
#define CASE(H) case H: return launch_split<H, DECODE, (QB > 1 && H > 80) ? 1 : QB, false>(a, jobs, s);
    CASE(16) CASE(32) CASE(48) CASE(64) CASE(80) CASE(96) CASE(112) CASE(128) CASE(256)
#undef CASE
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t rl_attention_decode(const AttnArgs& a, hipStream_t s) {
  if (a.share_k && (a.S % a.share_k != 0 || a.share_k * (a.Hq / a.lay.Hkv) > 16)) return hipErrorInvalidValue;
  return dispatch<true, 1>(a, (a.share_k ? a.S / a.share_k : a.S) * a.lay.Hkv, s);
}
// Waves to a decode job: by what the context can hold, so that a sequence's sums do not depend on the batch it is in.  Where
// the jobs alone give a SIMD a wave or two (wide heads need fewer, they hold more in registers), sharing one only costs the
// meeting in LDS.  Measured, one wave / four waves to a job, the kernel alone: 128 jobs at head size 256 50 / 21 us, 2048 at head
// size 64 37.8 / 35.9 us, 2048 at head size 128 125 / 148 us.  A decode layer on either side of the borders (us, 256 and 1500 keys):
// twice the upper one, one wave / four: 1024 jobs of size 256 127 / 144 and 324 / 320, 3264 of size 80 155 / 157 and 345 / 337; twice
// the lower one, four waves / eight: 1024 of size 64 50 / 49 and 100 / 96, 800 of size 80 102 / 110 and 150 / 158, 512 of size 128
// 176 / 221 and 223 / 294.  Of head sizes 80 and 96 a CU holds one block of eight waves: they pay while every job has a CU (the kernel
// alone, four / eight, 1000 and 2000 keys: 224 jobs of size 80 17.2 / 17.4 and 28.6 / 27.3 us, 256 18.0 / 18.4 and 29.5 / 30.2, 288
// 22.6 / 28.2 and 37.6 / 45.9; of size 96 192 jobs 18.6 / 17.3 and 30.3 / 27.9, 256 21.4 / 20.8 and 35.2 / 34.9, 288 27.4 / 31.5 and
// 47.4 / 51.9).  Eight waves leave a wave 256 registers, in which the super-blocks of wider heads hardly fit (300 and 2000 keys: 64 jobs
// of size 128 10.3 / 11.0 and 32.2 / 30.4, 128 10.7 / 12.0 and 34.3 / 33.2, 192 12.0 / 13.3 and 36.6 / 42.8): half as many there.
int rl_attention_decode_split(long long cap_jobs, int h) {
  const long long size = cap_jobs * (h > 64 ? h : 64);
  return size <= (h <= 64 ? 32768 : h <= 96 ? 256 * h : 16384) ? 8 : size <= 131072 ? 4 : 1;
}
// The same for a prompt pass of at most cap_rows rows: up to four jobs a CU (654 rows of 8 heads of size 256: 57 ->
// 21 us a layer).  A layer of prompts of 500 / 128 tokens, the waves of a block sharing super-blocks against sharing jobs (us): 256 jobs
// at 1B width 122 / 101 against 107 / 99, at 2.8B 156 / 105 and 150 / 104, at 410M 58 / 49 and 50 / 47; 512 jobs at 1B 171 / 151 and
// 167 / 155, at 410M 74 / 66 and 69 / 66, at 8B 280 / 190 both; 1024 jobs at 1B 277 / 262 and 297 / 275, else within 1 %; 2048 jobs
// 495 / 478 and 566 / 517, at 2.8B 451 / 448 and 467 / 465, at 8B 479 / 467 and 489 / 472.  (The border is by what a context can
// hold; calls that fill half of it lie where sharing jobs is ahead.)
int rl_attention_prefill_split(int cap_rows, int Hq, int h) {
  const long long jobs = (long long)((cap_rows + 15) / 16) * Hq / (h <= 80 ? 2 : 1);
  return jobs <= 1024 ? 4 : 1;
}
// waves of a block of attention_prompt_kernel that differ in the query head
static int prompt_heads(int G) { return G % 4 == 0 ? 4 : G % 2 == 0 ? 2 : 1; }
int rl_attention_prefill_jobs(int cap_rows, int Hq, int Hkv, int h, int precise) {
  if (precise || rl_attention_prefill_split(cap_rows, Hq, h) > 1) return h <= 80 ? 2 : 1;
  return 4 / prompt_heads(Hq / Hkv);
}
hipError_t rl_attention_prefill(const AttnArgs& a, hipStream_t s) {
  if (a.precise || a.split > 1) {
    const int qb = a.lay.h <= 80 ? 2 : 1;
    if (a.njobs % qb != 0) return hipErrorInvalidValue;
    return dispatch<false, 2>(a, a.njobs / qb * a.Hq, s);
  }
  if (a.njobs <= 0) return hipSuccess;
  const int hb = prompt_heads(a.Hq / a.lay.Hkv), per = 4 / hb;
  if (a.njobs % per != 0) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((long long)a.njobs / per * (a.Hq / hb)));
  switch (a.lay.h) {
#define CASE(H) case H: hipLaunchKernelGGL((attention_prompt_kernel<H>), grid, dim3(256), 0, s, a, hb); break;
    CASE(16) CASE(32) CASE(48) CASE(64) CASE(80) CASE(96) CASE(112) CASE(128) CASE(256)
#undef CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
