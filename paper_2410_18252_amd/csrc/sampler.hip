// Second phase of the fused LM-head sampler and scorer.  The LM-head GEMM (EPI_LMHEAD) leaves, per
// row and per group of 64 vocabulary columns, the max and the sum of exp of the tempered logits --
// never the logits or the probabilities.  Here one block per row combines them into log Z, walks
// the group sums in ascending vocabulary order (fp64) to find the group in which the CDF crosses
// u, recomputes that group's 64 logits and finishes the scan inside it (one column per lane).
#include "kernels.h"

namespace {

__device__ __forceinline__ double wave_incl_scan(double v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double t = __shfl_up(v, o, WAVE);
    if (lane >= o) v += t;
  }
  return v;
}

// log Z of one row from its partials, one wave, coalesced; all lanes get M, the largest logit, and Z, relative to it.
__device__ __forceinline__ void row_logz(const float2* p, int ngroups, int lane, float& M, double& Z) {
  float mx = -INFINITY;
  for (int g = lane; g < ngroups; g += 64) mx = fmaxf(mx, p[g].x);
  M = wave_max(mx);
  double z = 0.0;
  for (int g = lane; g < ngroups; g += 64) z += (double)(p[g].y * __expf(p[g].x - M));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) z += __shfl_xor(z, o, WAVE);
  Z = z;
}

// One block of four waves per row.  The stage is a chain of short passes that wait for memory (the row's partials, then
// 64 lines of the LM head per K block), so the waves divide both: 256 contiguous runs of groups instead of 64, and a quarter
// of the K blocks each (2.8B width, 64 rows: 72 us with one wave per row).
__global__ __launch_bounds__(256) void sample_kernel(SampleArgs a) {
  constexpr int NW = 4;
  __shared__ float s_max[NW];
  __shared__ double s_sum[NW], s_base;
  __shared__ int s_first[NW];
  __shared__ float s_logit[NW][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = blockIdx.x;
  const size_t idx = (size_t)(a.io_index ? a.io_index[row] : row) * a.io_stride + a.io_add;
  // the token's row of the embedding is where the next step starts: taken along here (first .. by step, 8 dims each), it is a launch
  // and a hand-over less per step
  auto embed = [&](int tok, int first, int step) {
    if (a.x == nullptr) return;
    for (int i = 8 * first; i < a.d; i += 8 * step) widen_bf16x8(a.x + (size_t)row * a.d + i, *(const u32x4*)(a.embed + (size_t)tok * a.d + i));
  };
  if (a.finished && a.finished[row]) {            // the completion ended at an earlier step
    if (threadIdx.x == 0) {
      a.tokens[idx] = a.eos;
      a.logprobs[idx] = 0.f;
      if (a.next_token) a.next_token[row] = a.eos;
    }
    embed(a.eos, threadIdx.x, 256);
    return;
  }
  float u = a.greedy ? 0.f : a.uniforms[idx];
  if (!(u >= 0.f && u < 1.f)) {
    if (threadIdx.x == 0) atomicOr(a.status, RLGEN_FAULT_UNIFORM);
    u = (u >= 1.f) ? 0.99999994f : 0.f;
  }
  int forced = a.forced ? a.forced[idx] : -1;
  if (forced >= a.vocab) {
    if (threadIdx.x == 0) atomicOr(a.status, RLGEN_FAULT_TOKEN);
    forced = a.vocab - 1;
  }
  const float2* p = a.partial + (size_t)row * a.ngroups;
  // threads own contiguous runs of groups, in ascending order; the first HELD of a run stay in registers
  constexpr int HELD = 8;                         // vocabularies up to 131072
  const int per = (a.ngroups + 255) / 256;
  const int g0 = min((int)threadIdx.x * per, a.ngroups), n = min(g0 + per, a.ngroups) - g0;
  float2 held[HELD];
#pragma unroll
  for (int i = 0; i < HELD; ++i) held[i] = i < n ? p[g0 + i] : make_float2(-INFINITY, 0.f);
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < HELD; ++i) mx = fmaxf(mx, held[i].x);
  for (int i = HELD; i < n; ++i) mx = fmaxf(mx, p[g0 + i].x);
  mx = wave_max(mx);
  if (lane == 0) s_max[wave] = mx;
  __syncthreads();
  const float M = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
  auto weight = [&](const float2& q) { return (double)(q.y * __expf(q.x - M)); };
  double own = 0.0;
#pragma unroll
  for (int i = 0; i < HELD; ++i)
    if (i < n) own += weight(held[i]);
  for (int i = HELD; i < n; ++i) own += weight(p[g0 + i]);
  const double incl = wave_incl_scan(own, lane);
  if (lane == 63) s_sum[wave] = incl;
  __syncthreads();
  double before = 0.0, Z = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if (w < wave) before += s_sum[w];
    Z += s_sum[w];
  }
  const double logZ = (double)M + log(Z);
  const double target = (double)u * Z;

  // the first group in which the CDF crosses the target (greedy: that holds the largest logit)
  int gsel = 0x7fffffff;
  double base = 0.0;
  {
    double r = before + (incl - own);             // exclusive prefix of this thread
    auto look = [&](const float2& q, int g) {
      const double w = weight(q);
      if (gsel == 0x7fffffff && (a.greedy ? q.x == M : r + w > target)) {
        gsel = g;
        base = r;
      }
      r += w;
    };
#pragma unroll
    for (int i = 0; i < HELD; ++i)
      if (i < n) look(held[i], g0 + i);
    for (int i = HELD; i < n; ++i) look(p[g0 + i], g0 + i);
  }
  int gmin = gsel;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) gmin = min(gmin, __shfl_xor(gmin, o, WAVE));
  if (lane == 0) s_first[wave] = gmin;
  __syncthreads();
  gmin = min(min(s_first[0], s_first[1]), min(s_first[2], s_first[3]));
  if (gmin == 0x7fffffff) {
    // u < 1 is always crossed unless rounding or a NaN stands in the way: stay in bounds
    gmin = a.greedy ? 0 : a.ngroups - 1;
    if (threadIdx.x == 0) s_base = -INFINITY;      // no column is hit: the last one of positive probability
  } else if (gsel == gmin) {
    s_base = base;
  }
  if (forced >= 0) gmin = forced >> 6;

  // Recompute the 64 tempered logits of group gmin, wave w taking the K blocks w, w + 4, ...  Both operands are K-block
  // major (a column's 64 K values are one 128-byte line), so the lanes work in groups of eight: lane l reads the 16-byte
  // chunk l % 8 of the lines of columns l / 8 + 8 j, j = 0..7 -- every wave-wide load is eight whole lines -- and the
  // eight partial sums of a column are added across its lane group at the end, then those of the four waves.
  const int chunk = lane & 7, cgroup = lane >> 3;
  float part[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) part[j] = 0.f;
  // Two K blocks per trip: their 18 loads are requested before the first product, so a trip waits for memory once.
  constexpr int KB = 2;
  for (int kb = 64 * wave; kb < a.d; kb += 64 * NW * KB) {
    u32x4 hv[KB], hl[KB], wv[KB][8];
    bool live[KB];
#pragma unroll
    for (int q = 0; q < KB; ++q) {
      const int k = kb + 64 * NW * q + 8 * chunk;
      live[q] = k < a.d;                   // d is a multiple of 32: the last K block may be half full
      if (!live[q]) continue;
      hv[q] = *(const u32x4*)(a.hfin + kblk_off(row, k, a.R));
      if (a.precise) hl[q] = *(const u32x4*)(a.hfin + a.hfin_lo_off + kblk_off(row, k, a.R));
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int c = min(gmin * 64 + cgroup + 8 * j, a.vocab - 1);       // columns past the end are left out below
        wv[q][j] = *(const u32x4*)(a.lm_head + kblk_off(c, k, a.vocab));
      }
    }
#pragma unroll
    for (int q = 0; q < KB; ++q) {
      if (!live[q]) continue;
      float h[8];
      if (a.precise) {
        // the normalised row as bf16 hi/lo pairs: their sum is formed in fp32, where it is exact
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          h[2 * e] = __uint_as_float(hv[q][e] << 16) + __uint_as_float(hl[q][e] << 16);
          h[2 * e + 1] = __uint_as_float(hv[q][e] & 0xffff0000u) + __uint_as_float(hl[q][e] & 0xffff0000u);
        }
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          h[2 * e] = f16_bits_to_f32((uint16_t)(hv[q][e] & 0xffffu));
          h[2 * e + 1] = f16_bits_to_f32((uint16_t)(hv[q][e] >> 16));
        }
      }
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (a.precise) {                    // bf16 weights
            part[j] += __uint_as_float(wv[q][j][e] << 16) * h[2 * e];
            part[j] += __uint_as_float(wv[q][j][e] & 0xffff0000u) * h[2 * e + 1];
          } else {
            part[j] += f16_bits_to_f32((uint16_t)(wv[q][j][e] & 0xffffu)) * h[2 * e];
            part[j] += f16_bits_to_f32((uint16_t)(wv[q][j][e] >> 16)) * h[2 * e + 1];
          }
        }
    }
  }
  // lane L ends up with column 64 gmin + L = cgroup' + 8 j' for cgroup' = L % 8, j' = L / 8: the sum of lane group cgroup'
  float acc = 0.f;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    float v = part[j];
    v += __shfl_xor(v, 1, WAVE);
    v += __shfl_xor(v, 2, WAVE);
    v += __shfl_xor(v, 4, WAVE);
    const float t = __shfl(v, 8 * (lane & 7), WAVE);
    if ((lane >> 3) == j) acc = t;
  }
  s_logit[wave][lane] = acc;
  __syncthreads();
  if (wave != 0) return;
  acc = (s_logit[0][lane] + s_logit[1][lane]) + (s_logit[2][lane] + s_logit[3][lane]);
  base = s_base;
  const int col = gmin * 64 + lane;
  const float logit = col < a.vocab ? acc / a.temperature : -INFINITY;
  int tok;
  if (forced >= 0) {
    tok = forced;
  } else if (a.greedy) {
    const float best = wave_max(logit);
    const unsigned long long at = __ballot(logit == best);
    tok = min(gmin * 64 + (at ? __ffsll((long long)at) - 1 : 0), a.vocab - 1);
  } else {
    const double e = (logit == -INFINITY) ? 0.0 : (double)__expf(logit - M);
    const double cum = base + wave_incl_scan(e, lane);
    const unsigned long long hit = __ballot(cum > target && e > 0.0);
    const unsigned long long pos = __ballot(e > 0.0);
    int j;
    if (hit) j = __ffsll((long long)hit) - 1;
    else if (pos) j = 63 - __clzll((long long)pos);   // rounding left the crossing outside: last positive column
    else j = 0;
    tok = min(gmin * 64 + j, a.vocab - 1);
  }
  const float ltok = __shfl(logit, tok & 63, WAVE);
  if (lane == 0) {
    a.tokens[idx] = tok;
    a.logprobs[idx] = (float)((double)ltok - logZ);
    if (a.next_token) a.next_token[row] = tok;
    if (a.finished && tok == a.eos) a.finished[row] = 1;
  }
  embed(tok, lane, 64);
}

__global__ __launch_bounds__(256) void score_finalize_kernel(const float2* partial, int ngroups, const float* target_logit,
                                                            const int* out_index, float* out, int R) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= R) return;
  float M;
  double Z;
  row_logz(partial + (size_t)row * ngroups, ngroups, lane, M, Z);
  if (lane == 0) out[out_index[row]] = (float)((double)target_logit[row] - ((double)M + log(Z)));
}

}  // namespace

hipError_t rl_sample(const SampleArgs& a, hipStream_t s) {
  if (a.R <= 0) return hipSuccess;
  hipLaunchKernelGGL(sample_kernel, dim3(a.R), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t rl_score_finalize(const float2* partial, int ngroups, const float* target_logit, const int* out_index,
                             float* out, int R, hipStream_t s) {
  if (R <= 0) return hipSuccess;
  hipLaunchKernelGGL(score_finalize_kernel, dim3((R + 3) / 4), dim3(256), 0, s, partial, ngroups, target_logit, out_index, out, R);
  return hipGetLastError();
}
