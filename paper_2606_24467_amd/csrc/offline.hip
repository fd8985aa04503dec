// Offline analyses of CompressKV (include/compresskv_offline.h): the SRH
// score of every head (section 3.2, equation 1), each layer's SRH set
// (section 3.3) and the layer budgets from the layers' eviction errors
// (section 3.4; the errors themselves are computed in decode_error.hip).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "../../include/compresskv_offline.h"
#include "api_common.h"

namespace ckv {

struct SrhArgs {
  const float *attn;
  const int32_t *gen, *ctx, *spans;
  float *scores;
  int32_t S, N, H, L;
};

constexpr int kSrhHeads = 2;        // heads per workgroup
constexpr int kSrhSplit = 8;        // waves per head
constexpr int kSrhBatch = 4;        // answer steps whose span loads a wave issues together
constexpr int kSrhTokens = 8;       // span tokens whose loads a lane of the test issues together
constexpr int kSrhPairs = 2048;     // (sample, step) pairs tested per pass

// Bound by latency (a few answer steps per head, each a short run of a row of
// its own), so every chain is kept short.  A workgroup of 16 waves covers 2
// consecutive heads; two workgroups share a CU, so that the 512 of 1024 heads
// run in one round (every workgroup tests all pairs, a second round would do
// that again).  That needs at most 64 VGPRs and 80 SGPRs: the uniform row
// pointers of 4 spans a batch leave it at 66 SGPRs, those of 8 take 90, and one
// workgroup runs on a CU.  Per block of (sample, step) pairs:
//   - each pair is tested by as many lanes as 1024 threads give it (1 to 64),
//     strided over the span's tokens, 8 tokens in flight a lane (with one lane
//     a pair the walk over the tokens is what the call waits for), and joined
//     by a ballot;
//   - the answer steps are listed in LDS in step order (ballot, popcount and
//     a prefix over the 64-pair chunks);
//   - the eight waves of a head take every eighth entry of the list, load 4
//     spans together (lanes over positions) and add them per lane in fp64 in
//     list order: one butterfly per head and wave at the end.  The loads are
//     unconditional, past a span's end on its last position: guarded by the
//     span's length, the compiler puts a load's conversion to fp64, and so the
//     wait for it, before the next load.
// Score call alone in us, for (samples x steps, heads, span, share of answer
// steps); "walk" is one thread per pair, no list, 4 heads a workgroup and a
// butterfly per step, "guarded" this kernel with 16 guarded loads a batch and
// one token at a time:
//                                     walk  guarded     now
//   4 x 32,   1024,   32 tokens, 1/2    32.9     20.0    10.8
//   64 x 64,  1024,   32 tokens, all   648.9    724.2   294.5
//   1 x 512,  1024,  400 tokens, 0.3   110.2    194.1    67.4
//   22 x 99,   448, 1611 tokens, 0.87 2072.5   3374.4  1337.1
// The waves' totals are added in wave order, so the result does not depend on
// scheduling.
__global__ __launch_bounds__(64 * kSrhHeads * kSrhSplit) void srh_score_kernel(const SrhArgs a) {
  constexpr int NW = kSrhHeads * kSrhSplit, NT = 64 * NW, CH = kSrhPairs / 64;
  static_assert(kSrhPairs % 64 == 0, "whole 64-pair chunks");
  __shared__ int a0_s[kSrhPairs], n_s[kSrhPairs];   // span of each pair; length 0: no answer step
  __shared__ uint16_t list_s[kSrhPairs];            // the block's answer steps, ascending
  __shared__ int cnt_s[CH];                         // answer steps per 64-pair chunk
  __shared__ double part_s[NW];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int h = blockIdx.x * kSrhHeads + wave / kSrhSplit, sub = wave % kSrhSplit;
  const int SN = a.S * a.N;
  double acc = 0.0;
  for (int p0 = 0; p0 < SN; p0 += kSrhPairs) {
    const int np = min(kSrhPairs, SN - p0);
    int lpp = 1;                                    // lanes per pair, a power of two
    while (lpp < 64 && 2 * lpp * np <= NT) lpp *= 2;
    const int sl = lane & (lpp - 1), lane0 = lane - sl;
    const uint64_t group = (lpp == 64 ? ~0ull : (1ull << lpp) - 1) << lane0;
    for (int qb = 0; qb < np; qb += NT / lpp) {     // uniform: every lane takes part in the ballot
      const int q = qb + tid / lpp;
      int a0 = 0, n = 0;
      bool hit = false;
      if (q < np) {
        const int p = p0 + q, s = p / a.N;
        const int32_t y = a.gen[p];
        a0 = a.spans[2 * s];
        n = a.spans[2 * s + 1];
        const int32_t *tok = a.ctx + (int64_t)s * a.L + a0;
        int j = sl;
        for (; j - sl + kSrhTokens * lpp <= n; j += kSrhTokens * lpp) {
          int32_t x[kSrhTokens];
#pragma unroll
          for (int u = 0; u < kSrhTokens; ++u) x[u] = tok[j + u * lpp];
#pragma unroll
          for (int u = 0; u < kSrhTokens; ++u) hit |= (x[u] == y);
        }
        if (j - sl < n) {   // the rest, with the last token in the place of those past it
          int32_t x[kSrhTokens];
#pragma unroll
          for (int u = 0; u < kSrhTokens; ++u) x[u] = tok[min(j + u * lpp, n - 1)];
#pragma unroll
          for (int u = 0; u < kSrhTokens; ++u) hit |= (x[u] == y);
        }
      }
      const bool any = (__ballot(hit) & group) != 0;
      if (q < np && sl == 0) {
        a0_s[q] = a0;
        n_s[q] = any ? n : 0;
      }
    }
    __syncthreads();
    for (int ch = wave; ch < CH; ch += NW) {
      const int q = 64 * ch + lane;
      const uint64_t m = __ballot(q < np && n_s[q] > 0);
      if (lane == 0) cnt_s[ch] = __popcll(m);
    }
    __syncthreads();
    int nh = 0;                                     // answer steps of the block
    for (int ch = 0; 64 * ch < np; ++ch) {
      if (ch % NW == wave) {
        const int q = 64 * ch + lane;
        const bool hit = q < np && n_s[q] > 0;
        const uint64_t m = __ballot(hit);
        if (hit) list_s[nh + __popcll(m & ((1ull << lane) - 1))] = (uint16_t)q;
      }
      nh += cnt_s[ch];
    }
    nh = __builtin_amdgcn_readfirstlane(nh);
    __syncthreads();
    if (h < a.H) {
      for (int i0 = sub; i0 < nh; i0 += kSrhSplit * kSrhBatch) {
        const float *row[kSrhBatch];
        int len[kSrhBatch], nmax = 0;
#pragma unroll
        for (int b = 0; b < kSrhBatch; ++b) {
          const int i = i0 + kSrhSplit * b;
          const int q = __builtin_amdgcn_readfirstlane((int)list_s[min(i, nh - 1)]);
          const int n = __builtin_amdgcn_readfirstlane(n_s[q]);   // >= 1: the list's entries
          const int a0 = __builtin_amdgcn_readfirstlane(a0_s[q]);
          len[b] = i < nh ? n : 0;
          row[b] = a.attn + ((int64_t)(p0 + q) * a.H + h) * (int64_t)a.L + a0;
          nmax = max(nmax, len[b]);
        }
        for (int j0 = 0; j0 < nmax; j0 += 64) {
          const int j = j0 + lane;
          float x[kSrhBatch];
#pragma unroll
          for (int b = 0; b < kSrhBatch; ++b) x[b] = row[b][min(j, max(len[b], 1) - 1)];
#pragma unroll
          for (int b = 0; b < kSrhBatch; ++b) acc += (double)(j < len[b] ? x[b] : 0.f);
        }
      }
    }
    __syncthreads();   // the spans and the list are rewritten by the next block
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o);
  if (lane == 0) part_s[wave] = acc;
  __syncthreads();
  if (sub == 0 && lane == 0 && h < a.H) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kSrhSplit; ++w) t += part_s[wave + w];
    a.scores[h] = (float)t;
  }
}

// One workgroup per layer, one thread per head: a head's rank is the number of
// heads with a higher score or an equal score and a lower index.
__global__ __launch_bounds__(1024) void select_srh_kernel(const float *scores, int hp, int top_k,
                                                          uint8_t *mask) {
  const int l = blockIdx.x, h = threadIdx.x;
  if (h >= hp) return;
  const float *sc = scores + (int64_t)l * hp;
  const float me = sc[h];
  int rank = 0;
  for (int o = 0; o < hp; ++o) {
    const float x = sc[o];
    rank += (x > me) || (x == me && o < h);
  }
  mask[(int64_t)l * hp + h] = rank < top_k ? 1 : 0;
}

}  // namespace ckv

using ckv_api::fail;
using ckv_api::ok;

extern "C" {

int compresskv_srh_scores(const ckv_srh_problem *p, const float *attn, const int32_t *gen_tokens,
                          const int32_t *ctx_tokens, const int32_t *spans, float *scores,
                          void *stream) {
  if (!p) return fail(CKV_INVALID_ARGUMENT, "problem is NULL");
  if (p->n_samples < 1 || p->n_steps < 1 || p->n_heads < 1 || p->ctx_len < 1)
    return fail(CKV_INVALID_ARGUMENT, "n_samples, n_steps, n_heads and ctx_len must be >= 1");
  if (!p->spans_host) return fail(CKV_INVALID_ARGUMENT, "spans_host is NULL");
  for (int s = 0; s < p->n_samples; ++s) {
    const int a0 = p->spans_host[2 * s], n = p->spans_host[2 * s + 1];
    if (a0 < 0 || n < 1 || (int64_t)a0 + n > p->ctx_len)
      return fail(CKV_INVALID_ARGUMENT, "sample %d: span (%d, %d) outside [0, %d)", s, a0, n,
                  p->ctx_len);
  }
  const void *ptrs[] = {attn, gen_tokens, ctx_tokens, spans, scores};
  const char *names[] = {"attn", "gen_tokens", "ctx_tokens", "spans", "scores"};
  for (int i = 0; i < 5; ++i) {
    if (!ptrs[i]) return fail(CKV_INVALID_ARGUMENT, "%s is NULL", names[i]);
    if (!ckv_api::aligned(ptrs[i], 4))
      return fail(CKV_UNSUPPORTED, "%s must be 4-byte aligned", names[i]);
  }
  ckv::SrhArgs a{attn, gen_tokens, ctx_tokens, spans, scores,
                 p->n_samples, p->n_steps, p->n_heads, p->ctx_len};
  hipLaunchKernelGGL(ckv::srh_score_kernel, dim3((p->n_heads + ckv::kSrhHeads - 1) / ckv::kSrhHeads),
                     dim3(64 * ckv::kSrhHeads * ckv::kSrhSplit), 0, (hipStream_t)stream, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess)
    return fail(CKV_HIP_ERROR, "srh score launch failed: %s", hipGetErrorString(e));
  return ok();
}

int compresskv_select_srh(int32_t n_layers, int32_t heads_per_layer, const float *scores,
                          int32_t top_k, uint8_t *srh_mask, void *stream) {
  if (n_layers < 1 || n_layers > 65535)
    return fail(CKV_INVALID_ARGUMENT, "n_layers must be in [1, 65535] (got %d)", n_layers);
  if (heads_per_layer < 1 || heads_per_layer > 1024)
    return fail(CKV_UNSUPPORTED, "heads_per_layer must be in [1, 1024] (got %d)",
                heads_per_layer);
  if (top_k < 1 || top_k > heads_per_layer)
    return fail(CKV_INVALID_ARGUMENT, "top_k must be in [1, heads_per_layer] (got %d)", top_k);
  if (!scores || !srh_mask) return fail(CKV_INVALID_ARGUMENT, "scores and srh_mask are required");
  if (!ckv_api::aligned(scores, 4)) return fail(CKV_UNSUPPORTED, "scores must be 4-byte aligned");
  hipLaunchKernelGGL(ckv::select_srh_kernel, dim3(n_layers), dim3(heads_per_layer), 0,
                     (hipStream_t)stream, scores, (int)heads_per_layer, (int)top_k, srh_mask);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess)
    return fail(CKV_HIP_ERROR, "select srh launch failed: %s", hipGetErrorString(e));
  return ok();
}

int compresskv_allocate_budgets(int32_t n_layers, const float *errors_host, int64_t total,
                                int32_t min_budget, int32_t max_budget, int32_t *budgets_host) {
  if (n_layers < 1) return fail(CKV_INVALID_ARGUMENT, "n_layers must be >= 1 (got %d)", n_layers);
  if (!errors_host || !budgets_host)
    return fail(CKV_INVALID_ARGUMENT, "errors_host and budgets_host are required");
  if (min_budget < 1 || max_budget < min_budget)
    return fail(CKV_INVALID_ARGUMENT, "need 1 <= min_budget <= max_budget");
  const int n = n_layers;
  if (total < (int64_t)n * min_budget || total > (int64_t)n * max_budget)
    return fail(CKV_INVALID_ARGUMENT, "total must lie in [n_layers * min, n_layers * max]");
  double esum = 0.0;
  for (int i = 0; i < n; ++i) {
    const float e = errors_host[i];
    if (!std::isfinite(e) || e < 0.f)
      return fail(CKV_INVALID_ARGUMENT, "layer %d: error must be finite and >= 0", i);
    esum += e;
  }
  // normalised errors (a layer set of all-zero errors shares evenly)
  std::vector<double> w(n), share(n, 0.0);
  for (int i = 0; i < n; ++i) w[i] = esum > 0.0 ? (double)errors_host[i] / esum : 0.0;
  std::vector<char> capped(n, 0);
  for (;;) {
    int n_free = 0;
    double wsum = 0.0;
    for (int i = 0; i < n; ++i)
      if (!capped[i]) {
        ++n_free;
        wsum += w[i];
      }
    const double rest =
        (double)(total - (int64_t)(n - n_free) * max_budget - (int64_t)n_free * min_budget);
    bool over = false;
    for (int i = 0; i < n; ++i) {
      if (capped[i]) continue;
      share[i] = wsum > 0.0 ? rest * w[i] / wsum : rest / n_free;
      over |= (min_budget + share[i] > max_budget);
    }
    if (!over) break;
    for (int i = 0; i < n; ++i)
      if (!capped[i] && min_budget + share[i] > max_budget) capped[i] = 1;
  }
  int64_t used = 0;
  std::vector<int> order;
  for (int i = 0; i < n; ++i) {
    if (capped[i]) {
      budgets_host[i] = max_budget;
    } else {
      budgets_host[i] = min_budget + (int32_t)std::floor(share[i]);
      order.push_back(i);
    }
    used += budgets_host[i];
  }
  // the units left by rounding down: largest fractional parts first
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
    return share[x] - std::floor(share[x]) > share[y] - std::floor(share[y]);
  });
  for (int64_t left = total - used, j = 0; left > 0 && j < (int64_t)order.size(); --left, ++j)
    budgets_host[order[j]] += 1;
  return ok();
}

}  // extern "C"
