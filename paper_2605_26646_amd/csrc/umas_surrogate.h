// What every path of the update does per selected row: the clipped surrogate, its statistics, and the clearing of rows that
// are not selected.
#pragma once

#include <math.h>

#include "umas_common.h"

namespace umas {
namespace {

// What a call defines on rows that are not selected, cleared in one launch (scoring through a selection, a launch for each array
// and in one: 20 rows of 2048 121.9 and 119.0 us, 3 rows of 1024 against 30 001 24.3 and 21.3).
struct ClearArgs {
  uint32_t* p[3];        // NULL: nothing
  int64_t words[3];
};
__device__ __forceinline__ void clear_words(const ClearArgs& A, int64_t i0, int64_t stride) {
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (A.p[k])
      for (int64_t i = i0; i < A.words[k]; i += stride) A.p[k][i] = 0u;
}

// Clipped PPO: ratio = exp(logp - logp_old), L = max(-A ratio, -A clip(ratio)), capped by dual_clip for A < 0, and the penalty
// towards the reference policy; g = dL / dlogp over norm rows.
struct Surrogate {
  int64_t norm;
  const int32_t* __restrict__ rowsel;
  const int32_t* __restrict__ ids;
  int V;
  const float* __restrict__ logp_old;
  const float* __restrict__ adv;
  const int32_t* __restrict__ tok_role;
  int n_roles;
  float clip_eps, dual_clip;
  const float* __restrict__ logp_ref;
  float kl_coef;
};
struct SurrogateRow {
  float L, clipped, en, kl, g;
  int role;              // -1: none
  bool valid;            // the token id exists; everything else is 0 where it does not
};
// `row`: the row of the caller's arrays; lp and en: its new log-prob and entropy (not looked at where the id is invalid).
__device__ __forceinline__ SurrogateRow surrogate_row(const Surrogate& S, int64_t row, bool valid, float lp, float en) {
  SurrogateRow r{0.f, 0.f, 0.f, 0.f, 0.f, -1, valid};
  if (valid) {
    const float lo = S.logp_old ? S.logp_old[row] : lp, A = S.adv[row];   // no old log-probs: the update is on-policy, ratio 1
    const float ratio = __expf(lp - lo);
    const float u = -A * ratio;
    const float c = -A * fminf(fmaxf(ratio, 1.f - S.clip_eps), 1.f + S.clip_eps);
    bool unclipped = u >= c;
    r.L = unclipped ? u : c;
    if (S.dual_clip > 0.f && A < 0.f && -A * S.dual_clip < r.L) {   // dual clip: the term of a negative advantage is capped
      r.L = -A * S.dual_clip;
      unclipped = false;
    }
    r.g = unclipped ? u / static_cast<float>(S.norm) : 0.f;
    r.clipped = unclipped ? 0.f : 1.f;
    if (S.kl_coef != 0.f) {   // kl_coef (e^x - x - 1), x = logp_ref - logp
      const float x = S.logp_ref[row] - lp, ex = __expf(x);
      r.L += S.kl_coef * (ex - x - 1.f);
      r.g += S.kl_coef * (1.f - ex) / static_cast<float>(S.norm);
    }
    r.en = en;
    r.kl = lo - lp;
  }
  r.role = (S.tok_role && S.n_roles > 0) ? S.tok_role[row] : -1;
  return r;
}

// Sums of (L, clipped, entropy, logp_old - logp, rows, invalid ids), in float64, and the record they make: k = 0 the model's, else a
// role's.
constexpr int kStat = 6;
__device__ __forceinline__ umas_loss_stats loss_stats(const double (&sum)[kStat], int k, float entropy_coef, int64_t norm_rows) {
  const double cnt = sum[4];
  umas_loss_stats s;
  // the model's loss over the caller's normaliser when one is given: micro-batch losses then add up
  const double den = (k == 0 && norm_rows > 0) ? static_cast<double>(norm_rows) : cnt;
  s.loss = cnt > 0 ? static_cast<float>((sum[0] - static_cast<double>(entropy_coef) * sum[2]) / den) : 0.f;
  s.clip_frac = cnt > 0 ? static_cast<float>(sum[1] / cnt) : 0.f;
  s.entropy_mean = cnt > 0 ? static_cast<float>(sum[2] / cnt) : 0.f;
  s.approx_kl = cnt > 0 ? static_cast<float>(sum[3] / cnt) : 0.f;
  s.n_scored = static_cast<int64_t>(cnt);
  s.n_invalid_ids = static_cast<int64_t>(sum[5]);
  return s;
}

}  // namespace
}  // namespace umas
