// Token-level shaping around the advantage step: the reference-policy KL folded into the rewards and
// advantage whitening per model or per (model, role).
//
// The worker groups compute "reference-policy log probabilities" next to the old log-probs (Section
// "PPO-Style Training Loop"); the paper prints no penalty, so the per-token estimate
// logp - logp_ref, scaled by beta and subtracted from the token reward, is taken.  Whitening keeps
// role identity (Section "Parameter Sharing in the System": roles stay distinct under sharing), so
// the statistics can be per role inside a model's stream.
// Both are streaming kernels: 16-byte loads and stores, block sums in float64, a fixed-order final
// reduction so that results do not depend on scheduling.
#include "umas_common.h"

namespace umas {
namespace {

constexpr int kST = 256;            // threads per workgroup
constexpr int kSIpt = 8;            // tokens per thread per step
constexpr int kSMaxGrid = 2048;

struct ModelOffsets {
  int64_t off[UMAS_MAX_MODELS + 1];
};

constexpr int64_t kCacheBytes = int64_t{256} << 20;      // the memory-side cache

// Eight tokens from p0 on, those behind n as masked ones: the rewards where they are wanted, both log-probs, the mask.
template <bool PAST, bool REWARDS>
__device__ __forceinline__ void load_eight(int64_t n, int64_t p0, const float* r, const float* __restrict__ logp, const float* __restrict__ logp_ref,
                                           const uint8_t* __restrict__ mask, float (&rr)[kSIpt], float (&a)[kSIpt], float (&b)[kSIpt],
                                           uint8_t (&m)[kSIpt]) {
  if (p0 + kSIpt <= n) {
#pragma unroll
    for (int k = 0; k < kSIpt / 4; ++k) {
      const float4 r4 = REWARDS ? *reinterpret_cast<const float4*>(r + p0 + 4 * k) : make_float4(0.f, 0.f, 0.f, 0.f);
      const float4 a4 = PAST ? load_stream<float4>(logp + p0 + 4 * k) : *reinterpret_cast<const float4*>(logp + p0 + 4 * k);
      const float4 b4 = PAST ? load_stream<float4>(logp_ref + p0 + 4 * k) : *reinterpret_cast<const float4*>(logp_ref + p0 + 4 * k);
      rr[4 * k] = r4.x; rr[4 * k + 1] = r4.y; rr[4 * k + 2] = r4.z; rr[4 * k + 3] = r4.w;
      a[4 * k] = a4.x; a[4 * k + 1] = a4.y; a[4 * k + 2] = a4.z; a[4 * k + 3] = a4.w;
      b[4 * k] = b4.x; b[4 * k + 1] = b4.y; b[4 * k + 2] = b4.z; b[4 * k + 3] = b4.w;
    }
    const uint2 m2 = *reinterpret_cast<const uint2*>(mask + p0);
#pragma unroll
    for (int k = 0; k < kSIpt; ++k) m[k] = static_cast<uint8_t>((k < 4 ? m2.x : m2.y) >> (8 * (k & 3)));
  } else {
#pragma unroll
    for (int k = 0; k < kSIpt; ++k) {
      const bool in = p0 + k < n;
      rr[k] = in && REWARDS ? r[p0 + k] : 0.f; a[k] = in ? logp[p0 + k] : 0.f; b[k] = in ? logp_ref[p0 + k] : 0.f;
      m[k] = in ? mask[p0 + k] : 0;
    }
  }
}
__device__ __forceinline__ void store_eight(int64_t n, int64_t p0, const float (&rr)[kSIpt], float* r_out) {
  if (p0 + kSIpt <= n) {
#pragma unroll
    for (int k = 0; k < kSIpt / 4; ++k)
      *reinterpret_cast<float4*>(r_out + p0 + 4 * k) = make_float4(rr[4 * k], rr[4 * k + 1], rr[4 * k + 2], rr[4 * k + 3]);
  } else {
    for (int k = 0; k < kSIpt && p0 + k < n; ++k) r_out[p0 + k] = rr[k];
  }
}
// r_out = r - beta (logp - logp_ref) on mask=1 tokens; per block (sum of logp - logp_ref, count).  With PAST the two log-probs are
// read past the caches, which hold the rewards that routing has just written and the scan reads next (25 million tokens 108 -> 85 us;
// with the next trip's loads under way as well 107 instead of 104: it is the memory's time).
template <bool PAST>
__global__ void __launch_bounds__(kST)
k_kl_rewards(int64_t n, const float* r, const float* __restrict__ logp, const float* __restrict__ logp_ref,
             const uint8_t* __restrict__ mask, float beta, float* r_out, double* __restrict__ blk) {   // r_out may be r
  __shared__ double smem[32];
  double ksum = 0.0, cnt = 0.0;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kST * kSIpt;
  for (int64_t p0 = (static_cast<int64_t>(blockIdx.x) * kST + threadIdx.x) * kSIpt; p0 < n; p0 += stride) {
    float rr[kSIpt], a[kSIpt], b[kSIpt];
    uint8_t m[kSIpt];
    load_eight<PAST, true>(n, p0, r, logp, logp_ref, mask, rr, a, b, m);
#pragma unroll
    for (int k = 0; k < kSIpt; ++k) {
      const float kl = a[k] - b[k];
      if (m[k]) {
        rr[k] -= beta * kl;
        ksum += static_cast<double>(kl);
        cnt += 1.0;
      }
    }
    store_eight(n, p0, rr, r_out);
  }
  const double s0 = block_sum<double>(ksum, smem);
  __syncthreads();
  const double s1 = block_sum<double>(cnt, smem);
  if (threadIdx.x == 0) {
    blk[2 * blockIdx.x] = s0;
    blk[2 * blockIdx.x + 1] = s1;
  }
}
__global__ void __launch_bounds__(256)
k_kl_mean(const double* __restrict__ blk, int nblk, float* __restrict__ kl_mean) {
  __shared__ double smem[32];
  double a = 0.0, c = 0.0;
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) { a += blk[2 * b]; c += blk[2 * b + 1]; }
  const double s0 = block_sum<double>(a, smem);
  __syncthreads();
  const double s1 = block_sum<double>(c, smem);
  if (threadIdx.x == 0) *kl_mean = s1 > 0 ? static_cast<float>(s0 / s1) : 0.f;
}

// Both in one launch for few tokens: the last workgroup does nothing but the mean, over all tokens itself, next to the others, which
// leave no sums behind.  A launch less: 46 000 tokens 9.4 us in two launches that follow each other, 7.0 in one, and 10.4 and 5.1 us of the
// host.  One workgroup reads 9 bytes a token at about 90 GB/s, so that from 65 536 tokens on the two launches are as fast.
constexpr int kKlThreads = 1024;
constexpr int64_t kKlAlone = 65536;
__global__ void __launch_bounds__(kKlThreads)
k_kl_rewards_few(int64_t n, const float* r, const float* __restrict__ logp, const float* __restrict__ logp_ref,
                 const uint8_t* __restrict__ mask, float beta, float* r_out, float* __restrict__ kl_mean) {   // r_out may be r
  __shared__ double smem[32];
  float rr[kSIpt], a[kSIpt], b[kSIpt];
  uint8_t m[kSIpt];
  if (blockIdx.x + 1 < gridDim.x) {
    const int64_t p0 = (static_cast<int64_t>(blockIdx.x) * kKlThreads + threadIdx.x) * kSIpt;
    if (p0 >= n) return;
    load_eight<false, true>(n, p0, r, logp, logp_ref, mask, rr, a, b, m);
#pragma unroll
    for (int k = 0; k < kSIpt; ++k)
      if (m[k]) rr[k] -= beta * (a[k] - b[k]);
    store_eight(n, p0, rr, r_out);
    return;
  }
  double ksum = 0.0;
  int cnt = 0;
#pragma unroll 2
  for (int64_t p0 = static_cast<int64_t>(threadIdx.x) * kSIpt; p0 < n; p0 += kKlThreads * kSIpt) {
    load_eight<false, false>(n, p0, nullptr, logp, logp_ref, mask, rr, a, b, m);
#pragma unroll
    for (int k = 0; k < kSIpt; ++k) {
      ksum += static_cast<double>(m[k] ? a[k] - b[k] : 0.f);
      cnt += __popcll(__ballot(m[k] != 0));           // of the wavefront, in one scalar
    }
  }
  cnt = (threadIdx.x & (kWave - 1)) == 0 ? cnt : 0;
  const double s0 = block_sum<double>(ksum, smem);
  __syncthreads();
  const int s1 = block_sum<int>(cnt, reinterpret_cast<int*>(smem));
  if (threadIdx.x == 0) *kl_mean = s1 > 0 ? static_cast<float>(s0 / s1) : 0.f;
}

// Group of a token: its model (scope MODEL) or model * n_roles + role (scope MODEL_ROLE).
__device__ __forceinline__ int model_of(const ModelOffsets& mo, int n_models, int64_t p) {
  int m = 0;
  while (m + 1 < n_models && mo.off[m + 1] <= p) ++m;
  return m;
}

// Sum over the wavefront, in its last lane: six moves between lanes that go with an add (row_shr 1, 2, 4, 8 inside the rows of
// 16 lanes, then lane 15 of every row handed to the next and lane 31 to the upper half), no trips through LDS. Lanes without a source add 0;
// every move writes all rows, so that it and its float32 add are one instruction (what the other lanes hold is not used).
template <int CTRL>
__device__ __forceinline__ int lane_move(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true); }
template <int CTRL>
__device__ __forceinline__ float lane_move(float v) { return __int_as_float(lane_move<CTRL>(__float_as_int(v))); }
template <int CTRL>
__device__ __forceinline__ double lane_move(double v) {
  return __hiloint2double(lane_move<CTRL>(__double2hiint(v)), lane_move<CTRL>(__double2loint(v)));
}
constexpr int kFewChanges = 8;
template <typename T>
__device__ __forceinline__ T last_lane_sum(T v) {
  v += lane_move<0x111>(v);
  v += lane_move<0x112>(v);
  v += lane_move<0x114>(v);
  v += lane_move<0x118>(v);
  v += lane_move<0x142>(v);   // row_bcast:15
  v += lane_move<0x143>(v);   // row_bcast:31
  return v;
}

__device__ __forceinline__ uint32_t last_lane_or(uint32_t b) {       // the same for bits, in every lane
  int v = static_cast<int>(b);
  v |= lane_move<0x111>(v);
  v |= lane_move<0x112>(v);
  v |= lane_move<0x114>(v);
  v |= lane_move<0x118>(v);
  v |= lane_move<0x142>(v);
  v |= lane_move<0x143>(v);
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(v, kWave - 1));
}

// Pass 1: per block and group (sum A, sum A^2, count) over the mask=1 tokens, float64.
// 9 B/token are read at 3.9-4.8 TB/s; what a wavefront executes per 256 tokens counts as much as the memory does. With the model found once
// per wavefront and the lanes' sums in one instruction a step (both were per token and two): 40 million tokens in turns of 400
// 99 -> 87 us, 25 million in turns of 256 60 -> 58, 5.6 million in turns of 700 16.3 -> 14.0, 11.5 million in turns of 16 43 -> 36.
__global__ void __launch_bounds__(kST)
k_whiten_sums(int64_t n, const float* __restrict__ adv, const uint8_t* __restrict__ mask, const int32_t* __restrict__ role,
              ModelOffsets mo, int n_models, int n_roles, int by_role, double* __restrict__ blk) {
  extern __shared__ double s_acc[];             // [groups][3]
  const int groups = by_role ? n_models * n_roles : n_models;
  for (int i = threadIdx.x; i < groups * 3; i += kST) s_acc[i] = 0.0;
  __syncthreads();
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kST * 4;
  const int lane = threadIdx.x & (kWave - 1);
  // whole wavefronts go round: their sums are taken across all lanes
  const int wave0 = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) - lane);
  for (int64_t w0 = (static_cast<int64_t>(blockIdx.x) * kST + wave0) * 4; w0 < n; w0 += stride) {
    const int64_t p0 = w0 + lane * 4;
    // the model, once for the 256 tokens where none begins among them
    const int mw = model_of(mo, n_models, w0);
    const bool one_model = mw + 1 == n_models || mo.off[mw + 1] >= w0 + 4 * kWave;
    float a[4];
    uint8_t m[4];
    int rl[4] = {0, 0, 0, 0};
    if (p0 + 4 <= n) {
      const float4 a4 = *reinterpret_cast<const float4*>(adv + p0);
      const uint32_t m4 = *reinterpret_cast<const uint32_t*>(mask + p0);
      a[0] = a4.x; a[1] = a4.y; a[2] = a4.z; a[3] = a4.w;
#pragma unroll
      for (int k = 0; k < 4; ++k) m[k] = static_cast<uint8_t>(m4 >> (8 * k));
      if (by_role) {
        const int4 r4 = *reinterpret_cast<const int4*>(role + p0);
        rl[0] = r4.x; rl[1] = r4.y; rl[2] = r4.z; rl[3] = r4.w;
      }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool in = p0 + k < n;
        a[k] = in ? adv[p0 + k] : 0.f;
        m[k] = in ? mask[p0 + k] : 0;
        rl[k] = (in && by_role) ? role[p0 + k] : 0;
      }
    }
    // group of each of the four tokens (-1 = not counted)
    int gk[4];
    const int per_model = by_role ? n_roles : 1;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool counted = m[k] && static_cast<unsigned>(rl[k]) < static_cast<unsigned>(per_model);   // a role outside [0, n_roles) joins no group
      gk[k] = counted ? mw * per_model + rl[k] : -1;
    }
    if (!one_model) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (gk[k] >= 0) gk[k] += (model_of(mo, n_models, p0 + k) - mw) * per_model;
    }
    // Usual case: every counted token of the wavefront's 256 belongs to one group.  Their sums are formed in
    // float32 across the lanes (256 values: rounding far below the float32 inputs' own) and one lane adds them
    // to the float64 accumulators.  Where turns of several groups meet in the 256 the groups take turns, in float64 (every lane
    // adding its own tokens in LDS queued on the groups' three words: 40 million tokens in turns of 400 by five roles 356 us,
    // in turns 87), or every lane adds its own: see below.
    auto first_group = [&]() {
      int g = -1;
#pragma unroll
      for (int k = 3; k >= 0; --k) g = gk[k] >= 0 ? gk[k] : g;
      return g;
    };
    int g0 = first_group();
    unsigned long long have = __ballot(g0 >= 0);
    if (!have) continue;                                     // the same for every lane of the wavefront
    int gref = __builtin_amdgcn_readlane(g0, __ffsll(static_cast<long long>(have)) - 1);
    bool same = true;
#pragma unroll
    for (int k = 0; k < 4; ++k) same = same && (gk[k] < 0 || gk[k] == gref);
    auto add = [&](double sa, double sq, int n_in) {         // the last lane has the sums
      if (lane == kWave - 1) {
        atomicAdd(s_acc + 3 * gref, sa);
        atomicAdd(s_acc + 3 * gref + 1, sq);
        atomicAdd(s_acc + 3 * gref + 2, static_cast<double>(n_in));
      }
    };
    if (__all(same)) {
      float sa = 0.f, sq = 0.f;
      int n_in = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (gk[k] >= 0) { sa += a[k]; sq = fmaf(a[k], a[k], sq); }
        n_in += __popcll(__ballot(gk[k] >= 0));
      }
      sa = last_lane_sum(sa);
      sq = last_lane_sum(sq);
      add(static_cast<double>(sa), static_cast<double>(sq), n_in);
      continue;
    }
    // Turns or lane by lane?  Turns cost by the groups, about 6 us each for 11.5 million tokens, on top of 17.  Adds of single lanes queue where
    // neighbouring lanes have the same group, and are four times as many in a lane of mixed tokens.  So few places where the
    // group changes: turns, without counting the groups; else by their number and by how many lanes are mixed.  11.5 million tokens, turns
    // and lanes: 16 roles, turns of 4 tokens 71 and 21 us, of 7 72 and 31, of 16 70 and 28, of 25 68 and 35, of 64 38 and 47; 3 roles, of 4 32 and
    // 26, of 7 32 and 48, of 64 30 and 46; 4 roles that change with every token 40 and 174, 8 roles 68 and 50.
    bool lane_mixed = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) lane_mixed = lane_mixed || (gk[k] >= 0 && gk[k] != g0);
    const int mixed = __popcll(__ballot(lane_mixed));
    const int changes = __popcll(__ballot(__builtin_amdgcn_update_dpp(g0, g0, 0x111, 0xF, 0xF, false) != g0));   // row_shr:1; not from row to row
    bool turns = one_model;
    if (one_model && changes + mixed > kFewChanges) {
      uint32_t lo = 0u, hi = 0u;                             // a bit per role of the model
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t r = static_cast<uint32_t>(gk[k] - mw * per_model), bit = gk[k] >= 0 ? 1u << (r & 31) : 0u;
        lo |= r < 32 ? bit : 0u;
        hi |= r < 32 ? 0u : bit;
      }
      const int present = __popc(last_lane_or(lo)) + (n_roles > 32 ? __popc(last_lane_or(hi)) : 0);
      turns = present <= (mixed > kWave / 2 ? 6 : mixed > 0 ? 4 : 2);
    }
    if (!turns) {
      double sa = 0.0, sq = 0.0;
      int n_in = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double x = gk[k] >= 0 ? static_cast<double>(a[k]) : 0.0;
        sa += x;
        sq = fma(x, x, sq);
        n_in += gk[k] >= 0;
      }
      if (lane_mixed) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (gk[k] >= 0) {
            const double x = static_cast<double>(a[k]);
            atomicAdd(s_acc + 3 * gk[k], x); atomicAdd(s_acc + 3 * gk[k] + 1, x * x); atomicAdd(s_acc + 3 * gk[k] + 2, 1.0);
          }
      } else if (n_in) {
        atomicAdd(s_acc + 3 * g0, sa); atomicAdd(s_acc + 3 * g0 + 1, sq); atomicAdd(s_acc + 3 * g0 + 2, static_cast<double>(n_in));
      }
      continue;
    }
    for (;;) {
      double sa = 0.0, sq = 0.0;
      int n_in = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool mine = gk[k] == gref;
        const double x = mine ? static_cast<double>(a[k]) : 0.0;
        sa += x;
        sq = fma(x, x, sq);
        n_in += __popcll(__ballot(mine));
        if (mine) gk[k] = -1;
      }
      sa = last_lane_sum(sa);
      sq = last_lane_sum(sq);
      add(sa, sq, n_in);
      g0 = first_group();
      have = __ballot(g0 >= 0);
      if (!have) break;
      gref = __builtin_amdgcn_readlane(g0, __ffsll(static_cast<long long>(have)) - 1);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < groups * 3; i += kST) blk[static_cast<size_t>(blockIdx.x) * groups * 3 + i] = s_acc[i];
}
__device__ __forceinline__ double2 mean_rstd(const double (&t)[3], float eps) {
  if (!(t[2] > 0)) return make_double2(0.0, 1.0);
  const double mu = t[0] / t[2];
  double var = t[1] / t[2] - mu * mu;
  if (var < 0) var = 0;
  return make_double2(mu, 1.0 / sqrt(var + static_cast<double>(eps)));
}
// Per group (one workgroup each): mean and 1/sqrt(var + eps) from the block sums, added in a fixed order.  Few block sums
// (kInlineSums) are added up by every workgroup of the second pass instead, the same way in each: a launch less
// (49 152 tokens in three groups: 5.3 + 3.2 + 3.5 us in three launches, 5.3 + 4.5 in two).
constexpr int kInlineSums = 256;
__global__ void __launch_bounds__(256)
k_whiten_stats(const double* __restrict__ blk, int nblk, int groups, float eps, double2* __restrict__ mu_rstd) {
  __shared__ double smem[32];
  const int g = blockIdx.x;
  double v[3] = {0.0, 0.0, 0.0};
  for (int b = threadIdx.x; b < nblk; b += blockDim.x) {
    const double* p = blk + (static_cast<size_t>(b) * groups + g) * 3;
    v[0] += p[0]; v[1] += p[1]; v[2] += p[2];
  }
  double t[3];
  for (int j = 0; j < 3; ++j) {
    t[j] = block_sum<double>(v[j], smem);
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  mu_rstd[g] = mean_rstd(t, eps);
}
// Pass 2: A' = (A - mu_g) rstd_g on mask=1 tokens, 0 elsewhere; with PAST stored past the caches, which hold what the first pass has
// read (25 million tokens 64 -> 56 us).
template <bool PAST>
__global__ void __launch_bounds__(kST)
k_whiten_apply(int64_t n, const float* adv, const uint8_t* __restrict__ mask, const int32_t* __restrict__ role,
               ModelOffsets mo, int n_models, int n_roles, int by_role, const double2* __restrict__ mu_rstd,
               const double* __restrict__ blk, int nblk, float eps, float* out) {   // out may be adv; mu_rstd NULL: from blk
  extern __shared__ double2 s_ms[];
  const int groups = by_role ? n_models * n_roles : n_models;
  if (mu_rstd) {
    for (int i = threadIdx.x; i < groups; i += kST) s_ms[i] = mu_rstd[i];
  } else {
    const int lane = threadIdx.x & (kWave - 1);
    for (int g = threadIdx.x / kWave; g < groups; g += kST / kWave) {
      double t[3] = {0.0, 0.0, 0.0};
      for (int b = lane; b < nblk; b += kWave)
#pragma unroll
        for (int j = 0; j < 3; ++j) t[j] += blk[(static_cast<size_t>(b) * groups + g) * 3 + j];
#pragma unroll
      for (int j = 0; j < 3; ++j) t[j] = wave_sum(t[j]);
      if (lane == 0) s_ms[g] = mean_rstd(t, eps);
    }
  }
  __syncthreads();
  const int64_t stride = static_cast<int64_t>(gridDim.x) * kST * 4;
  for (int64_t p0 = (static_cast<int64_t>(blockIdx.x) * kST + threadIdx.x) * 4; p0 < n; p0 += stride) {
    float a[4], o[4];
    uint8_t m[4];
    int rl[4] = {0, 0, 0, 0};
    const bool full = p0 + 4 <= n;
    if (full) {
      const float4 a4 = *reinterpret_cast<const float4*>(adv + p0);
      const uint32_t m4 = *reinterpret_cast<const uint32_t*>(mask + p0);
      a[0] = a4.x; a[1] = a4.y; a[2] = a4.z; a[3] = a4.w;
#pragma unroll
      for (int k = 0; k < 4; ++k) m[k] = static_cast<uint8_t>(m4 >> (8 * k));
      if (by_role) {
        const int4 r4 = *reinterpret_cast<const int4*>(role + p0);
        rl[0] = r4.x; rl[1] = r4.y; rl[2] = r4.z; rl[3] = r4.w;
      }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const bool in = p0 + k < n;
        a[k] = in ? adv[p0 + k] : 0.f;
        m[k] = in ? mask[p0 + k] : 0;
        rl[k] = (in && by_role) ? role[p0 + k] : 0;
      }
    }
    const int m0 = model_of(mo, n_models, p0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      o[k] = 0.f;
      if (m[k] && !(by_role && (rl[k] < 0 || rl[k] >= n_roles))) {
        const int md = (p0 + k < mo.off[m0 + 1] || m0 + 1 >= n_models) ? m0 : model_of(mo, n_models, p0 + k);
        const double2 ms = s_ms[by_role ? md * n_roles + rl[k] : md];
        o[k] = static_cast<float>((static_cast<double>(a[k]) - ms.x) * ms.y);   // the mean in full precision: groups of nearly equal values
      }
    }
    if (full && PAST) store_stream(out + p0, make_float4(o[0], o[1], o[2], o[3]));
    else if (full) *reinterpret_cast<float4*>(out + p0) = make_float4(o[0], o[1], o[2], o[3]);
    else
      for (int k = 0; k < 4 && p0 + k < n; ++k) out[p0 + k] = o[k];
  }
}

unsigned stream_grid(int64_t n, int per_block) {
  const int64_t b = (n + per_block - 1) / per_block;
  return static_cast<unsigned>(b < 1 ? 1 : b > kSMaxGrid ? kSMaxGrid : b);
}

}  // namespace
}  // namespace umas

using namespace umas;

extern "C" size_t umas_kl_rewards_workspace_bytes(int64_t n_tokens) {
  if (n_tokens < 0) return 0;
  Carver c(nullptr);
  c.take<double>(2 * static_cast<size_t>(stream_grid(n_tokens, kST * kSIpt)));
  return c.off;
}

extern "C" umas_status umas_kl_rewards(const float* tok_reward, const float* logp, const float* logp_ref,
                                       const uint8_t* tok_mask, int64_t n_tokens, float beta, float* tok_reward_out,
                                       float* kl_mean, void* workspace, size_t workspace_bytes, void* hip_stream) {
  UMAS_REQUIRE(n_tokens >= 0, UMAS_EINVAL, "negative size");
  UMAS_REQUIRE((tok_reward && logp && logp_ref && tok_mask && tok_reward_out) || n_tokens == 0, UMAS_EINVAL,
               "tok_reward, logp, logp_ref, tok_mask and tok_reward_out must not be NULL");
  UMAS_REQUIRE(kl_mean, UMAS_EINVAL, "kl_mean must not be NULL");
  UMAS_REQUIRE(beta == beta, UMAS_EINVAL, "beta must be a number");
  UMAS_REQUIRE(reinterpret_cast<uintptr_t>(tok_reward) % 16 == 0 && reinterpret_cast<uintptr_t>(logp) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(logp_ref) % 16 == 0 && reinterpret_cast<uintptr_t>(tok_mask) % 8 == 0 &&
                   reinterpret_cast<uintptr_t>(tok_reward_out) % 16 == 0,
               UMAS_EINVAL, "token arrays must be 16-byte aligned (the mask 8-byte)");
  const size_t need = umas_kl_rewards_workspace_bytes(n_tokens);
  UMAS_REQUIRE(workspace && reinterpret_cast<uintptr_t>(workspace) % kAlign == 0 && workspace_bytes >= need, UMAS_EWORKSPACE,
               "workspace must be 256-byte aligned and hold %zu bytes (got %zu)", need, workspace_bytes);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  prof_mark(st);
  // (its last workgroup reads the log-probs while the others write: not where they write over them)
  auto apart = [&](const float* p) { return tok_reward_out + n_tokens <= p || p + n_tokens <= tok_reward_out; };
  if (n_tokens <= kKlAlone && apart(logp) && apart(logp_ref)) {
    const unsigned wg = cdiv(static_cast<size_t>(n_tokens), kKlThreads * kSIpt) + 1;
    hipLaunchKernelGGL(k_kl_rewards_few, dim3(wg), dim3(kKlThreads), 0, st, n_tokens, tok_reward, logp, logp_ref, tok_mask, beta, tok_reward_out, kl_mean);
    UMAS_LAUNCHED("k_kl_rewards_few");
    return UMAS_OK;
  }
  const unsigned grid = stream_grid(n_tokens, kST * kSIpt);
  double* blk = static_cast<double*>(workspace);
  // Past the caches where the rewards fit them and the 13 bytes a token that are read do not.  Smaller: the log-probs may lie there as
  // well; larger: the rewards do not either.  In place again and again, through the caches and past them: 8 million tokens 27 and 30 us, 16 46
  // and 51, 25 69 and 75 (behind routing 108 and 85), 40 138 and 113, 64 216 and 209, 80 269 and 276, 101 342 and 351.
  const bool past = 13 * n_tokens > kCacheBytes && 4 * n_tokens <= kCacheBytes;
  if (past) hipLaunchKernelGGL(k_kl_rewards<true>, dim3(grid), dim3(kST), 0, st, n_tokens, tok_reward, logp, logp_ref, tok_mask, beta, tok_reward_out, blk);
  else hipLaunchKernelGGL(k_kl_rewards<false>, dim3(grid), dim3(kST), 0, st, n_tokens, tok_reward, logp, logp_ref, tok_mask, beta, tok_reward_out, blk);
  UMAS_LAUNCHED("k_kl_rewards");
  hipLaunchKernelGGL(k_kl_mean, dim3(1), dim3(256), 0, st, blk, static_cast<int>(grid), kl_mean);
  UMAS_LAUNCHED("k_kl_mean");
  return UMAS_OK;
}

extern "C" size_t umas_whiten_workspace_bytes(int64_t n_tokens, int32_t n_models, int32_t n_roles) {
  if (n_tokens < 0 || n_models < 1 || n_roles < 1) return 0;
  Carver c(nullptr);
  const size_t groups = static_cast<size_t>(n_models) * n_roles;
  c.take<double>(static_cast<size_t>(stream_grid(n_tokens, kST * 4)) * groups * 3);
  c.take<double2>(groups);
  return c.off;
}

extern "C" umas_status umas_whiten_advantages(const float* adv, const uint8_t* tok_mask, const int32_t* tok_role,
                                              const int64_t* model_tok_off, int32_t n_models, int32_t n_roles,
                                              int64_t n_tokens, int32_t scope, float eps, float* adv_out,
                                              void* workspace, size_t workspace_bytes, void* hip_stream) {
  UMAS_REQUIRE(n_tokens >= 0, UMAS_EINVAL, "negative size");
  UMAS_REQUIRE(n_models >= 1 && n_models <= UMAS_MAX_MODELS, UMAS_ESHAPE, "n_models=%d outside [1,%d]", n_models, UMAS_MAX_MODELS);
  UMAS_REQUIRE(n_roles >= 1 && n_roles <= UMAS_MAX_ROLES, UMAS_ESHAPE, "n_roles=%d outside [1,%d]", n_roles, UMAS_MAX_ROLES);
  UMAS_REQUIRE(scope == UMAS_WHITEN_MODEL || scope == UMAS_WHITEN_MODEL_ROLE, UMAS_EINVAL, "scope=%d is neither MODEL nor MODEL_ROLE", scope);
  UMAS_REQUIRE(eps > 0.f, UMAS_EINVAL, "eps must be positive");
  UMAS_REQUIRE(model_tok_off, UMAS_EINVAL, "model_tok_off must not be NULL");
  UMAS_REQUIRE(model_tok_off[0] == 0 && model_tok_off[n_models] == n_tokens, UMAS_EINVAL, "model_tok_off must run from 0 to n_tokens");
  for (int m = 0; m < n_models; ++m)
    UMAS_REQUIRE(model_tok_off[m] <= model_tok_off[m + 1], UMAS_EINVAL, "model_tok_off decreases at %d", m);
  const int by_role = scope == UMAS_WHITEN_MODEL_ROLE ? 1 : 0;
  UMAS_REQUIRE((adv && tok_mask && adv_out && (tok_role || !by_role)) || n_tokens == 0, UMAS_EINVAL,
               "adv, tok_mask, adv_out (and tok_role for the per-role scope) must not be NULL");
  UMAS_REQUIRE(reinterpret_cast<uintptr_t>(adv) % 16 == 0 && reinterpret_cast<uintptr_t>(adv_out) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(tok_mask) % 4 == 0 && reinterpret_cast<uintptr_t>(tok_role) % 16 == 0,
               UMAS_EINVAL, "token arrays must be 16-byte aligned (the mask 4-byte)");
  const size_t need = umas_whiten_workspace_bytes(n_tokens, n_models, n_roles);
  UMAS_REQUIRE(workspace && reinterpret_cast<uintptr_t>(workspace) % kAlign == 0 && workspace_bytes >= need, UMAS_EWORKSPACE,
               "workspace must be 256-byte aligned and hold %zu bytes (got %zu)", need, workspace_bytes);
  if (n_tokens == 0) return UMAS_OK;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  prof_mark(st);
  ModelOffsets mo;
  for (int m = 0; m <= UMAS_MAX_MODELS; ++m) mo.off[m] = m <= n_models ? model_tok_off[m] : n_tokens;
  const int groups = by_role ? n_models * n_roles : n_models;
  const unsigned grid = stream_grid(n_tokens, kST * 4);
  Carver c(workspace);
  double* blk = c.take<double>(static_cast<size_t>(grid) * n_models * n_roles * 3);
  double2* ms = c.take<double2>(static_cast<size_t>(n_models) * n_roles);
  hipLaunchKernelGGL(k_whiten_sums, dim3(grid), dim3(kST), groups * 3 * sizeof(double), st, n_tokens, adv, tok_mask, tok_role,
                     mo, n_models, n_roles, by_role, blk);
  UMAS_LAUNCHED("k_whiten_sums");
  const bool apart = static_cast<int64_t>(grid) * groups > kInlineSums;
  if (apart) {
    hipLaunchKernelGGL(k_whiten_stats, dim3(groups), dim3(256), 0, st, blk, static_cast<int>(grid), groups, eps, ms);
    UMAS_LAUNCHED("k_whiten_stats");
  }
  // Past the caches where the 9 bytes a token that the first pass reads (5 without roles) and the output do not fit them together; below, who
  // reads the output next finds it there.  Whitening and a kernel that scales the output, through the caches and past them: 8 million tokens
  // 48 and 50 us, 16 83 and 86 (with the advantages written right before 122 and 132), 20 104 and 105, 22 124 and 117, 25 149 and
  // 135, 40 238 and 235.
  const bool past = (by_role ? 13 : 9) * n_tokens > kCacheBytes;
  auto apply = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kST), groups * sizeof(double2), st, n_tokens, adv, tok_mask, tok_role, mo, n_models, n_roles,
                       by_role, apart ? ms : nullptr, blk, static_cast<int>(grid), eps, adv_out);
  };
  if (past) apply(k_whiten_apply<true>);
  else apply(k_whiten_apply<false>);
  UMAS_LAUNCHED("k_whiten_apply");
  return UMAS_OK;
}
