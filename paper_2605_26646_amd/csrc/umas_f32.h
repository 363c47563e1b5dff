// The float32 path of scoring and update: float32 operands, every product and sum in float64 (a float32 dot product of d
// terms would cost up to d 2^-24 of the sum of its terms' magnitudes), results rounded to float32 once.
//
// All four products (logits for the scoring pass, logits for dz, dH = dz W, dW = dz^T H) are contractions and run on the
// float64 matrix cores: v_mfma_f64_16x16x4 sustains 74 TFLOP/s here and asks for one converted float per lane and operand
// every 64 cycles, so a wavefront's 32 x 32 tile (2 x 2 blocks) is fed straight from L1 / L2 into registers, 16 k at a time, the
// next 16 in flight; no LDS, no barrier in the loop.  The k of an instruction may be any four as long as both operands
// agree: lane group l / 16 takes k = 4 (l / 16) .. + 3 of the 16 over four instructions, so that a K-contiguous operand is
// read 16 bytes a lane.  With one thread per output element and scalar float64 chains dz, dH and dW took 17, 52 and 189 us at
// 768 rows of 64 against 512, now 7 and, the two products together, 12.5; a step of 847 rows of 512 against 8192 took 10.1 ms, now 0.62.
//
// Operand layout of a block (lane l): index l % 16, k by lane group l / 16.  Accumulator r of lane l: row 4 r + l / 16 (A
// side), column l % 16 (B side); checked on the device.
#pragma once

#include "umas_common.h"
#include "umas_surrogate.h"

namespace umas {
namespace f32 {

typedef double double4v __attribute__((ext_vector_type(4)));
constexpr int kK = 16;                       // k of one round
constexpr int kTile = 32;                    // a wavefront's tile, both ways

// Operands of a tile of NB blocks of 16.  Stored K-contiguous: row i of the tile is a run of K floats.
template <int NB>
struct Rows {
  const float* p[NB];                        // the lane's row of each block
  bool vec;                                  // every row starts at a multiple of 16 bytes and K is a multiple of 4
  __device__ __forceinline__ void ahead(int, int) {}
  __device__ __forceinline__ void load(int k0, int K, float (&x)[NB][4]) const {
    const int k = k0 + 4 * ((threadIdx.x & 63) >> 4);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (vec) {
        const float4 v = k < K ? *reinterpret_cast<const float4*>(p[i] + k) : make_float4(0.f, 0.f, 0.f, 0.f);
        x[i][0] = v.x; x[i][1] = v.y; x[i][2] = v.z; x[i][3] = v.w;
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) x[i][s] = k + s < K ? p[i][k + s] : 0.f;
      }
    }
  }
};
// Stored K-major: k-row k (row map[k] of the matrix, where there is a map) holds the tile's entries next to each other.
template <int NB>
struct Cols {
  const float* p[NB];                        // the lane's entry of each block in k-row 0
  int64_t ld;
  const int32_t* map;
  int32_t row[4];                            // k-rows of the next round
  __device__ __forceinline__ void ahead(int k0, int K) {
    const int k = k0 + 4 * ((threadIdx.x & 63) >> 4);
#pragma unroll
    for (int s = 0; s < 4; ++s) row[s] = map ? map[k + s < K ? k + s : K - 1] : k + s;
  }
  __device__ __forceinline__ void load(int k0, int K, float (&x)[NB][4]) const {
    const int k = k0 + 4 * ((threadIdx.x & 63) >> 4);
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int s = 0; s < 4; ++s) x[i][s] = k + s < K ? p[i][row[s] * ld] : 0.f;
  }
};

// acc += A[., k] B[., k] over k in [k0, k1), K of them altogether; k0 a multiple of 16, k1 too unless it is K.  Loads run D rounds ahead:
// one for tiles of 32, more registers than that take wavefronts off the unit; three for the tiles of 16 of products that are
// a few rounds long and nothing but waiting.
template <int NB> constexpr int kRoundsAhead = NB == 1 ? 3 : 1;
template <int NB, class OA, class OB>
__device__ __forceinline__ void product(OA& a, OB& b, int k0, int k1, int K, double4v (&acc)[NB][NB]) {
  constexpr int D = kRoundsAhead<NB>;
  if (k0 >= k1) return;
  float xa[D + 1][NB][4], xb[D + 1][NB][4];
#pragma unroll
  for (int t = 0; t < D; ++t) {              // past the end: zeros, no access
    a.ahead(k0 + t * kK, K);
    b.ahead(k0 + t * kK, K);
    a.load(k0 + t * kK, k1, xa[t]);
    b.load(k0 + t * kK, k1, xb[t]);
  }
  a.ahead(k0 + D * kK, K);
  b.ahead(k0 + D * kK, K);
  for (int k = k0; k < k1; k += kK) {
    a.load(k + D * kK, k1, xa[D]);
    b.load(k + D * kK, k1, xb[D]);
    a.ahead(k + (D + 1) * kK, K);
    b.ahead(k + (D + 1) * kK, K);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(static_cast<double>(xa[0][i][s]), static_cast<double>(xb[0][j][s]), acc[i][j], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < D; ++t)
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int s = 0; s < 4; ++s) { xa[t][i][s] = xa[t + 1][i][s]; xb[t][i][s] = xb[t + 1][i][s]; }
  }
}
template <int NB>
__device__ __forceinline__ void zero(double4v (&acc)[NB][NB]) {
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = double4v{0.0, 0.0, 0.0, 0.0};
}
__device__ __forceinline__ int blk_index(int i) { return i * 16 + (threadIdx.x & 15); }                       // operand entry / column
__device__ __forceinline__ int blk_row(int i, int r) { return i * 16 + 4 * r + ((threadIdx.x & 63) >> 4); }   // accumulator row

// ------------------------------------------------------------------ scoring
// Softmax statistics of part of a row's logits: maximum, sum exp(z - m), sum exp(z - m) z, the second without the taken
// token, and the taken token's logit (0 elsewhere).
struct Stat {
  double m, s, t, rest, zy;
};
__device__ __forceinline__ Stat empty_stat() { return Stat{0.0, 0.0, 0.0, 0.0, 0.0}; }
__device__ __forceinline__ Stat merge(const Stat& x, const Stat& y) {
  if (x.s == 0.0) return Stat{y.m, y.s, y.t, y.rest, x.zy + y.zy};
  if (y.s == 0.0) return Stat{x.m, x.s, x.t, x.rest, x.zy + y.zy};
  const double M = fmax(x.m, y.m), ex = exp(x.m - M), ey = exp(y.m - M);
  return Stat{M, x.s * ex + y.s * ey, x.t * ex + y.t * ey, x.rest * ex + y.rest * ey, x.zy + y.zy};
}
__device__ __forceinline__ Stat shfl_xor(const Stat& x, int o) {
  return Stat{__shfl_xor(x.m, o, kWave), __shfl_xor(x.s, o, kWave), __shfl_xor(x.t, o, kWave), __shfl_xor(x.rest, o, kWave),
              __shfl_xor(x.zy, o, kWave)};
}
struct ScoreOut {
  double* z;                                 // the logits [n_sel][V] for the backward (NULL: not kept)
  double* rest_c;                            // compact arrays (NULL: none): sum of the probabilities of the tokens not taken
  float *logp_c, *lse_c, *ent_c;
  float *logp, *lse, *entropy;               // scattered (NULL: none)
};
struct Scores {
  bool ok;                                   // the token id exists
  float lse, lp, en;
  double rest;                               // relative to the rounded logsumexp, as dz is
};
__device__ __forceinline__ Scores scores_of(const Stat& a, int y, int V) {
  const bool ok = y >= 0 && y < V;
  const double l = a.m + log(a.s);
  const float lf = static_cast<float>(l);
  return Scores{ok, lf, ok ? static_cast<float>(a.zy - l) : 0.f, ok ? static_cast<float>(l - a.t / a.s) : 0.f, a.rest * exp(a.m - static_cast<double>(lf))};
}
__device__ __forceinline__ void write_scores(const Stat& a, int64_t n, int64_t row, int y, int V, const ScoreOut& o) {
  const Scores s = scores_of(a, y, V);
  if (o.logp_c) {
    o.logp_c[n] = s.lp; o.lse_c[n] = s.lse; o.ent_c[n] = s.en;
    o.rest_c[n] = s.rest;
  }
  if (o.logp) o.logp[row] = s.lp;
  if (o.lse) o.lse[row] = s.lse;
  if (o.entropy) o.entropy[row] = s.en;
}

// A workgroup takes 32 rows and every splits-th block of 128 vocabulary entries, 32 to a wavefront; a lane holds 8
// entries of each of two rows.  With NB = 1 it is half as many of both: four times as many workgroups, a quarter as many products in each,
// for updates that are few tiles altogether (see update).  Without `part` (one workgroup per row block) the scores are final, else the statistics go to
// part[splits][n_sel].  The workgroups behind them clear: behind, for two that multiply to meet on a compute unit while another one
// clears costs twice the time (100 rows of 512 against 8000 60 -> 71 us).  KEEP_Z: the logits go to out.z (asked at run time, 3 % slower also where they do not: 12 000 rows of 32 against 8000
// 368 and 378 us).
constexpr int kWaves = 4, kVocBlock = kWaves * kTile;
template <bool KEEP_Z, int NB>
__global__ void __launch_bounds__(kWaves* kWave)
k_score_f32(const float* __restrict__ W, const float* __restrict__ H, int d, int V, const int32_t* __restrict__ rowsel, int64_t n_sel,
            const int32_t* __restrict__ ids, Stat* __restrict__ part, ScoreOut out, int splits, ClearArgs clear) {
  constexpr int kSide = 16 * NB, kBlock = kWaves * kSide;
  __shared__ Stat s_stat[kWaves][kSide];
  if (static_cast<int>(blockIdx.y) >= splits) {
    const int64_t wg = static_cast<int64_t>(blockIdx.y - splits) * gridDim.x + blockIdx.x, n_wg = static_cast<int64_t>(gridDim.y - splits) * gridDim.x;
    clear_words(clear, wg * blockDim.x + threadIdx.x, n_wg * blockDim.x);
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t n0 = static_cast<int64_t>(blockIdx.x) * kSide;
  Rows<NB> h;
  h.vec = d % 4 == 0;
  int y[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int64_t n = min(n0 + blk_index(j), n_sel - 1), row = rowsel ? rowsel[n] : n;
    h.p[j] = H + row * d;
    y[j] = ids[row];
  }
  Stat st[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) st[j] = empty_stat();
  for (int64_t vb = static_cast<int64_t>(blockIdx.y) * kBlock; vb < V; vb += static_cast<int64_t>(splits) * kBlock) {
    const int v0 = static_cast<int>(vb) + wave * kSide;
    if (v0 >= V) continue;
    Rows<NB> w;
    w.vec = h.vec;
#pragma unroll
    for (int i = 0; i < NB; ++i) w.p[i] = W + static_cast<int64_t>(min(v0 + blk_index(i), V - 1)) * d;
    double4v acc[NB][NB];
    zero<NB>(acc);
    product<NB>(w, h, 0, d, d, acc);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      double m = -1e300;                     // below every finite logit that matters; infinities and NaN pass through the sums
      int have = 0;
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (v0 + blk_row(i, r) < V) { m = fmax(m, acc[i][j][r]); have = 1; }
      if (!have) continue;
      Stat q{m, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int v = v0 + blk_row(i, r);
          if (v >= V) continue;
          const double z = acc[i][j][r], e = exp(z - m);
          if (KEEP_Z && n0 + blk_index(j) < n_sel) out.z[(n0 + blk_index(j)) * V + v] = z;
          q.s += e;
          q.t = fma(e, z, q.t);
          if (v == y[j]) q.zy = z; else q.rest += e;
        }
      st[j] = merge(st[j], q);
    }
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    st[j] = merge(st[j], shfl_xor(st[j], 16));
    st[j] = merge(st[j], shfl_xor(st[j], 32));
    if (lane < 16) s_stat[wave][blk_index(j)] = st[j];
  }
  __syncthreads();
  const int64_t n = n0 + threadIdx.x;
  if (threadIdx.x >= kSide || n >= n_sel) return;
  Stat a = s_stat[0][threadIdx.x];
  for (int k = 1; k < kWaves; ++k) a = merge(a, s_stat[k][threadIdx.x]);
  if (part) {
    part[static_cast<int64_t>(blockIdx.y) * n_sel + n] = a;
    return;
  }
  const int64_t row = rowsel ? rowsel[n] : n;
  write_scores(a, n, row, ids[row], V, out);
}
// One workgroup per row, every thread walks the vocabulary entries tid, tid + 256, ...: one launch and no room needed.
template <bool KEEP_Z>
__global__ void __launch_bounds__(256)
k_score_f32_row(const float* __restrict__ W, const float* __restrict__ H, int d, int V, const int32_t* __restrict__ rowsel,
                const int32_t* __restrict__ ids, ScoreOut out) {
  extern __shared__ float s_h[];             // [d]
  __shared__ Stat s_stat[256 / kWave];
  const int64_t n = blockIdx.x, row = rowsel ? rowsel[n] : n;
  for (int k = threadIdx.x; k < d; k += 256) s_h[k] = H[row * d + k];
  __syncthreads();
  const int y = ids[row];
  Stat a = empty_stat();
  for (int v = threadIdx.x; v < V; v += 256) {
    const float* w = W + static_cast<int64_t>(v) * d;
    double z = 0.0;
    for (int k = 0; k < d; ++k) z = fma(static_cast<double>(s_h[k]), static_cast<double>(w[k]), z);
    if (KEEP_Z) out.z[n * V + v] = z;
    a = merge(a, Stat{z, 1.0, z, v == y ? 0.0 : 1.0, v == y ? z : 0.0});
  }
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) a = merge(a, shfl_xor(a, o));
  if ((threadIdx.x & 63) == 0) s_stat[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int k = 1; k < 256 / kWave; ++k) a = merge(a, s_stat[k]);
  write_scores(a, n, row, y, V, out);
}
// One wavefront per row.
__global__ void __launch_bounds__(256)
k_score_f32_merge(const Stat* __restrict__ part, int splits, int V, const int32_t* __restrict__ rowsel, int64_t n_sel,
                  const int32_t* __restrict__ ids, ScoreOut out) {
  const int lane = threadIdx.x & 63;
  const int64_t n = static_cast<int64_t>(blockIdx.x) * (256 / kWave) + threadIdx.x / kWave;
  if (n >= n_sel) return;
  Stat a = empty_stat();
  for (int k = lane; k < splits; k += kWave) a = merge(a, part[static_cast<int64_t>(k) * n_sel + n]);
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) a = merge(a, shfl_xor(a, o));
  if (lane != 0) return;
  const int64_t row = rowsel ? rowsel[n] : n;
  write_scores(a, n, row, ids[row], V, out);
}

// ------------------------------------------------------------------ backward
// dz[n, v] = g (onehot - exp(z - lse)) + entropy term for a chunk of selected rows, z recomputed with the sums of the
// forward pass.  The taken token's entry g (1 - p_y): for a confident token (p_y > 1/2) 1 - p_y cancels down to the error
// of p_y, and the sum of the other probabilities, which carries only their relative error, is taken in its place.
// Rows on the A side, so that sixteen lanes store consecutive vocabulary entries.
// v and y as numbers: with v == y handed over the compiler turns the branches round, and k_dz_f32 is 2 % slower.
template <class Rest>
__device__ __forceinline__ float dz_entry(double z, double l, double g, double en, double k_ent, int v, int y, Rest rest) {
  const double p = exp(z - l);
  const double e = k_ent != 0.0 ? k_ent * p * ((z - l) + en) : 0.0;     // entropy bonus: k p (log p + entropy)
  const double dense = v == y ? g * (p > 0.5 ? rest() : 1.0 - p) : -g * p;
  return static_cast<float>(dense + e);
}
__global__ void __launch_bounds__(kWaves* kWave)
k_dz_f32(const float* __restrict__ W, const float* __restrict__ H, int d, int V, const int32_t* __restrict__ rowsel, int64_t c0,
         int64_t rows, const int32_t* __restrict__ ids, const float* __restrict__ lse_c, const double* __restrict__ rest_c,
         const float* __restrict__ g_c, const float* __restrict__ ent_c, const float* __restrict__ kz_c, float* __restrict__ dz) {
  const int wave = threadIdx.x >> 6;
  const int64_t n0 = static_cast<int64_t>(blockIdx.y) * kTile, vb = static_cast<int64_t>(blockIdx.x) * kVocBlock + wave * kTile;
  if (vb >= V) return;
  const int v0 = static_cast<int>(vb);
  Rows<2> h, w;
  h.vec = w.vec = d % 4 == 0;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int64_t n = c0 + min(n0 + blk_index(i), rows - 1);
    h.p[i] = H + (rowsel ? rowsel[n] : n) * static_cast<int64_t>(d);
    w.p[i] = W + static_cast<int64_t>(min(v0 + blk_index(i), V - 1)) * d;
  }
  double4v acc[2][2];
  zero<2>(acc);
  product<2>(h, w, 0, d, d, acc);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t m = n0 + blk_row(i, r);
      if (m >= rows) continue;
      const int64_t n = c0 + m;
      const int y = ids[rowsel ? rowsel[n] : n];
      const double l = lse_c[n], g = g_c[n], en = ent_c[n], k_ent = kz_c[n];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int v = v0 + blk_index(j);
        if (v >= V) continue;
        dz[m * V + v] = dz_entry(acc[i][j][r], l, g, en, k_ent, v, y, [&] { return rest_c[n]; });
      }
    }
}
// The same from the logits that the scoring pass has kept, where the workspace holds them: one workgroup per row and 1024
// vocabulary entries.  2400 rows of 300 against 4000 156 us as a product, now 22 (and 25 more in the
// scoring pass), 1600 rows of 451 against 5001 253 and 17, 768 rows of 64 against 512 15 and 7.
__global__ void __launch_bounds__(256)
k_dz_kept_f32(const double* __restrict__ z, int V, const int32_t* __restrict__ rowsel, int64_t c0, const int32_t* __restrict__ ids,
              const float* __restrict__ lse_c, const double* __restrict__ rest_c, const float* __restrict__ g_c,
              const float* __restrict__ ent_c, const float* __restrict__ kz_c, float* __restrict__ dz) {
  const int64_t m = blockIdx.y, n = c0 + m;
  const int y = ids[rowsel ? rowsel[n] : n];
  const double l = lse_c[n], g = g_c[n], en = ent_c[n], k_ent = kz_c[n];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int v = blockIdx.x * 1024 + k * 256 + threadIdx.x;
    if (v < V) dz[m * V + v] = dz_entry(z[n * V + v], l, g, en, k_ent, v, y, [&] { return rest_c[n]; });
  }
}

// Few rows: the same, and before it what three more launches do elsewhere - the row's parts merged into its scores, its surrogate -
// by every workgroup of the row for itself, of which there are as many as fill the chip.  The first one leaves the scores.
__global__ void __launch_bounds__(256)
k_row_dz_f32(const double* __restrict__ z, const Stat* __restrict__ part, int splits, int64_t n_sel, int per_wg, Surrogate S, float k_ent,
             float* __restrict__ logp_c, float* __restrict__ ent_c, float* __restrict__ logp_new, float* __restrict__ dz) {
  const int lane = threadIdx.x & (kWave - 1), V = S.V;
  const int64_t n = blockIdx.y, row = S.rowsel ? S.rowsel[n] : n;
  const int y = S.ids[row];
  Stat a = empty_stat();
  for (int k = lane; k < splits; k += kWave) a = merge(a, part[k * n_sel + n]);
  if (a.s == 0.0) a = Stat{-INFINITY, 0.0, 0.0, 0.0, a.zy};   // logits of -infinity only: t is 0 times that
  // every lane's sums relative to the maximum of all, then plain sums: one exponential a lane
  const double m = wave_max(a.m), e = a.s == 0.0 ? 0.0 : exp(a.m - m);
  a = Stat{m, wave_sum(a.s * e), wave_sum(a.t * e), wave_sum(a.rest * e), wave_sum(a.zy)};
  const Scores sc = scores_of(a, y, V);
  const SurrogateRow r = surrogate_row(S, row, sc.ok, sc.lp, sc.en);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    logp_c[n] = sc.lp;
    ent_c[n] = sc.en;
    if (logp_new) logp_new[row] = sc.lp;
  }
  const double l = sc.lse, g = r.g, en = sc.en, kz = sc.ok ? k_ent : 0.f;
  const int v0 = blockIdx.x * per_wg, v1 = min(v0 + per_wg, V);
  for (int vb = v0; vb < v1; vb += 1024)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int v = vb + k * 256 + threadIdx.x;
      if (v < v1) dz[n * V + v] = dz_entry(z[n * V + v], l, g, en, kz, v, y, [&] { return sc.rest; });
    }
}

// The two gradient products, in one launch: neither needs the other, and each alone leaves compute units idle at its end (small ones
// all the time).  A workgroup of eight wavefronts takes WM x WN tiles of NB x NB blocks and 8 / (WM WN) parts of K, whose sums meet in
// LDS in a fixed order: 16 x 16 (SIZE 0) for products that are few tiles altogether, 32 x 32 (1), and 64 x 64 (2), which reads half as
// much from L2 (see gradient_sizes).
constexpr int kGradWaves = 8, kGradT = kGradWaves * kWave;
constexpr int grad_side(int size) { return 16 << size; }
template <int SIZE>
struct GradTile {
  static constexpr int NB = SIZE == 0 ? 1 : 2, W = SIZE == 2 ? 2 : 1;   // blocks of a wavefront and wavefronts, both ways
  static constexpr int kPerWave = NB * NB * 4;                         // accumulators of a lane
  static constexpr int kSums = kGradWaves / 2 * kPerWave * kWave;
};
template <int SIZE, class OA, class OB, class F>
__device__ __forceinline__ void gradient_tile(OA& a, OB& b, int K, double* s_acc, F store) {
  using T = GradTile<SIZE>;
  constexpr int WMN = T::W * T::W, WK = kGradWaves / WMN, NB = T::NB;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, part = wave / WMN;
  const int per = ((K + kK - 1) / kK + WK - 1) / WK * kK;            // k of one part
  double4v acc[NB][NB];
  zero<NB>(acc);
  product<NB>(a, b, min(part * per, K), min((part + 1) * per, K), K, acc);
#pragma unroll
  for (int o = WK / 2; o > 0; o >>= 1) {                             // parts o .. 2 o - 1 hand their sums to parts 0 .. o - 1
    double* const slot = s_acc + static_cast<size_t>(wave % (o * WMN)) * (T::kPerWave * kWave) + lane;
    if (part >= o && part < 2 * o)
#pragma unroll
      for (int q = 0; q < T::kPerWave; ++q) slot[q * kWave] = acc[q / (4 * NB)][q / 4 % NB][q % 4];
    __syncthreads();
    if (part < o)
#pragma unroll
      for (int q = 0; q < T::kPerWave; ++q) acc[q / (4 * NB)][q / 4 % NB][q % 4] += slot[q * kWave];
    __syncthreads();
  }
  if (part != 0) return;
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) store(blk_row(i, r), blk_index(j), acc[i][j][r]);
}
struct GradArgs {
  const float *dz, *W, *H;                   // dz: [rows][V], of the chunk
  int d, V;
  const int32_t* rowsel;
  int64_t c0;
  int rows, accumulate;
  float *dH, *dW;
  int n_dh, n_dw, dw_first;                  // tiles; the longer ones go first
};
// The statistics of the rows, in the gradients' launch: a workgroup for the model and one for each role.
struct StatArgs {
  Surrogate S;
  int64_t n_sel;
  const float *logp_c, *ent_c;
  float entropy_coef;
  int64_t norm_rows;
  umas_loss_stats* stats;                    // NULL: none, and no workgroups for it
};
__device__ __forceinline__ void row_stats(const StatArgs& A, int k, double* smem) {
  double v[kStat] = {}, sum[kStat];
  for (int64_t n = threadIdx.x; n < A.n_sel; n += kGradT) {
    const int64_t row = A.S.rowsel ? A.S.rowsel[n] : n;
    const int y = A.S.ids[row];
    const SurrogateRow r = surrogate_row(A.S, row, y >= 0 && y < A.S.V, A.logp_c[n], A.ent_c[n]);
    if (k > 0 && r.role != k - 1) continue;
    v[0] += r.L; v[1] += r.clipped; v[2] += r.en; v[3] += r.kl; v[4] += 1.0; v[5] += r.valid ? 0.0 : 1.0;
  }
#pragma unroll
  for (int j = 0; j < kStat; ++j) sum[j] = block_sum<double>(v[j], smem);
  if (threadIdx.x == 0) A.stats[k] = loss_stats(sum, k, A.entropy_coef, A.norm_rows);
}
// dH[row(n), j] = sum_v dz[n, v] W[v, j]
template <int SIZE>
__device__ __forceinline__ void dh_tile(const GradArgs& A, int tile, double* s_acc) {
  using T = GradTile<SIZE>;
  const int wave = threadIdx.x >> 6, side = grad_side(SIZE), gx = (A.rows + side - 1) / side;
  const int n0 = tile % gx * side + wave / T::W % T::W * (T::NB * 16), j0 = tile / gx * side + wave % T::W * (T::NB * 16);
  Rows<T::NB> a;
  a.vec = A.V % 4 == 0;
  Cols<T::NB> b;
  b.ld = A.d;
  b.map = nullptr;
#pragma unroll
  for (int i = 0; i < T::NB; ++i) {
    a.p[i] = A.dz + static_cast<int64_t>(min(n0 + blk_index(i), A.rows - 1)) * A.V;
    b.p[i] = A.W + min(j0 + blk_index(i), A.d - 1);
  }
  gradient_tile<SIZE>(a, b, A.V, s_acc, [&](int r, int c, double x) {
    const int m = n0 + r, j = j0 + c;
    if (m < A.rows && j < A.d) A.dH[(A.rowsel ? A.rowsel[A.c0 + m] : A.c0 + m) * A.d + j] = static_cast<float>(x);
  });
}
// dW[v, j] (+)= sum_n dz[n, v] H[row(n), j]
template <int SIZE>
__device__ __forceinline__ void dw_tile(const GradArgs& A, int tile, double* s_acc) {
  using T = GradTile<SIZE>;
  const int wave = threadIdx.x >> 6, side = grad_side(SIZE), gx = (A.V + side - 1) / side;
  const int v0 = tile % gx * side + wave / T::W % T::W * (T::NB * 16), j0 = tile / gx * side + wave % T::W * (T::NB * 16);
  Cols<T::NB> a, b;
  a.ld = A.V;
  a.map = nullptr;
  b.ld = A.d;
  b.map = A.rowsel ? A.rowsel + A.c0 : nullptr;
#pragma unroll
  for (int i = 0; i < T::NB; ++i) {
    a.p[i] = A.dz + min(v0 + blk_index(i), A.V - 1);
    b.p[i] = (A.rowsel ? A.H : A.H + A.c0 * A.d) + min(j0 + blk_index(i), A.d - 1);
  }
  gradient_tile<SIZE>(a, b, A.rows, s_acc, [&](int r, int c, double x) {
    const int v = v0 + r, j = j0 + c;
    if (v >= A.V || j >= A.d) return;
    float* dst = A.dW + static_cast<int64_t>(v) * A.d + j;
    *dst = A.accumulate ? static_cast<float>(static_cast<double>(*dst) + x) : static_cast<float>(x);
  });
}
template <int DH, int DW>
__global__ void __launch_bounds__(kGradT)
k_gradients_f32(GradArgs A, StatArgs T) {
  __shared__ double s_acc[GradTile<DH>::kSums > GradTile<DW>::kSums ? GradTile<DH>::kSums : GradTile<DW>::kSums];
  const int i = blockIdx.x, n_first = A.dw_first ? A.n_dw : A.n_dh;
  if (i >= A.n_dh + A.n_dw) {
    row_stats(T, i - A.n_dh - A.n_dw, s_acc);
    return;
  }
  if ((i < n_first) != (A.dw_first != 0)) dh_tile<DH>(A, i < n_first ? i : i - n_first, s_acc);
  else dw_tile<DW>(A, i < n_first ? i : i - n_first, s_acc);
}

// ------------------------------------------------------------------ launches
// Workgroups per block of 32 rows: enough of them to fill the chip, as far as the vocabulary and the room for their
// statistics go.
inline int score_splits(int64_t n_sel, int V, size_t room) {
  const int64_t row_blks = (n_sel + kTile - 1) / kTile;
  int64_t k = (1024 + row_blks - 1) / row_blks;
  k = k < cdiv(V, kVocBlock) ? k : cdiv(V, kVocBlock);
  const int64_t fit = static_cast<int64_t>(room / (static_cast<size_t>(n_sel) * sizeof(Stat)));
  return static_cast<int>(k < fit ? k : fit < 1 ? 1 : fit);
}
// Parts of the update in few launches: every block of the vocabulary, up to as many as a wavefront merges at once.  Tiles of 16 while those
// of 32 are about one to a compute unit.  Scores of 768 rows of 64 against 512 (96 tiles of 32) 16 -> 13 us, 300 of 500 against 300 (30)
// 47 -> 20.5, 1000 of 300 against 700 (192) 41 -> 25, 100 of 512 against 8000 (252) 59 -> 55, 1200 of 64 against 800 (266) 19 -> 17.
constexpr int kSmallScoreTiles = 300;
struct PartPlan {
  int side, splits;
};
inline PartPlan part_plan(int64_t n_sel, int V) {
  const int64_t wide = cdiv(n_sel, kTile) * static_cast<int64_t>(cdiv(V, kVocBlock));
  if (wide > kSmallScoreTiles) return PartPlan{kTile, score_splits(n_sel, V, SIZE_MAX)};
  const int blks = static_cast<int>(cdiv(V, kVocBlock / 2));
  return PartPlan{kTile / 2, blks < kWave ? blks : kWave};
}
inline size_t score_room(int64_t n_sel, int V) {
  if (n_sel <= 0) return 0;
  const int k = score_splits(n_sel, V, SIZE_MAX);
  return k > 1 ? static_cast<size_t>(k) * n_sel * sizeof(Stat) : 0;
}
// The row kernel where a thread of its has little to do (about 30 ns a product at 512 x 8192; the tiles cost a launch more):
// 24 rows against 512 of width 64 / 128 take 10 / 13 us, in tiles 20 / 22, 768 rows of 64 19 and 18, 1 row of 128 against 3000
// 47 and 20.  And where the room holds only `splits` of the parts that would be taken and the row kernel's rounds of 256
// workgroups are few: tiles take the time of five to six rounds divided by the splits.  512 x 8192 without room: 256 / 1024 /
// 1300 / 1500 / 8192 rows 0.57 / 2.11 / 3.17 / 3.14 / 17.4 ms in the row kernel, 2.88 / 2.88 / 2.87 / 2.87 / 3.04 in tiles; 256 x 32 000:
// 700 rows 2.73, with two parts in tiles 2.94, 500 rows 1.95, three parts 1.98, 256 rows 1.10, five parts 1.19, six 1.00.
inline umas_status score(const float* W, const float* H, int d, int V, const int32_t* rowsel, int64_t n_sel, const int32_t* ids, void* room,
                         size_t room_bytes, const ScoreOut& out, hipStream_t st) {
  const int splits = score_splits(n_sel, V, room_bytes);
  const int64_t per_thread = static_cast<int64_t>(cdiv(V, 256)) * d;
  const int64_t rounds = (n_sel + 255) / 256;
  const bool tight = splits < 6 && rounds < 6 && splits * rounds <= 6 && splits < score_splits(n_sel, V, SIZE_MAX);
  if ((n_sel <= 1024 && per_thread <= 128) || (n_sel <= 128 && per_thread <= 256) || tight) {
    auto row = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(n_sel)), dim3(256), d * sizeof(float), st, W, H, d, V, rowsel, ids, out); };
    if (out.z) row(k_score_f32_row<true>);
    else row(k_score_f32_row<false>);
    UMAS_LAUNCHED("k_score_f32_row");
    return UMAS_OK;
  }
  auto tiles = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(cdiv(n_sel, kTile), splits), dim3(kWaves * kWave), 0, st, W, H, d, V, rowsel, n_sel, ids,
                       splits > 1 ? static_cast<Stat*>(room) : nullptr, out, splits, ClearArgs{});
  };
  if (out.z) tiles(k_score_f32<true, 2>);
  else tiles(k_score_f32<false, 2>);
  UMAS_LAUNCHED("k_score_f32");
  if (splits > 1) {
    hipLaunchKernelGGL(k_score_f32_merge, dim3(cdiv(n_sel, 256 / kWave)), dim3(256), 0, st, static_cast<const Stat*>(room), splits, V,
                       rowsel, n_sel, ids, out);
    UMAS_LAUNCHED("k_score_f32_merge");
  }
  return UMAS_OK;
}
// 64 x 64 where its tiles fill whole rounds of 256 compute units, or nearly: it takes as long as the rounds, 32 x 32 a tenth longer than
// the tiles would in full ones (dW of 4000 x 300, 315 tiles: 257 us in 64 x 64, 184 in 32 x 32; 5001 x 451, 632: 221 and 202; 8192
// x 512, 1024: 164 and 179).  Nearly one round is no case for them: a single workgroup to a compute unit (dW of 15 000 x 64, 235 tiles, 2000 rows
// 166 in 64 x 64, 125 in 32 x 32, 4000 rows 338 and 235; 8000 x 120, 250: 153 and 124; 7600 x 128, 238: 87 and 70).
inline bool large_product(int64_t m, int64_t n) {
  const int64_t tiles = cdiv(m, 64) * static_cast<int64_t>(cdiv(n, 64));
  return tiles >= 256 && (tiles + 255) / 256 * 256 * 10 <= tiles * 11;
}
// 16 x 16 where the product's tiles of 32 x 32 are fewer than every second compute unit, or those of both together one each: then a
// launch lasts as long as one tile, and that is a quarter as many instructions a round.  Both products, in two launches of 32 x 32 and
// in one: 768 rows of 64 against 512 33 -> 12.5 us, 1500 of 64 against 2000 74 -> 38.5, 100 of 512
// against 8000 153 -> 66 (122 with dH in 32 x 32), 6000 of 128 against 512 88 -> 43.5 (69 with dW in 32 x 32).
constexpr int kSmallGradTiles = 256;
inline void launch_gradients(GradArgs A, const StatArgs& T, hipStream_t st) {
  auto tiles = [](int64_t m, int64_t n, int size) { return static_cast<int>(cdiv(m, grad_side(size)) * cdiv(n, grad_side(size))); };
  const int dh1 = tiles(A.rows, A.d, 1), dw1 = tiles(A.V, A.d, 1);
  const bool small = dh1 + dw1 <= kSmallGradTiles;
  auto size = [&](int64_t m, int tiles1) { return small || tiles1 <= kSmallGradTiles / 2 ? 0 : large_product(m, A.d) ? 2 : 1; };
  const int dh = size(A.rows, dh1), dw = size(A.V, dw1);
  const int n_dh = tiles(A.rows, A.d, dh), n_dw = tiles(A.V, A.d, dw);
  A.dw_first = A.rows > A.V ? 1 : 0;
  auto launch = [&](int some_dh, int some_dw, const StatArgs& S) {
    A.n_dh = some_dh;
    A.n_dw = some_dw;
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(some_dh + some_dw + (S.stats ? 1 + S.S.n_roles : 0))), dim3(kGradT), 0, st, A, S);
    };
    switch (3 * dh + dw) {
      case 0: return go(k_gradients_f32<0, 0>);
      case 1: return go(k_gradients_f32<0, 1>);
      case 2: return go(k_gradients_f32<0, 2>);
      case 3: return go(k_gradients_f32<1, 0>);
      case 4: return go(k_gradients_f32<1, 1>);
      case 5: return go(k_gradients_f32<1, 2>);
      case 6: return go(k_gradients_f32<2, 0>);
      case 7: return go(k_gradients_f32<2, 1>);
      default: return go(k_gradients_f32<2, 2>);
    }
  };
  const int64_t n_w = static_cast<int64_t>(A.V) * A.d;
  if (A.dW + n_w <= A.W || A.W + n_w <= A.dW) return launch(n_dh, n_dw, T);
  launch(n_dh, 0, StatArgs{});               // dW lies over the weights, which dH has to have read by then
  launch(0, n_dw, T);
}

// An update of one chunk of rows that keeps its logits, in three launches: the scores of parts of the vocabulary and the clearing, dz with all
// that is per row in front of it, both gradient products and the statistics.  In six or seven it takes, with the same gradients' launch, 768 rows of 64 against
// 512 45 us and now 28, 300 of 500 against 300 79 and 39, 1000 of 128 against 1000 70 and 54, 4000 of 64 against 4000 277 and 268.
struct UpdateArgs {
  const float *W, *H;
  int d;
  int64_t n_sel, n_rows;
  Surrogate S;
  float k_ent, entropy_coef;
  int64_t norm_rows;
  float *logp_c, *ent_c, *logp_new;
  double* z;
  Stat* part;
  float *dz, *dH, *dW;
  int accumulate;
  umas_loss_stats* stats;
};
inline umas_status update(const UpdateArgs& A, hipStream_t st) {
  const int V = A.S.V;
  const PartPlan plan = part_plan(A.n_sel, V);
  const int splits = plan.splits;
  ClearArgs clear{};
  unsigned n_clear = 0;                      // in rows of the grid
  if (A.S.rowsel) {
    clear = ClearArgs{{reinterpret_cast<uint32_t*>(A.logp_new), reinterpret_cast<uint32_t*>(A.dH), nullptr}, {A.n_rows, A.n_rows * A.d, 0}};
    const unsigned wg = cdiv(static_cast<size_t>(A.n_rows) * A.d, 2048);
    n_clear = cdiv(wg < 1024 ? wg : 1024, cdiv(A.n_sel, plan.side));
  }
  auto score = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(cdiv(A.n_sel, plan.side), splits + n_clear), dim3(kWaves * kWave), 0, st, A.W, A.H, A.d, V, A.S.rowsel, A.n_sel,
                       A.S.ids, A.part, ScoreOut{A.z, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr}, splits, clear);
  };
  if (plan.side == kTile) score(k_score_f32<true, 2>);
  else score(k_score_f32<true, 1>);
  UMAS_LAUNCHED("k_score_f32");
  const unsigned wgs = cdiv(2048, static_cast<size_t>(A.n_sel)), most = cdiv(V, 1024);      // eight workgroups to a compute unit
  const int per_wg = static_cast<int>(cdiv(most, wgs < most ? wgs : most)) * 1024;
  hipLaunchKernelGGL(k_row_dz_f32, dim3(cdiv(V, per_wg), static_cast<unsigned>(A.n_sel)), dim3(256), 0, st, A.z, A.part, splits, A.n_sel, per_wg, A.S, A.k_ent,
                     A.logp_c, A.ent_c, A.logp_new, A.dz);
  UMAS_LAUNCHED("k_dz_kept_f32");            // the timing aid's names are those of the steps, in few launches or many: kept logits into dz, the gradients
  launch_gradients(GradArgs{A.dz, A.W, A.H, A.d, V, A.S.rowsel, 0, static_cast<int>(A.n_sel), A.accumulate, A.dH, A.dW, 0, 0, 0},
                   StatArgs{A.S, A.n_sel, A.logp_c, A.ent_c, A.entropy_coef, A.norm_rows, A.stats}, st);
  UMAS_LAUNCHED("k_dw_f32");
  return UMAS_OK;
}

}  // namespace f32
}  // namespace umas
