// LM-head scoring, the clipped PPO surrogate and the backward through the LM head.
//
// Scoring ("old log probabilities", paragraph "Advantage computation and policy evaluation"):
// for every selected row z = W h, lse = log sum exp z, logp = z[y] - lse, entropy = lse -
// sum softmax(z) z.  The bf16 path computes 256x256 logit tiles with MFMA and reduces each tile
// to per-row (max, sum exp, sum exp*z, taken logit) in registers; logits never leave the chip.
// Update (paragraph "Model-specific updates and synchronization", PPO after Schulman et al.
// 2017): ratio = exp(logp - logp_old), L = max(-A ratio, -A clip(ratio)), g = dL/dlogp, then
// dH = dz W and dW = dz^T H with dz = g (onehot - softmax) run as MFMA GEMMs over a bf16 operand
// [rows, vocabulary] held in a bounded chunk buffer; W is read as it lies, of H dW reads a copy of the chunk's rows
// in column blocks (operands that are not K-contiguous go through transposing LDS reads); the one-hot part (one term
// per row) is added in float32.
// Without an entropy bonus the dense part of dz is a row factor times the softmax, so the scoring pass of
// the update itself leaves that operand behind: E = bf16(exp(z - z_y)), the softmax numerators relative to
// the taken token's logit, and the row factor -g exp(z_y - lse) is applied where dH is written and folded
// into the copy of H that dW reads; the logits are computed once.  With an entropy bonus the
// scoring pass leaves the float32 logits behind, which one pass over them turns into dz; in a workspace without room
// for them, for narrow heads (and for blocks of rows whose logits spread too far for E) dz is recomputed tile by tile from H, W and lse.
// The float32 path, for small shapes, carries its sums in float64 (umas_f32.h).
#include <math.h>

#include <algorithm>
#include <mutex>

#include "umas_common.h"
#include "umas_f32.h"
#include "umas_mfma.h"
#include "umas_plan.h"
#include "umas_surrogate.h"

namespace umas {
namespace {

using Cfg = TileCfg<256, 256, 2, 4>;   // 8 wavefronts, two per SIMD: one issues memory operations while the other feeds the matrix pipe
using Ring = Ring2Cfg<Cfg>;
constexpr int kLogitLds = Ring::LDS_BYTES;
constexpr int kGM = 4, kGN = 8;          // tile group resident on one XCD
constexpr int kTilesPerWg = 4;           // logit tiles a workgroup computes one after the other (short K: launch gaps and store drain overlap)
constexpr int kRowBlock = 256;
constexpr float kNegInf = -INFINITY;
constexpr float kMasked = -1e30f;        // stands for a logit that does not exist (vocabulary tail)

__device__ __forceinline__ uint16_t f2bf(float x) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(x));
}
// two floats rounded to bf16 in one word (first in the low half): one conversion instruction
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

// Online-softmax partial: m = max z, s = sum exp(z - m), t = sum exp(z - m) z.
struct Part {
  float m, s, t;
};
__device__ __forceinline__ Part part_merge(Part x, Part y) {
  if (x.m == kNegInf) return y;
  if (y.m == kNegInf) return x;
  const float M = fmaxf(x.m, y.m);
  const float ex = __expf(x.m - M), ey = __expf(y.m - M);
  return Part{M, fmaf(x.s, ex, y.s * ey), fmaf(x.t, ex, y.t * ey)};   // written out: the same rounding in every kernel
}

// ------------------------------------------------------------------ small helpers
__global__ void __launch_bounds__(256) k_clear(ClearArgs A) {
  clear_words(A, static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x, static_cast<int64_t>(gridDim.x) * blockDim.x);
}

// bytes are a multiple of 4 for every buffer cleared here
hipError_t clear_bytes(hipStream_t st, void* a, size_t bytes_a, void* b = nullptr, size_t bytes_b = 0, void* c = nullptr, size_t bytes_c = 0) {
  const ClearArgs A{{static_cast<uint32_t*>(a), static_cast<uint32_t*>(b), static_cast<uint32_t*>(c)},
                    {static_cast<int64_t>(bytes_a / 4), static_cast<int64_t>(bytes_b / 4), static_cast<int64_t>(bytes_c / 4)}};
  int64_t most = 0;
  for (int k = 0; k < 3; ++k) most = A.p[k] ? std::max(most, A.words[k]) : most;
  if (most == 0) return hipSuccess;
  hipLaunchKernelGGL(k_clear, dim3(static_cast<unsigned>(std::min<int64_t>(most / 256 + 1, 65536))), dim3(256), 0, st, A);
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess && g_prof_on) prof_kernel("k_clear", st);
  return e;
}

// Where every weight is read by one tile only (one column tile) and W is larger than the memory-side cache, it is read past it: 203
// rows of 3584 against 152 064, keeping 300 -> 270 us, 100 and 200 rows of 2048 against 151 936, scoring 153 -> 143 and 187 -> 182.
// A smaller W may still lie there from the call before (250 rows of 1024 against 30 001, 61 MB: 28 us, past the cache 31), and
// the better part of one that is a little larger: scoring 256 rows through the cache and past it on two cards, W of 257 MiB 102 and 114, 109 and
// 116 us (d = 2048), 87 and 96, 89 and 96 (4096), 272 MiB 108 and 116, 119 and 117, 288 MiB 115 and 117, 123 and 119, 312 MiB 117
// and 117, 125 and 120.  dH, which reads its other operand several times meanwhile, has its line at 256 MiB (update of 256 rows
// of 1024, 264 MiB: 370 and 343, 384 and 358).
constexpr int64_t kLogitsOnceBytes = int64_t{300} << 20, kDhOnceBytes = int64_t{256} << 20;
__device__ __forceinline__ bool beyond_cache(int d, int V, int64_t bytes) { return static_cast<int64_t>(V) * d * 2 > bytes; }

// Logit tile Z[v, n] = W[m0 + v, :] . H[row(n0 + n), :] for a 256x256 block of (vocabulary, selected rows),
// row(n) = rowsel[sel0 + n] or sel0 + n.  Rows past V and past n_lim are clamped to valid ones; the
// callers mask what comes out of them.
template <class C>
__device__ __forceinline__ void logit_tile(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, int d, int V,
                                           const int32_t* __restrict__ rowsel, int64_t sel0, int64_t n_lim, int m0,
                                           int64_t n0, bool w_once, uint16_t* lds, floatx4 (&acc)[C::MI][C::NI]) {
#pragma unroll
  for (int i = 0; i < C::MI; ++i)
#pragma unroll
    for (int j = 0; j < C::NI; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  using R = Ring2Cfg<C>;
  const uint32_t kofs = ring2_kofs();
  uint32_t oa[R::NA], ob[R::NB];
#pragma unroll
  for (int i = 0; i < R::NA; ++i) oa[i] = (static_cast<uint32_t>(min(ring2_row<C>(i), V - 1 - m0)) * d + kofs) * 2u;
#pragma unroll
  for (int i = 0; i < R::NB; ++i) {
    const int64_t n = sel0 + min(n0 + ring2_row<C>(i), n_lim - 1);
    ob[i] = (static_cast<uint32_t>(rowsel ? rowsel[n] : n) * d + kofs) * 2u;   // host checks n_rows*d*2 < 2^32
  }
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(W + static_cast<int64_t>(m0) * d), rb = make_rsrc(H);
  if (d % C::BK != 0) mfma_mainloop_ring2<C, true, kCached>(ra, oa, rb, ob, d, lds, acc);
  else if (w_once) mfma_mainloop_ring2<C, false, kStream>(ra, oa, rb, ob, d, lds, acc);
  else mfma_mainloop_ring2<C, false, kCached>(ra, oa, rb, ob, d, lds, acc);
}

// ------------------------------------------------------------------ bf16: logit tiles -> partials
// A = W (vocabulary rows on the M side, so one lane sees many vocabulary entries of one token),
// B = rows c0 .. c0 + mc - 1 of the selection.  partial[tile_m][n] = (m, s, t, taken logit or 0).
//
// The keeping variant serves the backward pass when the dense part of dz is a row factor times the softmax
// (no entropy bonus): it also writes E[n, v] = bf16(exp(z[n, v] - c_n)) to the chunk buffer [mcp, Vp], c_n a
// per-row reference known before the pass (the taken token's logit), so that dz = (a_n exp(c_n - lse_n)) E
// needs no second pass over the logits: the row factor is applied where dH is written and folded into the
// copy of H that dW reads.  A block of 256 rows in which some logit exceeds its reference by more than kKeepMaxGap
// (E could overflow) is flagged and gets its dz from the recomputing kernel instead.
constexpr float kKeepMaxGap = 50.f;
// The [rows, vocabulary] operand of the backward (E, or dz on the recomputing path) lies in blocks of 256 rows x 256
// vocabulary entries, 128 KB each, row-major inside, vocabulary blocks of one block row next to each other: what a
// gradient tile reads per K step is then one run of memory (32 KB of consecutive rows for dW, four steps per block
// for dH) instead of 256 or 64 pieces a row pitch of 300 KB apart.
constexpr int64_t kBlkElems = 256 * 256;
__host__ __device__ __forceinline__ int64_t blk_offset(int64_t row_blk, int64_t voc_blk, int64_t tiles_v) {
  return (row_blk * tiles_v + voc_blk) * kBlkElems;
}
template <class C>
struct Stage {                                                                  // every wavefront stages its block: WTN rows x WTM vocabulary entries
  static constexpr int kPitch = C::WTM * 2 + 16;                                // one staged row of bf16, 16-byte aligned
  static constexpr int kBytes = C::WM * C::WN * C::WTN * kPitch;
};
constexpr int kStagePitch = Stage<Cfg>::kPitch;
constexpr int kLogitPitch = Cfg::WTM * 4 + 16;                                  // one staged row of logits: 128 floats
static_assert(kLogitLds <= 160 * 1024, "LDS of one CU");

enum class Leave { kNothing, kNumerators, kLogits };   // what a scoring pass leaves behind for the backward
struct KeepArgs {
  const float* cref;   // [n_pad] reference per selected row, NaN for rows without a valid id
  uint16_t* E;         // [mcp, Vp]
  int64_t Vp;
  int32_t* flags;      // per block of 256 selected rows
  const int32_t* cidx; // per block of 256 selected rows: its place among the chunk's live blocks, -1 for a dead one
  float* Z;            // Leave::kLogits: the logits, in blocks of 256 x 256 floats in the place and order of the operand's blocks
};

template <Leave LEAVE, class C>
__device__ __forceinline__ void score_tile(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, int d, int V,
                                           const int32_t* __restrict__ rowsel, int64_t c0, int64_t mc,
                                           const int32_t* __restrict__ ids, int tile_m, int tile_n, bool w_once,
                                           float4* __restrict__ partial, int64_t n_pad, const KeepArgs& keep,
                                           uint16_t* lds) {
  constexpr bool KEEP = LEAVE == Leave::kNumerators;
  static_assert(LEAVE != Leave::kLogits || (C::BM == 256 && C::WTM == Cfg::WTM), "logits are kept in rows of 128 of a block's 256 entries");
  static_assert(256 % C::BM == 0 && 256 % C::BN == 0, "numerators are kept inside a block");
  constexpr int kPitch = Stage<C>::kPitch;
  constexpr int kLds = C::T == Cfg::T ? kLogitLds : Ring2Cfg<C>::LDS_BYTES;   // halves of a tile use the whole one's buffers
  static_assert(Ring2Cfg<C>::LDS_BYTES <= kLds, "the main loop's stages fit");
  static_assert((LEAVE == Leave::kNothing ? 0 : Stage<C>::kBytes) + (C::WM * C::BN * 3 + C::BN) * 4 <= kLds, "staging and the partials fit the tile buffers");
  static_assert(LEAVE != Leave::kLogits || 16 * kLogitPitch <= C::WTN * kPitch, "sixteen rows of logits fit a wavefront's stage");
  const int m0 = tile_m * C::BM;
  const int64_t n0 = static_cast<int64_t>(tile_n) * C::BN;   // chunk-relative
  floatx4 acc[C::MI][C::NI];
  // (a tile that lies past V as a whole, the second half of a block that is kept, reads the last entry)
  logit_tile<C>(W, H, d, V, rowsel, c0, mc, min(m0, V - 1), n0, w_once, lds, acc);

  // epilogue: the tile buffers are free now.  A lane holds, for each of its NI columns (selected rows), the
  // vocabulary entries vbase + 16 i + r (i < MI, r < 4); the four lanes l, l + 16, l + 32, l + 48 share a column.
  float* s_part = reinterpret_cast<float*>(reinterpret_cast<char*>(lds) + (LEAVE == Leave::kNothing ? 0 : Stage<C>::kBytes));   // [WM][BN][3], behind the staging area
  float* s_zy = s_part + C::WM * C::BN * 3;               // [BN]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / C::WN;
  char* stage = reinterpret_cast<char*>(lds) + wave * (LEAVE == Leave::kLogits ? 16 * kLogitPitch : C::WTN * kPitch);
  if (threadIdx.x < C::BN) s_zy[threadIdx.x] = 0.f;
  __syncthreads();                                        // every wavefront has left the main loop's LDS reads
  const int vbase = m0 + wm * C::WTM + (lane >> 4) * 4;   // vocabulary id of element (i = 0, r = 0)
  const bool tail = m0 + C::BM > V;
  if (tail) {   // vocabulary ids past V: a large negative logit whose exponential is 0 and whose products stay finite
#pragma unroll
    for (int i = 0; i < C::MI; ++i)
#pragma unroll
      for (int j = 0; j < C::NI; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (vbase + i * 16 + r >= V) acc[i][j][r] = kMasked;
  }
  constexpr float kLog2e = 1.44269504088896341f;
  bool over = false;
  // a block of rows none of which has a gradient (all advantages 0) keeps nothing: the backward never looks at it
  const int64_t row_blk = (c0 + n0) >> 8;
  const int out_blk = KEEP ? keep.cidx[row_blk] : -1;
  const bool keeping = KEEP && out_blk >= 0;
#pragma unroll
  for (int j = 0; j < C::NI; ++j) {
    const int col = acc_col<C>(j);
    const int64_t n = n0 + col;
    // exponentials of this lane's entries of column j relative to m (log2 domain), their sum s and sum of e z; the
    // keeping variant stages them as bf16 in this wavefront's LDS region, stored in full lines below
    float m = kMasked, s = 0.f, t = 0.f;
    auto column = [&](float ref, auto premultiplied) {
      const float r2 = ref * kLog2e;
      s = 0.f;
      t = 0.f;
#pragma unroll
      for (int i = 0; i < C::MI; ++i) {
        float e[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float z = acc[i][j][r];
          // without a reference from outside: z - m first, exact 0 where a lane holds nothing but vocabulary tail
          e[r] = decltype(premultiplied)::value ? __builtin_amdgcn_exp2f(fmaf(z, kLog2e, -r2)) : __builtin_amdgcn_exp2f((z - ref) * kLog2e);
          s += e[r];
          t = fmaf(e[r], z, t);
        }
        if (keeping) {
          const uint32_t p01 = pack_bf16x2(e[0], e[1]), p23 = pack_bf16x2(e[2], e[3]);
          *reinterpret_cast<uint2*>(stage + (j * 16 + (lane & 15)) * kPitch + (i * 16 + (lane >> 4) * 4) * 2) =
              make_uint2(p01, p23);
        }
      }
    };
    auto lane_max = [&]() {
      float mx = kMasked;
#pragma unroll
      for (int i = 0; i < C::MI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, acc[i][j][r]);
      return mx;
    };
    if (keeping) {
      // The keeping variant sums relative to the row's reference c_n instead of the lane's maximum (any reference
      // serves the merge as long as nothing overflows), so the exponentials it sums are the numerators it keeps,
      // and it does not look for the maximum first: a sum beyond 32 e^kKeepMaxGap (or not a number: rows without
      // a valid id have the reference NaN) shows afterwards that some logit may lie more than kKeepMaxGap above
      // c_n.  Only then is the column done again the long way, relative to the lane's maximum: a lane whose maximum
      // does lie that far above c_n flags the block (its dz is recomputed later); rows without a valid id flag
      // nothing, their row factor is 0.
      const float c = n < mc ? keep.cref[c0 + n] : 1e30f;   // rows past the chunk: every exponential is 0, E = 0
      m = c;
      column(c, std::true_type{});
      constexpr float kSumLimit = 1.6e23f;                   // 32 e^50 = 1.66e23
      if (!(s < kSumLimit)) {
        m = lane_max();
        const float gap = m - c;
        over |= gap > kKeepMaxGap;
        if (gap <= kKeepMaxGap) m = c;                       // many large terms, none too large: c serves after all
        else if (m == kMasked) m = 0.f;                     // nothing but vocabulary tail in this lane: exponentials 0 as well
        column(m, std::true_type{});
      }
    } else {
      m = lane_max();
      column(m, std::false_type{});
    }
    if (LEAVE == Leave::kLogits) {
      // sixteen rows of 128 logits through the wavefront's part of LDS, so that a store covers 512 bytes of two rows
#pragma unroll
      for (int i = 0; i < C::MI; ++i)
        *reinterpret_cast<floatx4*>(stage + (lane & 15) * kLogitPitch + (i * 16 + (lane >> 4) * 4) * 4) = acc[i][j];
      __builtin_amdgcn_wave_barrier();
      float* out = keep.Z + blk_offset(n0 >> 8, tile_m, keep.Vp >> 8) + ((n0 & 255) + wave % C::WN * C::WTN + j * 16 + (lane >> 5)) * 256 + wm * C::WTM + (lane & 31) * 4;
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (n0 + wave % C::WN * C::WTN + j * 16 + q * 2 + (lane >> 5) < mc)   // rows past the chunk: nobody reads them
          __builtin_nontemporal_store(*reinterpret_cast<const floatx4*>(stage + (q * 2 + (lane >> 5)) * kLogitPitch + (lane & 31) * 16),
                                      reinterpret_cast<floatx4*>(out + q * 512));
      __builtin_amdgcn_wave_barrier();
    }
    Part p{m, s, t};
#pragma unroll
    for (int o = 16; o < kWave; o <<= 1) {
      const Part q{__shfl_xor(p.m, o, kWave), __shfl_xor(p.s, o, kWave), __shfl_xor(p.t, o, kWave)};
      p = part_merge(p, q);
    }
    if (lane < 16) {
      float* dst = s_part + (wm * C::BN + col) * 3;
      dst[0] = p.m; dst[1] = p.s; dst[2] = p.t;
    }
    if (!KEEP && n < mc) {                                  // the keeping variant got the taken logits beforehand
      const int y = ids[rowsel ? rowsel[c0 + n] : c0 + n];
      const int rel = y - vbase;                           // offset from this lane's first element
      if (y >= 0 && y < V && rel >= 0 && rel < C::WTM && (rel & 12) == 0) {
        float zy = 0.f;
#pragma unroll
        for (int i = 0; i < C::MI; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (i * 16 + r == rel) zy = acc[i][j][r];
        s_zy[col] = zy;
      }
    }
  }
  if (keeping) {
    if (over) keep.flags[row_blk] = 1;
    // the staged block goes out 16 bytes per lane: one instruction covers 4 rows x 256 contiguous bytes (of 64 entries a row, 8 x 128)
    constexpr int kLanes = C::WTM / 8, kRows = kWave / kLanes;
    const int wn = wave % C::WN;
    uint16_t* out = keep.E + blk_offset(out_blk, m0 >> 8, keep.Vp >> 8) + ((n0 & 255) + wn * C::WTN) * 256 + (m0 & 255) + wm * C::WTM + lane % kLanes * 8;
#pragma unroll 8
    for (int i = 0; i < C::WTN / kRows; ++i) {
      const int row = i * kRows + lane / kLanes;
      const uint4 v = *reinterpret_cast<const uint4*>(stage + row * kPitch + lane % kLanes * 16);
      typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
      __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4*>(out + row * 256));
    }
  }
  __syncthreads();
  if (threadIdx.x < C::BN) {
    const int col = threadIdx.x;
    Part p{kNegInf, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < C::WM; ++w) {
      const float* src = s_part + (w * C::BN + col) * 3;
      p = part_merge(p, Part{src[0], src[1], src[2]});
    }
    if (c0 + n0 + col < n_pad) partial[static_cast<int64_t>(tile_m) * n_pad + c0 + n0 + col] = make_float4(p.m, p.s, p.t, s_zy[col]);
  }
  __syncthreads();                              // the LDS is the next tile's again
}

// The tiles of a workgroup.  With few column tiles a workgroup has one tile, and the last round of compute units is often nearly empty: the tiles of
// one that is at most half full are cut into two of 128 rows of the selection.  594 tiles on 256 compute units, 256 rows: 2048 columns 190 -> 173 us, 3584
// 283 -> 270; 150 rows 188 -> 170 and 271 -> 262; the update of 203 rows of 3584 1037 -> 1022, with an entropy bonus 1056 -> 1026, 100 rows of 2048 609 ->
// 584.  (Up to 128 rows all tiles cut, whose other halves have no rows: 100 rows with a bonus 611, of 3584 957 -> 1036.)  Up to eight column tiles, beyond which
// a workgroup has several: 300, 1000 and 2000 rows of 1536 against 33 001 86.7 -> 76.6, 126.5 -> 114.9 and 204.9 -> 193.5, of 1024 against 100 001
// 130.1 -> 119.9, 217.8 -> 208.5 and 389.7 -> 382.4, of 2048 against 151 936 294.2 -> 276.9, 553.2 -> 547.4 and 1014 -> 1023, 900 of 3584 918 -> 900; where
// the last round is fuller nothing changes.
using HalfCfg = TileCfg<256, 128, 2, 4>;                 // the lanes of a row as in a whole tile: the same bits
template <Leave LEAVE, class C>
__device__ __forceinline__ void score_tiles(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, int d, int V,
                                            const int32_t* __restrict__ rowsel, int64_t c0, int64_t mc,
                                            const int32_t* __restrict__ ids, int tiles_m, int tiles_n, int panel,
                                            float4* __restrict__ partial, int64_t n_pad, const KeepArgs& keep,
                                            uint16_t* lds, int halved = 0) {
  const bool w_once = tiles_n == 1 && beyond_cache(d, V, kLogitsOnceBytes);
  if constexpr (C::BM == 256 && C::BN == 256) {
    if (halved > 0) {                             // the last `halved` tiles of every XCD
      const int per_xcd = (tiles_m * tiles_n + 7) / 8, xcd = static_cast<int>(blockIdx.x & 7), w = static_cast<int>(blockIdx.x >> 3), whole = per_xcd - halved;
      if (w >= whole) {
        const int in_xcd = whole + (w - whole) / 2, t = xcd * per_xcd + in_xcd, tile_m = t / tiles_n, half = t % tiles_n * 2 + ((w - whole) & 1);
        if (in_xcd < per_xcd && tile_m < tiles_m && half * HalfCfg::BN < mc)
          score_tile<LEAVE, HalfCfg>(W, H, d, V, rowsel, c0, mc, ids, tile_m, half, false, partial, n_pad, keep, lds);
        return;
      }
    }
  }
  for (int it = 0; it < kTilesPerWg; ++it) {     // a workgroup walks the same place of kTilesPerWg consecutive tile groups
    int tile_m, tile_n;
    if (!tile_coords<kGM, kGN>(tiles_m, tiles_n, panel, &tile_m, &tile_n, it, kTilesPerWg)) continue;
    score_tile<LEAVE, C>(W, H, d, V, rowsel, c0, mc, ids, tile_m, tile_n, w_once, partial, n_pad, keep, lds);
  }
}

// (kernel templates whose bodies use buffer resources do not get their host stubs emitted: plain kernels)
__global__ void __launch_bounds__(Cfg::T)
k_score_tiles(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, int d, int V,
              const int32_t* __restrict__ rowsel, int64_t n_sel, const int32_t* __restrict__ ids,
              int tiles_m, int tiles_n, int panel, int halved, float4* __restrict__ partial, int64_t n_pad) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[kLogitLds / 2];
  score_tiles<Leave::kNothing, Cfg>(W, H, d, V, rowsel, 0, n_sel, ids, tiles_m, tiles_n, panel, partial, n_pad, KeepArgs{}, lds, halved);
}
// Up to 128 selected rows: half-size tiles with a pipeline of their own, two workgroups to a compute unit, so that one
// fills its stages while the other multiplies (64 rows of 2048 / 3584 against 151 936: 156 / 215 us against 182 / 274 with
// the large tiles; 128x256 and 256x128 tiles 213 / 347 and 167 / 234).
using NarrowCfg = TileCfg<128, 128, 2, 2>;
constexpr int kNarrowLds = Ring2Cfg<NarrowCfg>::LDS_BYTES;
__global__ void __launch_bounds__(NarrowCfg::T)
k_score_narrow(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, int d, int V,
               const int32_t* __restrict__ rowsel, int64_t n_sel, const int32_t* __restrict__ ids,
               int tiles_m, int tiles_n, int panel, float4* __restrict__ partial, int64_t n_pad) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[kNarrowLds / 2];
  score_tiles<Leave::kNothing, NarrowCfg>(W, H, d, V, rowsel, 0, n_sel, ids, tiles_m, tiles_n, panel, partial, n_pad, KeepArgs{}, lds);
}
__global__ void __launch_bounds__(Cfg::T)
k_score_keep_tiles(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, int d, int V,
                   const int32_t* __restrict__ rowsel, int64_t c0, int64_t mc, const int32_t* __restrict__ ids,
                   int tiles_m, int tiles_n, int panel, int halved, float4* __restrict__ partial, int64_t n_pad,
                   const float* __restrict__ cref, uint16_t* __restrict__ E, int64_t Vp, int32_t* __restrict__ flags,
                   const int32_t* __restrict__ cidx) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[kLogitLds / 2];
  score_tiles<Leave::kNumerators, Cfg>(W, H, d, V, rowsel, c0, mc, ids, tiles_m, tiles_n, panel, partial, n_pad, KeepArgs{cref, E, Vp, flags, cidx, nullptr}, lds, halved);
}
// ... and what an update of so few rows keeps: half rows of half blocks of the operand, whose other rows are never read (100 rows of 3584 270 -> 211
// us; the update, with shorter sums for dW and half the products for dH, 1000 -> 887, of 2048 608 -> 518).
__global__ void __launch_bounds__(NarrowCfg::T)
k_score_keep_narrow(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, int d, int V,
                    const int32_t* __restrict__ rowsel, int64_t n_sel, const int32_t* __restrict__ ids,
                    int tiles_m, float4* __restrict__ partial, int64_t n_pad, const float* __restrict__ cref, uint16_t* __restrict__ E, int64_t Vp,
                    int32_t* __restrict__ flags, const int32_t* __restrict__ cidx) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[kNarrowLds / 2];
  score_tiles<Leave::kNumerators, NarrowCfg>(W, H, d, V, rowsel, 0, n_sel, ids, tiles_m, 1, kGN, partial, n_pad, KeepArgs{cref, E, Vp, flags, cidx, nullptr}, lds);
}
__global__ void __launch_bounds__(Cfg::T)
k_score_logits(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, int d, int V,
               const int32_t* __restrict__ rowsel, int64_t c0, int64_t mc, const int32_t* __restrict__ ids,
               int tiles_m, int tiles_n, int panel, int halved, float4* __restrict__ partial, int64_t n_pad, float* __restrict__ Z, int64_t Vp) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[kLogitLds / 2];
  score_tiles<Leave::kLogits, Cfg>(W, H, d, V, rowsel, c0, mc, ids, tiles_m, tiles_n, panel, partial, n_pad, KeepArgs{nullptr, nullptr, Vp, nullptr, nullptr, Z}, lds, halved);
}

// ------------------------------------------------------------------ bf16: a few rows
// Up to 32 selected rows (64 up to d = 2048): the pass is bound by reading W once, and a 256x256 tile with most of its columns empty spends
// its time filling and draining.  Here the rows of H stay in registers and W streams past them: the eight wavefronts of a
// workgroup split the hidden dimension (each takes PPW pieces of 64, next to each other across the wavefronts, so that a
// row of W is read in whole lines), a wavefront holds its pieces of up to 16 NI rows as MFMA operands for the whole kernel
// and walks a contiguous range of the vocabulary MB blocks of 16 entries at a time, W going straight to registers; a
// piece's registers are loaded again for the next step as soon as they have been used, so that 8 KB and more are in flight
// per wavefront all the time.  The eight partial logits meet in LDS (one barrier a step, two buffers), and every thread
// keeps the softmax statistics of one (row, place in the block of 16) over its workgroup's whole range.  One workgroup per
// compute unit; partials [workgroup][row].
// 24 rows of 2048 (3584) against 151 936: 256x256 tiles 183 (279) us, this kernel 117 (199) us = 5.3 (5.5) TB/s of W; 64
// rows of 2048 182 -> 122 us.
constexpr int kFewWaves = 8, kFewT = kFewWaves * kWave;
inline int few_pieces(int d) { return static_cast<int>(cdiv(d, kFewWaves * 64)); }   // PPW
inline int few_rows(int d) { return few_pieces(d) <= 4 ? 64 : few_pieces(d) <= 8 ? 32 : 0; }   // what the registers hold
template <int NI, int PPW>
__global__ void __launch_bounds__(kFewT)
k_score_few(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, int d, int V, const int32_t* __restrict__ rowsel, int n_sel,
            const int32_t* __restrict__ ids, float4* __restrict__ partial, int n_pad) {
  constexpr int MB = PPW <= 4 && NI <= 2 ? 2 : 1;            // blocks of 16 vocabulary entries per step
  constexpr int NL = (NI + 1) / 2;                           // logits per thread and block
  __shared__ __attribute__((aligned(16))) float s_z[2][kFewWaves][MB][NI][16][16];   // [.][wavefront][block][.][row][entry]
  __shared__ float4 s_part[NI * 16][16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int piece = (lane >> 4) * 8;
  bf16x8 hf[PPW][2][NI];
#pragma unroll
  for (int p = 0; p < PPW; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int n = min(j * 16 + (lane & 15), n_sel - 1), k = (p * kFewWaves + wave) * 64 + q * 32 + piece;
        const int64_t row = rowsel ? rowsel[n] : n;
        const uint4 v = k < d ? *reinterpret_cast<const uint4*>(H + row * d + k) : make_uint4(0u, 0u, 0u, 0u);
        hf[p][q][j] = __builtin_bit_cast(bf16x8, v);
      }
  // this workgroup's blocks of 16 vocabulary entries
  const int blocks = (V + 15) / 16;
  const int per = (blocks + static_cast<int>(gridDim.x) - 1) / static_cast<int>(gridDim.x);
  const int b0 = static_cast<int>(blockIdx.x) * per, b1 = min(b0 + per, blocks);
  uint4 w[MB][PPW][2];
  bool past[2];                                              // the last piece's columns that do not exist
#pragma unroll
  for (int q = 0; q < 2; ++q) past[q] = ((PPW - 1) * kFewWaves + wave) * 64 + q * 32 + piece >= d;
  auto load = [&](int b, int p, int q, int i) {              // past the hidden size: some entry of the row, cleared where it is used
    const int v = min((b + i) * 16 + (lane & 15), V - 1), k = min((p * kFewWaves + wave) * 64 + q * 32 + piece, d - 8);
    w[i][p][q] = *reinterpret_cast<const uint4*>(W + static_cast<int64_t>(v) * d + k);
  };
  if (b0 < b1)
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int p = 0; p < PPW; ++p) { load(b0, p, 0, i); load(b0, p, 1, i); }
  // thread -> (row, place): statistics of the logits of that row at that place of every block
  const bool mine = tid < NI * 256;
  const int my_n = (tid >> 4) & 15, my_v = tid & 15;
  int y[NL];
  float m[NL], s[NL], t[NL], zy[NL];
#pragma unroll
  for (int l = 0; l < NL; ++l) {
    const int n = (2 * l + (tid >> 8)) * 16 + my_n;
    y[l] = mine && n < n_sel ? ids[rowsel ? rowsel[n] : n] : -1;
    // kMasked as in the tiles: against a maximum of -infinity a logit of -infinity makes the sums NaN, and the merge drops
    // a partial whose maximum a NaN logit has left there
    m[l] = kMasked; s[l] = t[l] = zy[l] = 0.f;
  }
  int buf = 0;
  for (int b = b0; b < b1; b += MB, buf ^= 1) {
    floatx4 acc[MB][NI];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int nb = b + MB < b1 ? b + MB : b;                 // past the range: loaded again, not used
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int p = 0; p < PPW; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          // zeros of H alone would not do: their product with a weight that is not finite is NaN
          const bf16x8 a = __builtin_bit_cast(bf16x8, p == PPW - 1 && past[q] ? make_uint4(0u, 0u, 0u, 0u) : w[i][p][q]);
#pragma unroll
          for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, hf[p][q][j], acc[i][j], 0, 0, 0);
          load(nb, p, q, i);
        }
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) *reinterpret_cast<floatx4*>(&s_z[buf][wave][i][j][lane & 15][(lane >> 4) * 4]) = acc[i][j];
    __syncthreads();
    if (mine) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int l = 0; l < NL; ++l) {
          float z = 0.f;
#pragma unroll
          for (int k = 0; k < kFewWaves; ++k) z += s_z[buf][k][i][2 * l + (tid >> 8)][my_n][my_v];
          const int v = (b + i) * 16 + my_v;
          if (v < V && b + i < b1) {
            if (v == y[l]) zy[l] = z;
            const float gap = z - m[l], e = __expf(-fabsf(gap));  // one exponential: of the smaller relative to the larger
            if (gap > 0.f) { s[l] = fmaf(s[l], e, 1.f); t[l] = fmaf(t[l], e, z); m[l] = z; }
            else { s[l] += e; t[l] = fmaf(e, z, t[l]); }
          }
        }
    }
  }
#pragma unroll
  for (int l = 0; l < NL; ++l)
    if (mine) s_part[(2 * l + (tid >> 8)) * 16 + my_n][my_v] = make_float4(m[l], s[l], t[l], zy[l]);
  __syncthreads();
  if (tid < NI * 16) {
    Part p{kNegInf, 0.f, 0.f};
    float z = 0.f;
    for (int k = 0; k < 16; ++k) {
      const float4 q = s_part[tid][k];
      p = part_merge(p, Part{q.x, q.y, q.z});
      z += q.w;
    }
    partial[static_cast<int64_t>(blockIdx.x) * n_pad + tid] = make_float4(p.m, p.s, p.t, z);
  }
}

// Merge the per-tile partials of each selected row; compact results and optional scatter.  Eight lanes of a wavefront
// share a row (lane = 8 * part + row within the group of 8 rows, so a load covers whole 128-byte lines), four loads in
// flight each.  Where there are few rows the four wavefronts of the workgroup share the group's tiles as well (SPLIT):
// 24 rows of 594 tiles 41 -> 7 us, 16 100 rows 53 -> 36; with enough rows to fill the chip the extra merge only costs
// (39 000 rows, 373 MB: 82 us split, 69 not).
constexpr int64_t kFinSplitRows = 20000;
// Row n's parts merged; true in the thread that has the result (SPLIT: one of the first eight of the workgroup).
template <bool SPLIT>
__device__ __forceinline__ bool merge_parts(const float4* __restrict__ partial, int tiles_m, int64_t n_pad, int64_t n, bool live, Part& p, float& zy) {
  __shared__ float4 s_part[4][8];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  constexpr int kParts = SPLIT ? 32 : 8;
  p = Part{kNegInf, 0.f, 0.f};
  zy = 0.f;
  if (live) {
    for (int t0 = SPLIT ? threadIdx.x >> 3 : lane >> 3; t0 < tiles_m; t0 += 4 * kParts) {
      float4 q[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        q[k] = t0 + k * kParts < tiles_m ? partial[static_cast<int64_t>(t0 + k * kParts) * n_pad + n] : make_float4(kNegInf, 0.f, 0.f, 0.f);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        p = part_merge(p, Part{q[k].x, q[k].y, q[k].z});
        zy += q[k].w;
      }
    }
  }
#pragma unroll
  for (int o = 8; o < kWave; o <<= 1) {
    const Part q{__shfl_xor(p.m, o, kWave), __shfl_xor(p.s, o, kWave), __shfl_xor(p.t, o, kWave)};
    p = part_merge(p, q);
    zy += __shfl_xor(zy, o, kWave);
  }
  if constexpr (SPLIT) {
    if (lane < 8) s_part[wave][lane] = make_float4(p.m, p.s, p.t, zy);
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int k = 1; k < 4; ++k) {
        const float4 q = s_part[k][lane & 7];
        p = part_merge(p, Part{q.x, q.y, q.z});
        zy += q.w;
      }
    }
  }
  return lane < 8 && live && (!SPLIT || wave == 0);
}
struct RowScore {
  float logp, lse, entropy;
};
__device__ __forceinline__ RowScore row_score(const Part& p, float zy, bool ok) {
  const float l = p.m + logf(p.s);
  return RowScore{ok ? zy - l : 0.f, l, ok ? l - p.t / p.s : 0.f};
}
template <bool SPLIT>
__global__ void __launch_bounds__(256)
k_score_finalize(const float4* __restrict__ partial, int tiles_m, int64_t n_pad, int64_t n_begin,
                 int64_t n_end, const float* __restrict__ zy_c, const int32_t* __restrict__ rowsel,
                 const int32_t* __restrict__ ids, int V,
                 float* __restrict__ logp_c, float* __restrict__ lse_c, float* __restrict__ ent_c,
                 float* __restrict__ logp, float* __restrict__ lse, float* __restrict__ entropy) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t n = n_begin + (SPLIT ? static_cast<int64_t>(blockIdx.x) : static_cast<int64_t>(blockIdx.x) * 4 + wave) * 8 + (lane & 7);
  Part p;
  float zy;
  if (!merge_parts<SPLIT>(partial, tiles_m, n_pad, n, n < n_end, p, zy)) return;
  if (zy_c) zy = zy_c[n];                                   // taken logits computed beforehand
  const int64_t row = rowsel ? rowsel[n] : n;
  const int y = ids[row];
  const RowScore r = row_score(p, zy, y >= 0 && y < V);
  if (logp_c) { logp_c[n] = r.logp; lse_c[n] = r.lse; ent_c[n] = r.entropy; }
  if (logp) logp[row] = r.logp;
  if (lse) lse[row] = r.lse;
  if (entropy) entropy[row] = r.entropy;
}

// ------------------------------------------------------------------ clipped surrogate
// Per selected row its surrogate, and what the backward needs of it; per block of rows the sums of the statistics for the model and for
// each role.
__global__ void __launch_bounds__(kRowBlock)
k_ppo_rows(Surrogate S, int64_t n_begin, int64_t n_end, const float* __restrict__ logp_c, const float* __restrict__ ent_c,
           float k_ent, int label_apart, const float* __restrict__ lse_c, float* __restrict__ g_c,
           float* __restrict__ a_c, float* __restrict__ kz_c, double* __restrict__ blk_stats) {
  extern __shared__ double s_acc[];   // [wavefronts][(1+n_roles) * kStat]
  const int n_roles = S.n_roles, nacc = (1 + n_roles) * kStat;
  const int lane = threadIdx.x & (kWave - 1);
  double* const w_acc = s_acc + threadIdx.x / kWave * nacc;
  for (int i = lane; i < nacc; i += kWave) w_acc[i] = 0.0;
  __builtin_amdgcn_wave_barrier();
  SurrogateRow R{0.f, 0.f, 0.f, 0.f, 0.f, -1, false};
  const int64_t n = n_begin + static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;   // n_begin is a multiple of the block size
  if (n < n_end) {
    const int64_t row = S.rowsel ? S.rowsel[n] : n;
    const int y = S.ids[row];
    const bool ok = y >= 0 && y < S.V;
    const float lp = ok ? logp_c[n] : 0.f, en = ok ? ent_c[n] : 0.f;
    R = surrogate_row(S, row, ok, lp, en);
    // With label_apart the taken token's column is left out of the dense (bf16) part of dz and g_c carries all of
    // dz[n, y] = g (1 - p_y) + k_ent p_y (log p_y + entropy) in float32: for a confident token g and g p_y nearly
    // cancel, and the rounding of a bf16 g p_y would be as large as what is left.
    g_c[n] = label_apart && ok ? fmaf(R.g, -expm1f(lp), k_ent * __expf(lp) * (lp + en)) : R.g;
    // coefficients of the backward's dense part dz = p (a + kz z): -g from the surrogate, the rest from the
    // entropy bonus k_ent p (log p + entropy); a row with an invalid id has neither
    a_c[n] = ok ? -R.g + k_ent * (en - lse_c[n]) : 0.f;
    kz_c[n] = ok ? k_ent : 0.f;
  }
  const float L = R.L, clipped = R.clipped, en = R.en, kl = R.kl;
  const int role = R.role, valid = R.valid;
  // Sums over the wavefront's rows, the model's and then each role's that occurs among them (usually one or two); the
  // wavefronts' sums are added in a fixed order.  (256 threads adding to six float64 words by atomics took 18 us.)
  const unsigned long long in = __ballot(n < n_end);
  auto sum_into = [&](unsigned long long group, double* acc) {
    const bool mine = (group >> lane) & 1;
    const double sl = wave_sum(mine ? static_cast<double>(L) : 0.0), se = wave_sum(mine ? static_cast<double>(en) : 0.0);
    const double sk = wave_sum(mine ? static_cast<double>(kl) : 0.0);
    const int c = __popcll(__ballot(mine && clipped != 0.f)), bad = __popcll(__ballot(mine && !valid));
    if (lane == 0) { acc[0] = sl; acc[1] = c; acc[2] = se; acc[3] = sk; acc[4] = __popcll(group); acc[5] = bad; }
  };
  sum_into(in, w_acc);
  unsigned long long left = in & __ballot(role >= 0 && role < n_roles);
  while (left) {                                              // the same for every lane
    const int r = __shfl(role, __ffsll(static_cast<long long>(left)) - 1, kWave);
    const unsigned long long group = left & __ballot(role == r);
    sum_into(group, w_acc + (1 + r) * kStat);
    left &= ~group;
  }
  __syncthreads();
  const int64_t blk = n_begin / kRowBlock + blockIdx.x;
  for (int i = threadIdx.x; i < nacc; i += blockDim.x) {
    double v = 0.0;
    for (int w = 0; w < kRowBlock / kWave; ++w) v += s_acc[w * nacc + i];
    blk_stats[blk * nacc + i] = v;
  }
}

// The record of the model (k = 0) or of a role, a workgroup to each.
__device__ __forceinline__ void
ppo_stats(int k, int nblk, int n_roles, float entropy_coef, int64_t norm_rows, const double* __restrict__ blk_stats,
            umas_loss_stats* __restrict__ stats) {
  __shared__ double smem[32];
  const int nacc = (1 + n_roles) * kStat;
  double v[kStat] = {}, sum[kStat];
  for (int b = threadIdx.x; b < nblk; b += blockDim.x)
#pragma unroll
    for (int j = 0; j < kStat; ++j) v[j] += blk_stats[static_cast<int64_t>(b) * nacc + k * kStat + j];
#pragma unroll
  for (int j = 0; j < kStat; ++j) sum[j] = block_sum<double>(v[j], smem);
  if (threadIdx.x != 0) return;
  stats[k] = loss_stats(sum, k, entropy_coef, norm_rows);
}

// The same from the rows, where they are few and k_rows_few has left no sums.
__device__ __forceinline__ void ppo_stats_by_row(int k, const Surrogate& S, int64_t n_sel, float entropy_coef, int64_t norm_rows, const float* __restrict__ logp_c,
                                                 const float* __restrict__ ent_c, umas_loss_stats* __restrict__ stats) {
  __shared__ double smem[32];
  double v[kStat] = {}, sum[kStat];
  for (int64_t n = threadIdx.x; n < n_sel; n += blockDim.x) {
    const int64_t row = S.rowsel ? S.rowsel[n] : n;
    const int y = S.ids[row];
    const SurrogateRow R = surrogate_row(S, row, y >= 0 && y < S.V, logp_c[n], ent_c[n]);
    if (k > 0 && R.role != k - 1) continue;
    v[0] += static_cast<double>(R.L);
    v[1] += R.clipped != 0.f ? 1.0 : 0.0;
    v[2] += static_cast<double>(R.en);
    v[3] += static_cast<double>(R.kl);
    v[4] += 1.0;
    v[5] += R.valid ? 0.0 : 1.0;
  }
#pragma unroll
  for (int j = 0; j < kStat; ++j) sum[j] = block_sum<double>(v[j], smem);
  if (threadIdx.x != 0) return;
  stats[k] = loss_stats(sum, k, entropy_coef, norm_rows);
}

// ------------------------------------------------------------------ bf16: blocks of rows that have a gradient
// A selected row whose advantage is 0 has g = 0 and (without an entropy bonus or a KL term) no gradient at all; group-normalised
// outcome rewards make whole trajectory groups such rows.  The keeping pass therefore works on the chunk's live blocks
// of 256 selected rows only: E and the scaled copy of H hold them packed, dH has as many row tiles and dW as many K
// steps as there are, and everything that depends on their number is worked out on the device.
struct LiveInfo {
  int32_t n_live;        // live blocks of the chunk
  int32_t k_rows;        // rows of the packed operands that exist (the chunk's last block may be partly filled)
  XcdShares dw;          // dW tiles per XCD (see share_dw)
  int32_t next[8];       // per XCD: next place of its sequence of tiles, counted up by the workgroups of k_gemm_dh_dw
};
// Shares of the dW tiles per XCD for k_gemm_dh_dw: every XCD first works through its eighth of the dH tiles (contiguous
// ranges, slice after slice; a tile costs about Vp / slices of K), then dW tiles (k_len of K each) go to the XCDs so that all
// finish as evenly as possible.  Shares are whole groups where there are many: an XCD's workgroups that work on parts of two
// groups at a time read a third more through its L2 (39 000 rows of 2048: 6 % of the step).
constexpr int64_t kTileOverheadK = 768;   // what a tile costs besides its K steps (first loads, epilogue), as a length of K
__device__ __forceinline__ int share_unit(int tiles, int slices) { return slices == 1 && tiles >= 8 * kGM * kGN ? kGM * kGN : 1; }
__device__ __forceinline__ int dh_first(int tiles_dh, int slices, int xcd) {
  const int unit = share_unit(tiles_dh, slices), units = (tiles_dh + unit - 1) / unit;
  return min(static_cast<int>(static_cast<int64_t>(units) * xcd / 8) * unit, tiles_dh);
}
// K of the dW tiles: whole steps of 64 rows.  (With whole blocks of 256, and dH tiles that read and
// multiply the rows that are not there as well: both products of 30 / 100 rows of 3584 672 us, now 612 / 620; update of 300 / 550 rows of 2048 976 / 1327,
// now 890 / 1252.)
__device__ __forceinline__ int dw_k(int k_rows) { return (k_rows + 63) / 64 * 64; }
// Called by one wavefront; lane x of every eight works for XCD x (all eights do the same).  (One thread walking the eight XCDs took 20 us.)
__device__ void share_dw(int tiles_r, int tiles_v, int tiles_d, int64_t Vp, int slices, int64_t k_len, XcdShares* out) {
  const int x = threadIdx.x & 7;
  auto sum8 = [](int64_t v) {
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) v += static_cast<int64_t>(__shfl_xor(static_cast<long long>(v), o, kWave));
    return v;
  };
  const int tiles_dh = tiles_r * tiles_d * slices;
  const int64_t load = (dh_first(tiles_dh, slices, x + 1) - dh_first(tiles_dh, slices, x)) * (Vp / slices + kTileOverheadK);
  const int tiles_dw = tiles_v * tiles_d, unit = share_unit(tiles_dw, 1);
  const int64_t units = (tiles_dw + unit - 1) / unit;
  k_len *= unit;
  int64_t cnt;
  if (k_len <= 0 || units == 0) {                      // nothing to even out
    cnt = units / 8 + (x < units % 8 ? 1 : 0);
  } else {
    // the level up to which the XCDs would be filled if units could be cut: those that stand above it as they are take nothing ...
    // (a search for it among whole numbers took 23 rounds: k_live_scan 9.6 us, now 5.1)
    double level = 0.0;
    bool takes = true;
    for (int round = 0; round < 8; ++round) {
      level = static_cast<double>(units * k_len + sum8(takes ? load : 0)) / static_cast<double>(sum8(takes ? 1 : 0));
      const bool above = takes && static_cast<double>(load) >= level;
      if (!__any(above)) break;
      takes = takes && !above;
    }
    cnt = takes ? static_cast<int64_t>((level - static_cast<double>(load)) / static_cast<double>(k_len)) : 0;
    // ... and of the few units that are left every one goes where it is done first (or comes, by rounding, from where it would be last)
    for (int64_t left = units - sum8(cnt); left != 0; left -= left > 0 ? 1 : -1) {
      const int64_t end = left > 0 ? -(load + cnt * k_len) : cnt > 0 ? load + cnt * k_len : INT64_MIN;
      int64_t best = end;
#pragma unroll
      for (int o = 4; o > 0; o >>= 1) best = max(best, static_cast<int64_t>(__shfl_xor(static_cast<long long>(best), o, kWave)));
      if (x == __ffsll(static_cast<long long>(__ballot(end == best))) - 1) cnt += left > 0 ? 1 : -1;
    }
  }
  int first = static_cast<int>(cnt);                   // inclusive prefix sums: where the next XCD's units start
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) {
    const int t = __shfl_up(first, o, kWave);
    if (x >= o) first += t;
  }
  if (threadIdx.x == 0) out->first[0] = 0;
  if (threadIdx.x < 8) out->first[x + 1] = static_cast<int>(min(static_cast<int64_t>(first) * unit, static_cast<int64_t>(tiles_dw)));
}
// Packs the live blocks of a chunk, blk0 its first block; one workgroup, thread t has block t and knows if it is live.
struct LiveArgs {
  int blk0, nblk;
  int64_t rows;
  int all_live, tiles_v, tiles_d;
  int64_t Vp;
  int slices;
  const int32_t* blk_live;
  int32_t *blk_cidx, *blk_orig;
  LiveInfo* info;
};
__device__ __forceinline__ void live_scan(const LiveArgs& A, int live) {
  __shared__ int smem[32];
  __shared__ int s_last_live;
  const int t = threadIdx.x;
  int total;
  const int pos = block_excl_scan<int>(live, smem, &total);
  if (t < A.nblk) {
    A.blk_cidx[A.blk0 + t] = live ? pos : -1;
    if (live) A.blk_orig[A.blk0 + pos] = t;
  }
  if (t == A.nblk - 1) s_last_live = live;
  __syncthreads();
  const int64_t last_rows = A.rows - static_cast<int64_t>(A.nblk - 1) * 256;   // rows of the chunk's last block
  const int k_rows = static_cast<int>(s_last_live ? static_cast<int64_t>(total - 1) * 256 + last_rows : static_cast<int64_t>(total) * 256);
  if (t == 0) {
    A.info->n_live = total;
    A.info->k_rows = k_rows;
  }
  if (t < 8) A.info->next[t] = 0;
  if (t < kWave) share_dw(total, A.tiles_v, A.tiles_d, A.Vp, A.slices, total > 0 ? dw_k(k_rows) + kTileOverheadK : 0, &A.info->dw);
}
// One launch per chunk (all blocks live with all_live).
__global__ void __launch_bounds__(512)
k_live_scan(LiveArgs A) {
  const int t = threadIdx.x;
  live_scan(A, t < A.nblk && (A.all_live || A.blk_live[A.blk0 + t]));
}

// What opens the keeping update, in one launch: the first nblk workgroups mark the live blocks of 256 selected rows and
// clear their flags, the others take the rows' references and clear what the call defines everywhere (logp_new when rows
// are left out, dH), each its share.  Up to kFewBlocks blocks in one chunk the first workgroup alone marks them and packs them as well, under the
// others' work (203 rows of 3584 1025 -> 1018 us, 2000 of 2048 3137 -> 3099).
constexpr int kFewBlocks = 8;
struct OpenArgs {
  const uint16_t* H;
  const uint16_t* W;
  int d, V;
  const int32_t* rowsel;
  int64_t n_sel;
  const int32_t* ids;
  const float* adv;
  int nblk;
  int32_t* blk_live;
  int32_t* flags;
  float* cref;
  uint32_t* dH;          // n_rows * d bf16 as words
  int64_t dh_words;
  float* logp_new;       // NULL: nothing to clear
  int64_t n_rows;
  int pack;              // few blocks: nblk is 1, the blocks are live.nblk
  LiveArgs live;
};
// ------------------------------------------------------------------ bf16: row references and row factors of the keeping pass
__device__ __forceinline__ void bf16x8_to_f32(const uint4 v, float (&o)[8]) {
  o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xffff0000u);
  o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xffff0000u);
  o[4] = __uint_as_float(v.z << 16); o[5] = __uint_as_float(v.z & 0xffff0000u);
  o[6] = __uint_as_float(v.w << 16); o[7] = __uint_as_float(v.w & 0xffff0000u);
}
__global__ void __launch_bounds__(256)
k_update_open(OpenArgs A) {
  if (A.pack && blockIdx.x == 0) {
    float adv[kFewBlocks];
#pragma unroll
    for (int b = 0; b < kFewBlocks; ++b) {
      const int64_t n = b * 256 + threadIdx.x;
      adv[b] = n < A.n_sel ? A.adv[A.rowsel ? A.rowsel[n] : n] : 0.f;
    }
    int live = 0;
#pragma unroll
    for (int b = 0; b < kFewBlocks; ++b) {
      const int any = __syncthreads_or(adv[b] != 0.f);
      if (static_cast<int>(threadIdx.x) == b && b < A.live.nblk) {
        live = any || A.live.all_live;
        A.flags[b] = 0;
      }
    }
    live_scan(A.live, live);
    return;
  }
  if (static_cast<int>(blockIdx.x) < A.nblk) {
    const int64_t n = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int live = n < A.n_sel && A.adv[A.rowsel ? A.rowsel[n] : n] != 0.f;
    const int any = __syncthreads_or(live);
    if (threadIdx.x == 0) {
      A.blk_live[blockIdx.x] = any;
      A.flags[blockIdx.x] = 0;
    }
    return;
  }
  const int64_t blk = static_cast<int64_t>(blockIdx.x) - A.nblk, nb = static_cast<int64_t>(gridDim.x) - A.nblk;
  {
    const int64_t n4 = A.dh_words / 4, stride = nb * 256;
    uint4* const p = reinterpret_cast<uint4*>(A.dH);
    if (reinterpret_cast<uintptr_t>(p) % 16 == 0) {
      for (int64_t i = blk * 256 + threadIdx.x; i < n4; i += stride) p[i] = make_uint4(0u, 0u, 0u, 0u);
      for (int64_t i = 4 * n4 + blk * 256 + threadIdx.x; i < A.dh_words; i += stride) A.dH[i] = 0u;
    } else {
      for (int64_t i = blk * 256 + threadIdx.x; i < A.dh_words; i += stride) A.dH[i] = 0u;
    }
    if (A.logp_new)
      for (int64_t i = blk * 256 + threadIdx.x; i < A.n_rows; i += stride) A.logp_new[i] = 0.f;
  }
  // cref[n] = h_n . W[y_n], the taken token's logit (never above the row's logsumexp); NaN for an invalid id.
  // One wavefront per selected row.
  const int lane = threadIdx.x & 63;
  for (int64_t n = blk * 4 + threadIdx.x / kWave; n < A.n_sel; n += nb * 4) {
    const int64_t row = A.rowsel ? A.rowsel[n] : n;
    const int y = A.ids[row];
    if (y < 0 || y >= A.V) {
      if (lane == 0) A.cref[n] = NAN;
      continue;
    }
    const uint4* h = reinterpret_cast<const uint4*>(A.H + row * A.d);
    const uint4* w = reinterpret_cast<const uint4*>(A.W + static_cast<int64_t>(y) * A.d);
    float s = 0.f;
    for (int k = lane; k < A.d / 8; k += kWave) {
      float a[8], b[8];
      bf16x8_to_f32(h[k], a);
      bf16x8_to_f32(w[k], b);
#pragma unroll
      for (int j = 0; j < 8; ++j) s = fmaf(a[j], b[j], s);
    }
    s = wave_sum(s);
    if (lane == 0) A.cref[n] = s;
  }
}
// Row factor sc[n] = a_n exp(c_n - lse_n) of dz = sc E, and Hs[n - c0, :] = bf16(sc[n] h_n), the operand dW reads, in
// column blocks [d / 256][mcp][256].
// Rows of a flagged block get factor 1: their dz comes complete from the recomputing kernel.  The entry of the
// taken token is cleared in the [rows, V] operand (see k_ppo_rows).
struct KeptRows {
  const uint16_t* H;
  int d, V;
  uint16_t* E;
  int64_t tiles_v;
  const float* cref;
  const int32_t* flags;
  const int32_t* cidx;
  float* sc;
  uint16_t* Hs;
  int64_t mcp;
};
// blk: place of the row's block among the live ones
__device__ __forceinline__ float kept_factor(int blk, int flag, float cref, float a, float lse) {
  if (blk < 0) return 0.f;                                   // a dead block: no row of it has a gradient
  if (flag) return 1.f;
  return a != 0.f ? a * __expf(cref - lse) : 0.f;            // a = 0: invalid id (reference NaN) or no gradient
}
// one wavefront; m: the row's place in the chunk, n: in the selection
__device__ __forceinline__ void kept_row(const KeptRows& K, int64_t m, int64_t n, int blk, int64_t row, int y, float f) {
  const int lane = threadIdx.x & 63;
  if (lane == 0) K.sc[n] = f;
  if (blk < 0) return;
  const int64_t mp = static_cast<int64_t>(blk) * 256 + (m & 255);   // row in the packed operands
  if (lane == 0 && y >= 0 && y < K.V)                        // the taken token's column goes through g_c in float32
    K.E[blk_offset(blk, y >> 8, K.tiles_v) + (m & 255) * 256 + (y & 255)] = 0;
  const uint4* h = reinterpret_cast<const uint4*>(K.H + row * K.d);
  for (int k = lane; k < K.d / 8; k += kWave) {
    uint4* o = reinterpret_cast<uint4*>(K.Hs + (static_cast<int64_t>(k >> 5) * K.mcp + mp) * 256);   // column block k / 32 of the row
    float x[8];
    bf16x8_to_f32(h[k], x);
    uint4 v;
    v.x = pack_bf16x2(x[0] * f, x[1] * f);
    v.y = pack_bf16x2(x[2] * f, x[3] * f);
    v.z = pack_bf16x2(x[4] * f, x[5] * f);
    v.w = pack_bf16x2(x[6] * f, x[7] * f);
    o[k & 31] = v;
  }
}
__global__ void __launch_bounds__(256)
k_keep_rows(KeptRows K, const int32_t* __restrict__ rowsel, int64_t c0, int64_t rows, const int32_t* __restrict__ ids, const float* __restrict__ lse_c,
            const float* __restrict__ a_c) {
  const int64_t m = static_cast<int64_t>(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave;
  if (m >= rows) return;
  const int64_t n = c0 + m, row = rowsel ? rowsel[n] : n;
  // what the row needs is asked for together (place, flag and reference one after the other: 3738 rows of 2048 11.9 us, like this 11.55)
  const int blk = K.cidx[n >> 8], flag = K.flags[n >> 8];
  const float a = a_c[n], lse = lse_c[n], cref = K.cref[n];
  kept_row(K, m, n, blk, row, ids[row], kept_factor(blk, flag, cref, a, lse));
}
// Few rows (one chunk of up to kFewBlocks blocks): k_score_finalize, k_ppo_rows and k_keep_rows in one launch, eight rows to a workgroup; the statistics are left
// to k_update_close, which goes over the rows once more.  Bound by its chain of loads, as the three were: update of 203 rows of 1096 against 50 001 191.6 and
// 184.5 us, 60 rows of 1024 against 151 936 271 and 266, 500 of 512 against 30 001 138.9 and 126.7, 2000 270.3 and 262.2, 2000 of 2048 against 151 936
// 3218 and 3194, of 3584 against 50 001 1875 and 1868.
struct RowsArgs {
  const float4* partial;
  int tiles_m;
  int64_t n_pad, n_sel;
  Surrogate S;
  float *logp_c, *lse_c, *ent_c, *logp_new, *g_c, *a_c, *kz_c;
  KeptRows K;
};
__global__ void __launch_bounds__(256)
k_rows_few(RowsArgs A) {
  __shared__ float s_f[8];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t n0 = static_cast<int64_t>(blockIdx.x) * 8, n = n0 + (lane & 7);
  Part p;
  float zy;
  if (merge_parts<true>(A.partial, A.tiles_m, A.n_pad, n, n < A.n_sel, p, zy)) {
    const int64_t row = A.S.rowsel ? A.S.rowsel[n] : n;
    const int y = A.S.ids[row];
    const bool ok = y >= 0 && y < A.S.V;
    const float cref = A.K.cref[n];
    const RowScore r = row_score(p, cref, ok);
    const SurrogateRow R = surrogate_row(A.S, row, ok, r.logp, r.entropy);
    const float a = ok ? -R.g : 0.f;
    A.logp_c[n] = r.logp;
    A.lse_c[n] = r.lse;
    A.ent_c[n] = r.entropy;
    if (A.logp_new) A.logp_new[row] = r.logp;
    A.g_c[n] = ok ? R.g * -expm1f(r.logp) : R.g;             // all of dz[n, y] (see k_ppo_rows)
    A.a_c[n] = a;                                            // for the blocks that are computed once more
    A.kz_c[n] = 0.f;
    s_f[lane] = kept_factor(A.K.cidx[n >> 8], A.K.flags[n >> 8], cref, a, r.lse);
  }
  __syncthreads();
#pragma unroll
  for (int k = wave; k < 8; k += 4) {
    if (n0 + k >= A.n_sel) continue;
    const int64_t row = A.S.rowsel ? A.S.rowsel[n0 + k] : n0 + k;
    kept_row(A.K, n0 + k, n0 + k, A.K.cidx[(n0 + k) >> 8], row, A.S.ids[row], s_f[k]);
  }
}

// ------------------------------------------------------------------ bf16: dz tiles into the chunk buffer
// For blocks of rows whose numerators do not serve, and with an entropy bonus for narrow heads and in a small workspace (16 100 rows of 2048 in 2 GB,
// chunks of 3300: 31.3 ms; chunks of logits of half that many rows would add to dW twice as often).  Same tile product as k_score_tiles; the epilogue forms the dense part of dz = g (onehot - softmax),
// -g exp(z - lse), plus the entropy bonus's term when its coefficient is not 0, and writes it as bf16 to
// dZ [mcp, Vp].  Rows past the chunk and vocabulary ids past V get 0.  The one-hot part g at v = y is a single term per row and is added in
// float32 where dH and dW are written, so that it never meets the bf16 rounding of the dense part.
// CLEAR: the taken token's entry of every row is left at 0 (see k_ppo_rows); the others leave that to who goes over the rows afterwards.
template <bool CLEAR>
__device__ __forceinline__ void dz_tile(int tile_m, int tile_n, const uint16_t* __restrict__ W, const uint16_t* __restrict__ H,
                                        int d, int V, const int32_t* __restrict__ rowsel, int64_t c0, int64_t mc, const int32_t* __restrict__ ids,
                                        const float* __restrict__ lse_c, const float* __restrict__ a_c,
                                        const float* __restrict__ kz_c, uint16_t* __restrict__ dZ, int64_t Vp, int out_blk,
                                        uint16_t* lds) {
  using C = Cfg;
  const int m0 = tile_m * C::BM;
  const int64_t n0 = static_cast<int64_t>(tile_n) * C::BN;   // chunk-relative
  floatx4 acc[C::MI][C::NI];
  logit_tile<C>(W, H, d, V, rowsel, c0, mc, m0, n0, false, lds, acc);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / C::WN;
  const int vbase = m0 + wm * C::WTM + (lane >> 4) * 4;
  const bool tail = m0 + C::BM > V;
  // each wavefront stages its 64 (rows) x 128 (vocabulary) block; the 272-byte pitch keeps 16-byte alignment
  char* stage = reinterpret_cast<char*>(lds) + wave * (C::WTN * kStagePitch);
  __syncthreads();                              // every wavefront has left the main loop's LDS reads
  if (tail) {                                   // vocabulary ids past V: the exponential below is 0, the factor next to it finite
#pragma unroll
    for (int i = 0; i < C::MI; ++i)
#pragma unroll
      for (int j = 0; j < C::NI; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (vbase + i * 16 + r >= V) acc[i][j][r] = kMasked;
  }
#pragma unroll
  for (int j = 0; j < C::NI; ++j) {
    const int64_t n = n0 + acc_col<C>(j);
    // dz = p (a + kz z) with p = exp(z - lse), a = -g + k (entropy - lse), kz = k = entropy_coef / n_sel: the
    // dense part of g (onehot - p) plus the entropy bonus's k p (log p + entropy).  Rows past the chunk: p = 0.
    float l2 = 1e30f, a = 0.f, kz = 0.f;
    if (n < mc) {
      l2 = lse_c[c0 + n] * 1.44269504088896341f;
      a = a_c[c0 + n];
      kz = kz_c[c0 + n];
    }
#pragma unroll
    for (int i = 0; i < C::MI; ++i) {
      float dz[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float z = acc[i][j][r];
        dz[r] = __builtin_amdgcn_exp2f(fmaf(z, 1.44269504088896341f, -l2)) * fmaf(kz, z, a);
      }
      const uint32_t p01 = pack_bf16x2(dz[0], dz[1]), p23 = pack_bf16x2(dz[2], dz[3]);
      // staged in this wavefront's LDS region, stored in full lines below
      *reinterpret_cast<uint2*>(stage + (j * 16 + (lane & 15)) * kStagePitch + (i * 16 + (lane >> 4) * 4) * 2) =
          make_uint2(p01, p23);
    }
  }
  const int wn = wave % C::WN;
  if constexpr (CLEAR) {                        // a lane per staged row (every entry compared above: 60 bytes of scratch a lane, like this 20; with no block flagged 6.9 us and 6.55)
    static_assert(C::WTN == kWave, "a row a lane");
    __builtin_amdgcn_wave_barrier();
    const int64_t n = n0 + wn * C::WTN + lane;
    const int y = (n < mc ? ids[rowsel ? rowsel[c0 + n] : c0 + n] : -1) - (m0 + wm * C::WTM);
    const uint16_t none = 0;
    if (y >= 0 && y < C::WTM) __builtin_memcpy(stage + lane * kStagePitch + y * 2, &none, 2);
    __builtin_amdgcn_wave_barrier();
  }
  // the staged block goes out 16 bytes per lane: one instruction covers 4 rows x 256 contiguous bytes
  uint16_t* out = dZ + blk_offset(out_blk, tile_m, Vp >> 8) + (wn * C::WTN) * 256 + wm * C::WTM + (lane & 15) * 8;
#pragma unroll 8
  for (int i = 0; i < C::WTN / 4; ++i) {
    const int row = i * 4 + (lane >> 4);
    const uint4 v = *reinterpret_cast<const uint4*>(stage + row * kStagePitch + (lane & 15) * 16);
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4*>(out + row * 256));
  }
  __syncthreads();                              // the LDS is the next tile's again
}
__global__ void __launch_bounds__(Cfg::T)
k_dz_tiles(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, int d, int V,
           const int32_t* __restrict__ rowsel, int64_t c0, int64_t mc,
           const float* __restrict__ lse_c, const float* __restrict__ a_c, const float* __restrict__ kz_c,
           int tiles_m, int tiles_n, int panel, uint16_t* __restrict__ dZ, int64_t Vp) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[kLogitLds / 2];
  for (int it = 0; it < kTilesPerWg; ++it) {     // a workgroup walks the same place of kTilesPerWg consecutive tile groups
    int tile_m, tile_n;
    if (!tile_coords<kGM, kGN>(tiles_m, tiles_n, panel, &tile_m, &tile_n, it, kTilesPerWg)) continue;
    dz_tile<false>(tile_m, tile_n, W, H, d, V, rowsel, c0, mc, nullptr, lse_c, a_c, kz_c, dZ, Vp, tile_n, lds);
  }
}
// The same tiles for the blocks of 256 rows that the keeping scoring pass has flagged, and only those: a fixed,
// small grid walks (flagged block, vocabulary tile) pairs, so that the usual case of no flag costs next to nothing.
constexpr int kFlaggedGrid = 256;
__global__ void __launch_bounds__(Cfg::T)
k_dz_flagged(const uint16_t* __restrict__ W, const uint16_t* __restrict__ H, int d, int V,
             const int32_t* __restrict__ rowsel, int64_t c0, int64_t mc, const int32_t* __restrict__ ids,
             const float* __restrict__ lse_c, const float* __restrict__ a_c, const float* __restrict__ kz_c,
             int tiles_m, int tiles_n, uint16_t* __restrict__ dZ, int64_t Vp, const int32_t* __restrict__ flags,
             const int32_t* __restrict__ cidx) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[kLogitLds / 2];
  for (int tile_n = 0; tile_n < tiles_n; ++tile_n) {
    const int out_blk = cidx[(c0 >> 8) + tile_n];
    if (!flags[(c0 >> 8) + tile_n] || out_blk < 0) continue;        // the same for every thread of the grid
    for (int tile_m = blockIdx.x; tile_m < tiles_m; tile_m += gridDim.x)
      dz_tile<true>(tile_m, tile_n, W, H, d, V, rowsel, c0, mc, ids, lse_c, a_c, kz_c, dZ, Vp, out_blk, lds);
  }
}

// dz from the logits that k_score_logits has left, in place: a block of 256 x 256 floats becomes bf16 in its first half (so
// the operand's blocks lie two block lengths apart).  A workgroup turns one block, 32 rows at a time, a row to a wavefront's
// load; a group of rows is written once all wavefronts have what lies there and in front of it in registers, and the
// next one is on its way meanwhile.  Bound by the 6 bytes a logit that are read and written: 16 100 rows against 151 936 in 2.75
// ms (5.3 TB/s).  With the logits stored (1.05 ms more for the scoring pass) instead of computed twice, and so these two in place
// of 7.6 ms of k_dz_tiles, that update takes 27.0 ms in two chunks instead of 30.2; 203 rows of 3584 1.21 instead of 1.43.
constexpr int kTurnRows = 32, kTurnWaves = 4, kRowsPerWave = kTurnRows / kTurnWaves;
__global__ void __launch_bounds__(kTurnWaves * kWave)
k_dz_from_logits(float* Z, int tiles_v, int64_t c0, int64_t mc, const float* __restrict__ lse_c, const float* __restrict__ a_c,
                 const float* __restrict__ kz_c) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t n0 = static_cast<int64_t>(blockIdx.x / tiles_v) * 256;     // chunk-relative
  float* const blk = Z + static_cast<int64_t>(blockIdx.x) * kBlkElems;
  uint16_t* const out = reinterpret_cast<uint16_t*>(blk);
  floatx4 z[2][kRowsPerWave];
  auto fetch = [&](int g, floatx4 (&x)[kRowsPerWave]) {
#pragma unroll
    for (int r = 0; r < kRowsPerWave; ++r) {
      const int row = g * kTurnRows + wave * kRowsPerWave + r;
      x[r] = floatx4{0.f, 0.f, 0.f, 0.f};
      if (n0 + row < mc) x[r] = __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(blk + row * 256 + lane * 4));
    }
  };
  fetch(0, z[0]);
#pragma unroll
  for (int g = 0; g < 256 / kTurnRows; ++g) {
    // this group has arrived: its registers are taken as used here, or the loads could sink below the barrier and meet what
    // another wavefront has written there
#pragma unroll
    for (int r = 0; r < kRowsPerWave; ++r) asm volatile("" : "+v"(z[g & 1][r]) : : "memory");
    __syncthreads();
    if (g + 1 < 256 / kTurnRows) fetch(g + 1, z[(g + 1) & 1]);
#pragma unroll
    for (int r = 0; r < kRowsPerWave; ++r) {
      const int row = g * kTurnRows + wave * kRowsPerWave + r;
      float l2 = 1e30f, a = 0.f, kz = 0.f;                                 // rows past the chunk: 0
      if (n0 + row < mc) {
        l2 = lse_c[c0 + n0 + row] * 1.44269504088896341f;
        a = a_c[c0 + n0 + row];
        kz = kz_c[c0 + n0 + row];
      }
      float dz[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float x = z[g & 1][r][k];
        dz[k] = __builtin_amdgcn_exp2f(fmaf(x, 1.44269504088896341f, -l2)) * fmaf(kz, x, a);
      }
      *reinterpret_cast<uint2*>(out + row * 256 + lane * 4) = make_uint2(pack_bf16x2(dz[0], dz[1]), pack_bf16x2(dz[2], dz[3]));
    }
  }
}

// What the gradient products need besides dZ: the taken token's entry of every row is cleared (that column goes through
// g_c in float32, see k_ppo_rows), and the row of H goes to the operand that dW reads, in the column blocks of k_keep_rows.
// One wavefront per row.  (dW reading the rows through the selection: two kinds of loads in flight, whose waits have to be
// for all of them, 16 100 rows of 2048: both products 16.3 ms, with the copy, 25 us, 14.9.)
__global__ void __launch_bounds__(256)
k_dz_rows(const uint16_t* __restrict__ H, int d, int V, const int32_t* __restrict__ rowsel, int64_t c0, int64_t rows,
          const int32_t* __restrict__ ids, uint16_t* __restrict__ dZ, int64_t tiles_v, int blk_pitch, uint16_t* __restrict__ Hs, int64_t mcp) {
  const int lane = threadIdx.x & 63;
  const int64_t m = static_cast<int64_t>(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave;
  if (m >= rows) return;
  const int64_t row = rowsel ? rowsel[c0 + m] : c0 + m;
  const int y = ids[row];
  if (lane == 0 && y >= 0 && y < V) dZ[blk_offset(m >> 8, y >> 8, tiles_v) * blk_pitch + (m & 255) * 256 + (y & 255)] = 0;
  const uint4* h = reinterpret_cast<const uint4*>(H + row * d);
  for (int k = lane; k < d / 8; k += kWave) reinterpret_cast<uint4*>(Hs + (static_cast<int64_t>(k >> 5) * mcp + m) * 256)[k & 31] = h[k];
}

// ------------------------------------------------------------------ bf16: the two gradient products
// dH = dZ W: A = dZ [mcp, Vp] (or the kept numerators E) is K-contiguous (K = vocabulary), B = W [V, d] is K-major and is read as it lies.
//   dH[rowsel[c0 + m], j] = bf16(sc[m] C[m, j] + g[m] W[y[m], j]) for m < mc (sc: the keeping pass's row factor, else 1)
// dW = dZ^T H: K = rows of the chunk; A = dZ [mcp, Vp] and B = the selected rows of H, copied (and scaled), are both K-major.
//   dW[v, j] (+)= C[v, j]
// (kernel templates whose bodies use buffer resources do not get their host stubs emitted: plain kernels)
template <class C>
__device__ __forceinline__ void zero_acc(floatx4 (&acc)[C::MI][C::NI]) {
#pragma unroll
  for (int i = 0; i < C::MI; ++i)
#pragma unroll
    for (int j = 0; j < C::NI; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
}
// K-contiguous operand tile: block row `row_blk` of the blocked [rows, vocabulary] operand from vocabulary block `voc_blk` on, of which the
// first `rows` rows are wanted: a pass of loads behind them takes the lines of the first one again, which are on their way to this
// compute unit anyhow (the last row for all of them made one line hot: 203 rows of 2048 613 -> 650 us); K runs over the vocabulary, four steps of 64 per block
template <class C>
__device__ __forceinline__ KContig blocked_rows_tile(const uint16_t* X, int blk_pitch, int64_t tiles_v, int64_t row_blk, int voc_blk, int rows) {
  KContig c;
  c.rsrc = make_rsrc(X + blk_offset(row_blk, voc_blk, tiles_v) * blk_pitch);
  c.hi_bytes = static_cast<uint32_t>(kBlkElems * 2 * blk_pitch - 4 * 128);        // from the fourth step of a block to the next block
  const int tid = tile_thread();
  const uint32_t kofs = ring2_kofs(tid);
#pragma unroll
  for (int i = 0; i < 4; ++i) c.off[i] = (static_cast<uint32_t>(ring2_row<C>(ring2_row<C>(i, 0) < rows ? i : 0, tid)) * 256u + kofs) * 2u;
  return c;
}

// A tile's accumulators go out as float32 rows, `ld` floats apart from `out` on (or are added to what is there); rows and cols
// of them exist, cols a multiple of 4.  A 16x16 block's registers cover 64 bytes of four rows each; stored like that, half a
// line at a time, they kept the dW tiles of short selections waiting (725 rows of 2048 against 151 936: both products 2.1
// ms, through LDS 1.3 ms).  Every wavefront turns its 128 x 64 block through its own part of LDS, 32 rows at a time, and
// stores 256 bytes of four rows.  In a tile that exists as a whole nothing depends on the row: what is there already is
// under way during the turn, and a piece's LDS reads and stores go out together (waiting for each of 32 pieces by itself:
// both products of 725 rows of 2048 that add to dW 1155 us, together 1020; 64 rows without adding 459 and 443).  With `past` what is there is read
// past the caches, which leaves them to the operands (see past_caches).  Such a piece is addressed by 32-bit offsets from the wavefront's first row; rows farther apart than
// kPieceLd take the way of the tiles that end early, with 64-bit addresses.
constexpr int kTurnBytes = 32 * 64 * 4;                              // 32 rows of 64 floats per wavefront
constexpr int64_t kPieceLd = int64_t{1} << 22;                       // floats
static_assert(((Cfg::WTM - 1) * kPieceLd + Cfg::WTN) * 4 < int64_t{1} << 31, "the last row of a wavefront's block is in reach");
static_assert(Cfg::WTN == 64 && Cfg::WM * Cfg::WN == 8 && 8 * kTurnBytes <= 2 * Cfg::BM * 128, "the turn fits two stages of an operand");
// 32 rows (blocks 2 h and 2 h + 1) of a wavefront's accumulators into its part of LDS, and four columns of four rows (4 i + lane /
// 16) back.  The 16-byte unit u of row r lies in unit u ^ 4 ((r >> 2) & 3): neither side meets a bank twice.
__device__ __forceinline__ void turn_in(const floatx4 (&acc)[Cfg::MI][Cfg::NI], int h, char* turn, int lane) {
#pragma unroll
  for (int bj = 0; bj < Cfg::NI; ++bj)
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *reinterpret_cast<float*>(turn + (bi * 16 + (lane >> 4) * 4 + r) * 256 + (((bj * 4 + ((lane >> 2) & 3)) ^ (4 * (lane >> 4))) * 16) + (lane & 3) * 4) =
            acc[h * 2 + bi][bj][r];
  __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ floatx4 turn_out(const char* turn, int i, int lane) {
  return *reinterpret_cast<const floatx4*>(turn + (i * 4 + (lane >> 4)) * 256 + (((lane & 15) ^ (4 * (i & 3))) * 16));
}
// dW that is added to is read past the caches (two updates of which the second adds, 203 rows of 2048 1454 -> 1380 us, 300 1950 -> 1885, 725 rows four times 5.82 ->
// 5.73 ms) unless its rows start in the middle of 64 bytes: then every piece of a row shares lines with its neighbours, which read them once more.  Four updates of 200
// rows of 2048 against 115 915, first of all through the caches, past them: 2056 columns 1943.6 and 2199.1 us (both products), 3592 against 60 001 1777.9 and
// 2136.5, but 2064 1861.1 and 1930.8 in an update of 2966.7 and 2806.  A dW that the memory-side cache holds is read past the others all the same: eight of 367 rows
// of 1096 against 50 001 (209 MiB) 2461 us and 2383.
__device__ __forceinline__ bool past_caches(int d, int V) { return d % 16 == 0 || !beyond_cache(d, V, int64_t{128} << 20); }   // twice that in dW
// `turn` is the wavefront's own part of LDS
template <class C>
__device__ __forceinline__ void store_acc_f32(const floatx4 (&acc)[C::MI][C::NI], char* turn, float* out, int64_t ld, int64_t rows, int cols,
                                              int accumulate, bool past) {
  static_assert(C::WTM == Cfg::WTM && C::WTN == Cfg::WTN, "the turn is written for these");
  typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));   // dW has the alignment of a float
  const int tid = tile_thread(), lane = tid & 63, wave = tid >> 6;
  const int r0 = wave / C::WN * C::WTM, c0 = wave % C::WN * C::WTN + (lane & 15) * 4;
  const bool whole = rows >= C::BM && cols >= C::BN && ld <= kPieceLd;   // the same for every thread
  float* const dst = out + (r0 + (lane >> 4)) * ld + c0;
  constexpr int kPieces = C::MI / 2;
  // Each case is a run of its own: with the branches inside, the waits cannot tell what is under way and are for everything, the stores of
  // the piece before included.
  auto pieces = [&](auto add, auto past) {
    constexpr bool kAdd = decltype(add)::value;
    constexpr int kRead = decltype(past)::value ? kStream : kCached;
    // (one offset a lane and one a piece: 32 addresses of 64 bits would be a quarter of the registers)
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const int w_row = __builtin_amdgcn_readfirstlane(r0), w_col = __builtin_amdgcn_readfirstlane(wave) % C::WN * C::WTN;
    const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(out + w_row * ld + w_col);
    const int at = static_cast<int>((lane >> 4) * ld + (lane & 15) * 4) * 4, step = static_cast<int>(ld) * 16;   // four rows
    floatx4 have[8];                                                 // what is there already, a piece ahead
    auto fetch = [&](int h) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        have[i] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, at, (h * 8 + i) * step, kRead));
    };
    if constexpr (kAdd) fetch(0);
#pragma unroll
    for (int h = 0; h < kPieces; ++h) {
      turn_in(acc, h, turn, lane);
      floatx4 x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = turn_out(turn, i, lane);
      if constexpr (kAdd) {
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] += have[i];
        if (h + 1 < kPieces) fetch(h + 1);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x[i]), rsrc, at, (h * 8 + i) * step, kStream);
      }
      __builtin_amdgcn_wave_barrier();
    }
  };
  if (whole && accumulate && past) {
    pieces(std::true_type(), std::true_type());
  } else if (whole && accumulate) {
    pieces(std::true_type(), std::false_type());
  } else if (whole) {
    pieces(std::false_type(), std::false_type());
  } else {
#pragma unroll
    for (int h = 0; h < kPieces; ++h) {
      turn_in(acc, h, turn, lane);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const floatx4 x = turn_out(turn, i, lane);
        if (r0 + h * 32 + i * 4 + (lane >> 4) < rows && c0 < cols) {
          f32x4_a4* const at = reinterpret_cast<f32x4_a4*>(dst + (h * 32 + i * 4) * ld);
          *at = accumulate ? x + *at : x;
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
}
typedef uint32_t u32x2_a2 __attribute__((ext_vector_type(2), aligned(2)));     // dH has the alignment of its entries
// What the sliced products leave behind: partial sums in blocks of 256 x 256 floats [slice][row tile][column tile].
struct DhSlices {
  int n;                // slices of the vocabulary (1: the tiles write dH themselves)
  int voc_blks;         // vocabulary blocks of 256 per slice (the last slice may have fewer)
  float* part;
};
// tile_m counts the chunk's live blocks of rows, of m_rows rows, nobody looks at those behind; orig_blk is the block's place in the chunk
__device__ __forceinline__ void dh_tile(int tile_m, int m_rows, int orig_blk, int tile_n, int slice, const DhSlices& sl, int tiles_r, int tiles_d,
                                        const uint16_t* __restrict__ dZ, int blk_pitch, int64_t Vp,
                                        const uint16_t* __restrict__ W, int d, int V, uint16_t* __restrict__ dH,
                                        const int32_t* __restrict__ rowsel, int64_t c0, int64_t rows,
                                        const int32_t* __restrict__ ids, const float* __restrict__ g_c,
                                        const float* __restrict__ sc, bool w_once, uint16_t* lds) {
  using C = Cfg;
  const int64_t m0 = static_cast<int64_t>(orig_blk) * C::BM;
  const int n0 = tile_n * C::BN;
  const int voc_blk = slice * sl.voc_blks, tiles_v = static_cast<int>(Vp >> 8);
  const int k_len = min(sl.voc_blks, tiles_v - voc_blk) * 256;       // a multiple of 256, at least 256
  const KContig ca = blocked_rows_tile<C>(dZ, blk_pitch, tiles_v, tile_m, voc_blk, m_rows);
  KMajor kb;
  kb.base = reinterpret_cast<const char*>(W + static_cast<int64_t>(voc_blk) * 256 * d + n0);
  kb.ld_bytes = static_cast<int64_t>(d) * 2;
  kb.hi_bytes = 0;
  kb.k_rows = V - voc_blk * 256;                                     // dz is zero for vocabulary ids past V
  kb.n_units = min(32, (d - n0) / 8);
  floatx4 acc[C::MI][C::NI];
  zero_acc<C>(acc);
  // the third LDS stage goes to W: every group of row tiles streams all of it (twice the bytes of the [rows, V] operand).  With one
  // row tile W is read once: past the caches where it is larger than they are, so that the operand, which every column tile
  // reads, stays there (both products of 203 rows of 3584 762 -> 707 us, of 60 rows of 2048 449 -> 384; with up to four row tiles
  // 725 rows that add to dW gain 1.7 %, 1000 rows lose 1 to 3).
  // Up to half a tile of rows is multiplied by half of the wavefronts only, which halves the time of the matrix cores: every SIMD has one of either
  // half.  (With the same loop for all numbers of rows 203 and 725 rows take 0.4 % longer.)
  if (m_rows <= C::WTM && w_once) mfma_mainloop_mixed<C, false, true, 2, true, true>(ca, KMajor{}, KContig{}, kb, k_len, lds, acc, m_rows);
  else if (m_rows <= C::WTM) mfma_mainloop_mixed<C, false, true, 2, false, true>(ca, KMajor{}, KContig{}, kb, k_len, lds, acc, m_rows);
  else if (w_once) mfma_mainloop_mixed<C, false, true, 2, true>(ca, KMajor{}, KContig{}, kb, k_len, lds, acc);
  else mfma_mainloop_mixed<C, false, true, 2>(ca, KMajor{}, KContig{}, kb, k_len, lds, acc);
  if (sl.n > 1) {
    float* out = sl.part + ((static_cast<int64_t>(slice) * tiles_r + tile_m) * tiles_d + tile_n) * (C::BM * C::BN);
    store_acc_f32<C>(acc, reinterpret_cast<char*>(lds) + (tile_thread() >> 6) * kTurnBytes, out, C::BN, C::BM, C::BN, 0, false);
    return;
  }
  // dH rows leave like the float32 ones: 32 rows at a time through LDS, 128 bytes of four rows to a store, the row numbers,
  // factors and rows of W of a piece fetched together.  (One 2-byte entry after the other, each with its own chain of loads:
  // both products of 39 000 rows of 2048 37.43 ms, like this 37.16, 12 000 rows 11.48 and 11.37.)
  const int tid = tile_thread(), lane = tid & 63, wave = tid >> 6;
  char* turn = reinterpret_cast<char*>(lds) + wave * kTurnBytes;
  const int64_t r0 = m0 + wave / C::WN * C::WTM + (lane >> 4);
  const int j = n0 + wave % C::WN * C::WTN + (lane & 15) * 4, jw = min(j, d - 4);   // d is a multiple of 8: four columns are all inside or all outside
#pragma unroll
  for (int h = 0; h < C::MI / 2; ++h) {
    int64_t row[8];
    float g[8], f[8];
    uint2 w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t n = c0 + min(r0 + h * 32 + i * 4, rows - 1);
      row[i] = rowsel ? rowsel[n] : n;
      g[i] = g_c[n];
      f[i] = sc ? sc[n] : 1.f;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {                                    // g = 0 for invalid ids
      const int64_t id = g[i] != 0.f ? ids[row[i]] : 0;
      w[i] = *reinterpret_cast<const uint2*>(W + id * d + jw);
    }
    turn_in(acc, h, turn, lane);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      floatx4 v = turn_out(turn, i, lane);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        v[k] = sc ? f[i] * v[k] : v[k];
        const uint32_t wk = k < 2 ? w[i].x : w[i].y;
        if (g[i] != 0.f) v[k] += g[i] * __uint_as_float(k & 1 ? wk & 0xffff0000u : wk << 16);
      }
      if (r0 + h * 32 + i * 4 < rows && j < d)
        *reinterpret_cast<u32x2_a2*>(dH + row[i] * d + j) = u32x2_a2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    }
    __builtin_amdgcn_wave_barrier();
  }
}
// Hs: the rows of H that go with the rows of dZ (scaled by the keeping pass), in column blocks [d / 256][mcp][256] so that a
// tile's k-rows are one run of memory
// k_len: rows of the packed [rows, V] operand, whole steps of 64 (0 when no block is live); rows: those that exist
__device__ __forceinline__ void dw_tile(int tile_m, int tile_n, const uint16_t* __restrict__ dZ, int blk_pitch, int64_t mcp, int64_t Vp,
                                        const uint16_t* __restrict__ Hs, int d, int V, int k_len, int rows, float* __restrict__ dW,
                                        int accumulate, uint16_t* lds) {
  using C = Cfg;
  const int64_t m0 = static_cast<int64_t>(tile_m) * C::BM;
  const int n0 = tile_n * C::BN;
  KMajor ka;                                                         // blocked dZ: k = row of the chunk, entries = vocabulary
  ka.base = reinterpret_cast<const char*>(dZ + blk_offset(0, tile_m, Vp >> 8) * blk_pitch);
  ka.ld_bytes = 512;
  ka.hi_bytes = (Vp >> 8) * kBlkElems * 2 * blk_pitch - 256 * 512;               // from the last row of a block to the block below
  ka.k_rows = k_len;
  ka.n_units = 32;
  KMajor kb;                                                         // rows of H: k = row of the chunk, entries = hidden columns
  kb.base = reinterpret_cast<const char*>(Hs + static_cast<int64_t>(tile_n) * mcp * 256);
  kb.ld_bytes = 512;
  kb.hi_bytes = 0;
  kb.k_rows = rows;                                                  // dz is zero for rows past the chunk
  kb.n_units = min(32, (d - n0) / 8);
  floatx4 acc[C::MI][C::NI];
  zero_acc<C>(acc);
  if (k_len > 0) mfma_mainloop_mixed<C, true, true, 1>(KContig{}, ka, KContig{}, kb, k_len, lds, acc);
  store_acc_f32<C>(acc, reinterpret_cast<char*>(lds) + (tile_thread() >> 6) * kTurnBytes, dW + m0 * d + n0, d, V - m0, d - n0, accumulate, past_caches(d, V));   // d is a multiple of 8
}

// dW of at most 256 rows.  A tile of 256 x 256 that a compute unit works on alone is products, then stores, and the next tile's first loads wait for these
// stores (a wavefront's memory operations are counted in order): 203 rows of 3584 against 152 064 485 us, of which the products alone are 235 and the
// stores of 2.2 GB 396 (5.5 TB/s, as much as a kernel that only stores such tiles reaches).  Here tiles of 256 x 128 have two workgroups to
// a compute unit, so that one multiplies while the other stores, and a workgroup of its own each, which ends without waiting for its stores: 400
// to 430 us.  K is walked in steps of 32 rows through three LDS stages of 24 KB, loaded two steps ahead, the fragments half a step ahead (read when they are
// wanted: updates of 100 and 203 rows 1 % slower).  (Stored through the caches: 1075 us for
// the update in place of 972.)
using ShortCfg = TileCfg<256, 128, 2, 2>;
constexpr int kShortA = 32 * 512, kShortStage = kShortA + 32 * 256, kShortLds = 3 * kShortStage;
static_assert(2 * kShortLds <= 160 * 1024 && 3 * kTurnBytes <= kShortStage, "two workgroups to a compute unit; the turns of three wavefronts fit a stage");
constexpr int kShortGM = 4, kShortGN = 16;               // tiles that the 64 workgroups of an XCD work on together
__global__ void __launch_bounds__(ShortCfg::T, 2)
k_dw_short(const uint16_t* __restrict__ dZ, int blk_pitch, int64_t Vp, int64_t mcp, const uint16_t* __restrict__ Hs, int d, int V, int tiles_v,
           int tiles_n, const LiveInfo* __restrict__ info, float* __restrict__ dW, int accumulate) {
  using C = ShortCfg;
  __shared__ __attribute__((aligned(16))) char lds[kShortLds];
  const int total = tiles_v * tiles_n, per = (total + 7) / 8, t = static_cast<int>(blockIdx.x & 7) * per + static_cast<int>(blockIdx.x >> 3);
  if (static_cast<int>(blockIdx.x >> 3) >= per || t >= total) return;
  int tile_m, tile_n;
  tile_of_groups<kShortGM, kShortGN>(t, tiles_v, tiles_n, &tile_m, &tile_n);
  const int k_rows = info->k_rows, nsub = (k_rows + 31) / 32;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / C::WN, wn = wave % C::WN;
  const char* const a0 = reinterpret_cast<const char*>(dZ + blk_offset(0, tile_m, Vp >> 8) * blk_pitch);
  const int64_t blk_row = (Vp >> 8) * kBlkElems * 2 * blk_pitch;                                     // from a block of rows to the next
  const char* const b0 = reinterpret_cast<const char*>(Hs + (static_cast<int64_t>(tile_n >> 1) * mcp) * 256 + (tile_n & 1) * 128);
  // loads (K-major operands as in mfma_mainloop_mixed): one fills two k-rows of A, four of B
  const int ka = 2 * wave + (lane >> 5), kb = 4 * wave + (lane >> 4);                                // + 8 p; + 16 p
  const uint32_t ua = static_cast<uint32_t>((lane & 31) ^ (4 * (ka & 3))), ub = static_cast<uint32_t>((lane & 15) ^ (4 * (kb & 3)) ^ (2 * ((kb >> 3) & 1)));
  auto load = [&](int sub) {
    char* const st = lds + sub % 3 * kShortStage;
    const int k0 = sub * 32;
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(a0 + (k0 >> 8) * blk_row + (k0 & 255) * 512), rb = make_rsrc(b0 + static_cast<int64_t>(k0) * 512);
#pragma unroll
    for (int p = 0; p < 4; ++p)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, reinterpret_cast<uint32_t*>(st + (8 * p + 2 * wave) * 512), 16,
                                               static_cast<uint32_t>(8 * p + ka) * 512u + (ua ^ (2u * (p & 1))) * 16u, 0, 0, kCached);
#pragma unroll
    for (int p = 0; p < 2; ++p)                            // dz is zero for rows that do not exist: the last one in their place
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, reinterpret_cast<uint32_t*>(st + kShortA + (16 * p + 4 * wave) * 256), 16,
                                               static_cast<uint32_t>(min(16 * p + kb, k_rows - 1 - k0)) * 512u + ub * 16u, 0, 0, kCached);
  };
  // fragments through the transposing reads
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)(lds)));
  const int tq = lane & 3, tj = (lane >> 2) & 3, tg = lane >> 4;
  uint32_t tra[C::MI], trb[C::NI];
#pragma unroll
  for (int i = 0; i < C::MI; ++i)
    tra[i] = lds0 + (tg * 8 + tj) * 512 + (tq & 1) * 8 + (((wm * (C::WTM / 8) + i * 2 + (tq >> 1)) ^ (4 * tj) ^ (2 * (tg & 1))) * 16);
#pragma unroll
  for (int j = 0; j < C::NI; ++j)
    trb[j] = lds0 + kShortA + (tg * 8 + tj) * 256 + (tq & 1) * 8 + (((wn * (C::WTN / 8) + j * 2 + (tq >> 1)) ^ (4 * tj) ^ (2 * (tg & 1))) * 16);
  typedef short short8v __attribute__((ext_vector_type(8)));
  constexpr int HA = C::MI / 2;
  bf16x8 af[2][HA], bfr[2][C::NI];
  auto read = [&](uint32_t addr, auto row_c) {
    short4v lo, hi;
    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(lo) : "v"(addr));
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(addr), "n"(4 * decltype(row_c)::value));
    const short8v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  };
  using RowA = std::integral_constant<int, 512>;
  using RowB = std::integral_constant<int, 256>;
  auto read_a = [&](int h, uint32_t st) {
#pragma unroll
    for (int i = 0; i < HA; ++i) af[h][i] = read(tra[h * HA + i] + st, RowA{});
  };
  auto read_b = [&](int buf, uint32_t st) {
#pragma unroll
    for (int j = 0; j < C::NI; ++j) bfr[buf][j] = read(trb[j] + st, RowB{});
  };
  auto wait_a = [&](int h) {
#pragma unroll
    for (int i = 0; i < HA; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(af[h][i]));
  };
  auto wait_b = [&](int buf) {
#pragma unroll
    for (int j = 0; j < C::NI; ++j) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(bfr[buf][j]));
  };
  floatx4 acc[C::MI][C::NI];
  zero_acc<C>(acc);
  auto mfmas = [&](int h, int buf) {
#pragma unroll
    for (int i = 0; i < HA; ++i)
#pragma unroll
      for (int jj = 0; jj < C::NI; ++jj) {
        const int j = i & 1 ? C::NI - 1 - jj : jj;
        acc[h * HA + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[h][i], bfr[buf][j], acc[h * HA + i][j], 0, 0, 0);
      }
  };
  auto stage = [&](int sub) { return static_cast<uint32_t>(sub % 3 * kShortStage); };
  // One step: the second half of its A fragments is read under the products of the first, the next step's B and first half under those of the
  // second.  The barrier in between: the next step's loads have landed, and everybody has read this step's stage, which is loaded again.
  auto step = [&](int sub, auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    wait_b(buf);
    wait_a(0);
    read_a(1, stage(sub));
    mfmas(0, buf);
    __builtin_amdgcn_sched_barrier(0);
    wait_a(1);
    if (sub + 1 < nsub) {
      if (sub + 2 < nsub) __builtin_amdgcn_s_waitcnt(0x0F70 | 6); else __builtin_amdgcn_s_waitcnt(0x0F70);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      if (sub + 3 < nsub) load(sub + 3);
      read_b(buf ^ 1, stage(sub + 1));
      read_a(0, stage(sub + 1));
    }
    mfmas(1, buf);
    __builtin_amdgcn_sched_barrier(0);
  };
  if (nsub > 0) {
    load(0);
    if (nsub > 1) load(1);
    if (nsub > 2) load(2);
    if (nsub > 2) __builtin_amdgcn_s_waitcnt(0x0F70 | 12); else if (nsub > 1) __builtin_amdgcn_s_waitcnt(0x0F70 | 6); else __builtin_amdgcn_s_waitcnt(0x0F70);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read_b(0, 0);
    read_a(0, 0);
    for (int sub = 0; sub < nsub; sub += 2) {
      step(sub, std::integral_constant<int, 0>());
      if (sub + 1 < nsub) step(sub + 1, std::integral_constant<int, 1>());
    }
  }
  // the turns lie in the two stages that nobody reads any more and no load is under way to
  char* const turn = lds + (nsub + (wave == 3 ? 1 : 0)) % 3 * kShortStage + (wave == 3 ? 0 : wave) * kTurnBytes;
  const int64_t m0 = static_cast<int64_t>(tile_m) * C::BM;
  const int n0 = tile_n * C::BN;
  store_acc_f32<C>(acc, turn, dW + m0 * d + n0, d, V - m0, d - n0, accumulate, past_caches(d, V));
}
// Both products in one launch, in groups of 4 x 8 tiles that are worked on together on one XCD.  Every XCD owns a contiguous
// range of the dH tiles (slice after slice, so that its workgroups share a slice of both operands) and behind it the share
// of the dW tiles that evens out the sum (share_dw): dH tiles are long (K = vocabulary, or a slice of it) and few, on their
// own they leave a fifth of the last round idle; they go first and the many short dW tiles fill up.  (Sliced dH tiles and
// dW tiles taking turns instead: +-1 % at 725 rows, 8 % slower at 203.)
// One workgroup per compute unit stays for the whole launch and takes the next place of its XCD's sequence whenever it is done
// (the number of the next place is fetched a tile ahead): a workgroup per tile paid for its start at every tile, of which short
// selections have many short ones, and workgroups without a tile (groups cut off by the edge, places kept free because
// the shares are known on the device only) waited for a whole compute unit like the others.  A workgroup whose sequence is at
// its end goes on with the one that has most left.  203 rows of 3584 1316 -> 845 us, 64 rows of 2048 841 -> 455, 725 rows
// 1098 -> 930, 2000 rows of 3584 3.93 -> 3.52 ms, 39 000 rows of 2048 37.5 -> 36.5 ms.
__global__ void __launch_bounds__(Cfg::T)
k_gemm_dh_dw(const uint16_t* __restrict__ dZ, int blk_pitch, int64_t Vp, int64_t mcp, const uint16_t* __restrict__ W,
             const uint16_t* __restrict__ Hs, int d, int V, int tiles_v,
             int tiles_d, DhSlices sl, int tiles_r, LiveInfo* __restrict__ info, const int32_t* __restrict__ blk_orig,
             uint16_t* __restrict__ dH, float* __restrict__ dW, int accumulate, const int32_t* __restrict__ rowsel,
             int64_t c0, int64_t rows, const int32_t* __restrict__ ids, const float* __restrict__ g_c,
             const float* __restrict__ sc) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[MixedLdsBytes<Cfg>::value / 2];
  const int n_live = info->n_live;                     // live blocks of rows: dH row tiles, dW K blocks
  const int k_rows = info->k_rows, tiles_mn = n_live * tiles_d, tiles_dh = tiles_mn * sl.n;
  // whose sequence of tiles the workgroup takes from, and the sequence: dH tiles, then dW tiles
  int xcd = static_cast<int>(blockIdx.x & 7), first_dh, n_dh, first_dw, n_all;
  auto sequence = [&]() {
    first_dh = dh_first(tiles_dh, sl.n, xcd);
    n_dh = dh_first(tiles_dh, sl.n, xcd + 1) - first_dh;
    first_dw = info->dw.first[xcd];
    n_all = n_dh + info->dw.first[xcd + 1] - first_dw;
  };
  sequence();
  volatile int* const word = reinterpret_cast<volatile int*>(lds);   // wavefront 0's own at the end of a tile
  int taken = threadIdx.x == 0 ? atomicAdd(&info->next[xcd], 1) : 0;
  for (;;) {
    if (threadIdx.x == 0) *word = taken;
    __syncthreads();
    int seq = __builtin_amdgcn_readfirstlane(*word);
    __syncthreads();
    while (seq >= n_all) {                               // the sequence is at its end: on with the one that has most left
      if (threadIdx.x < kWave) {
        const int x = threadIdx.x & 7;
        const int length = dh_first(tiles_dh, sl.n, x + 1) - dh_first(tiles_dh, sl.n, x) + info->dw.first[x + 1] - info->dw.first[x];
        const int left = length - __hip_atomic_load(&info->next[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int most = left;
#pragma unroll
        for (int o = 4; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, kWave));
        if (most > 0) xcd = __ffsll(static_cast<long long>(__ballot(left == most))) - 1;
        if (threadIdx.x == 0) {
          word[0] = most > 0 ? atomicAdd(&info->next[xcd], 1) : -1;
          word[1] = xcd;
        }
      }
      __syncthreads();
      seq = __builtin_amdgcn_readfirstlane(word[0]);
      xcd = __builtin_amdgcn_readfirstlane(word[1]);
      __syncthreads();
      if (seq < 0) return;
      sequence();
    }
    if (threadIdx.x == 0) taken = atomicAdd(&info->next[xcd], 1);
    int tile_m, tile_n;
    if (seq < n_dh) {
      const int t = first_dh + seq, slice = t / tiles_mn;
      tile_of_groups<kGM, kGN>(t - slice * tiles_mn, n_live, tiles_d, &tile_m, &tile_n);
      dh_tile(tile_m, min(k_rows - tile_m * 256, 256), blk_orig[(c0 >> 8) + tile_m], tile_n, slice, sl, tiles_r, tiles_d, dZ, blk_pitch, Vp, W, d, V, dH, rowsel, c0, rows, ids, g_c, sc, n_live == 1 && beyond_cache(d, V, kDhOnceBytes), lds);
    } else {
      tile_of_groups<kGM, kGN>(first_dw + seq - n_dh, tiles_v, tiles_d, &tile_m, &tile_n);
      dw_tile(tile_m, tile_n, dZ, blk_pitch, mcp, Vp, Hs, d, V, dw_k(k_rows), k_rows, dW, accumulate, lds);
    }
  }
}

// The slices' partial sums of dH added up in slice order, with what the tile epilogue does otherwise: row factor, one-hot
// part, bf16 row through the selection.  One workgroup per (row of the live blocks, 1024 columns), four columns a thread.
__device__ __forceinline__ void
dh_reduce(int live_row, int piece, const DhSlices& sl, int tiles_r, int tiles_d, const uint16_t* __restrict__ W, int d, const LiveInfo* __restrict__ info,
          const int32_t* __restrict__ blk_orig, uint16_t* __restrict__ dH, const int32_t* __restrict__ rowsel, int64_t c0,
          int64_t rows, const int32_t* __restrict__ ids, const float* __restrict__ g_c, const float* __restrict__ sc) {
  const int tile_m = live_row >> 8, r = live_row & 255;
  if (tile_m >= info->n_live) return;
  const int64_t m = static_cast<int64_t>(blk_orig[(c0 >> 8) + tile_m]) * 256 + r;
  const int j = (piece * 256 + static_cast<int>(threadIdx.x)) * 4;
  if (m >= rows || j >= d) return;
  const float* src = sl.part + (static_cast<int64_t>(tile_m) * tiles_d + (j >> 8)) * 65536 + r * 256 + (j & 255);
  const int64_t stride = static_cast<int64_t>(tiles_r) * tiles_d * 65536;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int k0 = 0; k0 < sl.n; k0 += 8) {                             // eight slices in flight
    float4 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = k0 + q < sl.n ? *reinterpret_cast<const float4*>(src + (k0 + q) * stride) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int q = 0; q < 8; ++q) { s.x += v[q].x; s.y += v[q].y; s.z += v[q].z; s.w += v[q].w; }
  }
  const int64_t row = rowsel ? rowsel[c0 + m] : c0 + m;
  const float f = sc ? sc[c0 + m] : 1.f, g = g_c[c0 + m];
  s.x *= f; s.y *= f; s.z *= f; s.w *= f;
  if (g != 0.f) {                                                    // g = 0 for invalid ids
    const uint2 w = *reinterpret_cast<const uint2*>(W + static_cast<int64_t>(ids[row]) * d + j);
    s.x += g * __uint_as_float(w.x << 16); s.y += g * __uint_as_float(w.x & 0xffff0000u);
    s.z += g * __uint_as_float(w.y << 16); s.w += g * __uint_as_float(w.y & 0xffff0000u);
  }
  *reinterpret_cast<u32x2_a2*>(dH + row * d + j) = u32x2_a2{pack_bf16x2(s.x, s.y), pack_bf16x2(s.z, s.w)};
}

// One-hot part of dW: dW[y_n, :] += g_n h_n for every selected row, in float32.  Rows that took the same token add
// into the same dW row, hence atomics - and token frequencies are skewed (a seventh of the rows of a Zipf(1.1) batch
// took the most frequent token), so adding row by row queues thousands of atomics on the same cache lines.  A
// workgroup therefore takes kOneHotRows consecutive selected rows and adds them up by token first: the first row of
// every token in the group is its leader; a wavefront sums the leader and its followers in registers, 2048 columns at
// a time (16-byte loads, a lane owning eight consecutive columns of each of four pieces), turns every piece through
// its corner of LDS so that consecutive lanes hold consecutive columns, and issues one atomic per element of the sum.
// A wavefront needs about a microsecond per token, so with few groups each is worked on by several workgroups; and the
// most frequent token's rows are a chain of loads, so they come four at a time (203 rows of 3584 37 -> 27 us, 725 of 2048 27 -> 20).
constexpr int kOneHotRows = 128;
constexpr int kOneHotPieces = 4;                    // pieces of 512 columns a wavefront holds at a time
constexpr int kOneHotAhead = 4;                     // rows a wavefront loads together
static_assert(kOneHotRows == 2 * kWave, "the rows of a token are two ballots");
__device__ __forceinline__ void
dw_onehot(int group, int part, int parts, const uint16_t* __restrict__ H, int d, const int32_t* __restrict__ rowsel, int64_t n_sel,
          const int32_t* __restrict__ ids, const float* __restrict__ g_c, float* __restrict__ dW) {
  __shared__ __attribute__((aligned(16))) int32_t s_id[kOneHotRows];   // token of the row, -1 when the row adds nothing
  __shared__ float s_g[kOneHotRows];
  __shared__ int64_t s_row[kOneHotRows];
  __shared__ int32_t s_leader[kOneHotRows];         // the group's leaders, compacted
  __shared__ int32_t s_n_leader[kOneHotRows / kWave];
  __shared__ float s_turn[256 / kWave][8 * kWave];  // one piece per wavefront, in column order
  const int tid = threadIdx.x, lane = tid & 63, wave = tid / kWave;
  if (tid < kOneHotRows) {
    const int64_t n = static_cast<int64_t>(group) * kOneHotRows + tid;
    float g = 0.f;
    int64_t row = 0;
    int32_t id = -1;
    if (n < n_sel) {
      g = g_c[n];                                  // 0: clipped rows, zero advantage, invalid ids
      row = rowsel ? rowsel[n] : n;
      if (g != 0.f) id = ids[row];
    }
    s_id[tid] = id; s_g[tid] = g; s_row[tid] = row;
  }
  __syncthreads();
  bool leader = false;
  if (tid < kOneHotRows) {
    const int32_t id = s_id[tid];
    int earlier = 0;                                // rows of the group in front of this one with its token
#pragma unroll 8
    for (int u = 0; u < kOneHotRows; u += 4) {
      const int4 o = *reinterpret_cast<const int4*>(s_id + u);
      earlier += (o.x == id && u < tid) + (o.y == id && u + 1 < tid) + (o.z == id && u + 2 < tid) + (o.w == id && u + 3 < tid);
    }
    leader = id >= 0 && earlier == 0;
  }
  const unsigned long long leaders = __ballot(leader);       // listed in row order: every workgroup of the group has the same list
  if (lane == 0 && wave < kOneHotRows / kWave) s_n_leader[wave] = __popcll(leaders);
  __syncthreads();
  int n_leader = 0, before = 0;
#pragma unroll
  for (int k = 0; k < kOneHotRows / kWave; ++k) { before += k < wave ? s_n_leader[k] : 0; n_leader += s_n_leader[k]; }
  if (leader) s_leader[before + __popcll(leaders & ((1ull << lane) - 1))] = tid;
  __syncthreads();
  float* turn = s_turn[wave];
  // the group's tokens are spread over the wavefronts of `parts` workgroups
  for (int li = wave + part * (256 / kWave); li < n_leader; li += 256 / kWave * parts) {
    const int32_t id = s_id[s_leader[li]];
    float* dst = dW + static_cast<int64_t>(id) * d;
    unsigned long long same[kOneHotRows / kWave];   // the rows of the group that took this token
#pragma unroll
    for (int k = 0; k < kOneHotRows / kWave; ++k) same[k] = __ballot(s_id[lane + kWave * k] == id);
    for (int c0 = 0; c0 < d; c0 += kOneHotPieces * 8 * kWave) {   // d is a multiple of 8: a lane's eight columns are all inside or all outside
      float acc[kOneHotPieces][8];
#pragma unroll
      for (int q = 0; q < kOneHotPieces; ++q)
#pragma unroll
        for (int k = 0; k < 8; ++k) acc[q][k] = 0.f;
      unsigned long long lo = same[0], hi = same[1];
      while (lo | hi) {                               // kOneHotAhead rows are in flight together
        uint4 hv[kOneHotAhead][kOneHotPieces];
        float g[kOneHotAhead];
#pragma unroll
        for (int b = 0; b < kOneHotAhead; ++b) {
          g[b] = 0.f;
          if (!(lo | hi)) {
#pragma unroll
            for (int q = 0; q < kOneHotPieces; ++q) hv[b][q] = make_uint4(0u, 0u, 0u, 0u);
            continue;
          }
          const int u = lo ? __ffsll(static_cast<long long>(lo)) - 1 : kWave + __ffsll(static_cast<long long>(hi)) - 1;
          if (lo) lo &= lo - 1; else hi &= hi - 1;
          const uint16_t* h = H + s_row[u] * d;
          g[b] = s_g[u];
#pragma unroll
          for (int q = 0; q < kOneHotPieces; ++q) {
            const int c = c0 + (q * kWave + lane) * 8;
            hv[b][q] = c < d ? *reinterpret_cast<const uint4*>(h + c) : make_uint4(0u, 0u, 0u, 0u);
          }
        }
#pragma unroll
        for (int b = 0; b < kOneHotAhead; ++b)
#pragma unroll
          for (int q = 0; q < kOneHotPieces; ++q) {
            const uint32_t w4[4] = {hv[b][q].x, hv[b][q].y, hv[b][q].z, hv[b][q].w};
#pragma unroll
            for (int k2 = 0; k2 < 4; ++k2) {
              acc[q][2 * k2] += g[b] * bf2f(static_cast<uint16_t>(w4[k2] & 0xFFFFu));
              acc[q][2 * k2 + 1] += g[b] * bf2f(static_cast<uint16_t>(w4[k2] >> 16));
            }
          }
      }
#pragma unroll
      for (int q = 0; q < kOneHotPieces; ++q) {
        const int cq = c0 + q * 8 * kWave;           // first column of the piece
        if (cq >= d) break;
        // column cq + 8 lane + k sits in this lane's acc[q][k]; after the turn, lane l adds columns cq + 64 k + l
        *reinterpret_cast<float4*>(turn + 8 * lane) = make_float4(acc[q][0], acc[q][1], acc[q][2], acc[q][3]);
        *reinterpret_cast<float4*>(turn + 8 * lane + 4) = make_float4(acc[q][4], acc[q][5], acc[q][6], acc[q][7]);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int c = cq + kWave * k + lane;
          if (c < d) unsafeAtomicAdd(dst + c, turn[kWave * k + lane]);
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
}

// What is left of an update when its products are there, in one launch, as none of it needs the other: the one-hot part of dW,
// the statistics, and the sum of the slices of dH.  The longest first: it is chains of loads, which the sum's bytes hide behind.
// 203 rows of 3584 against 152 064: launches of 18 to 23, 5 and 12 us, in one 24 to 27.
struct CloseArgs {
  unsigned onehot_groups, onehot_parts;   // workgroups of dw_onehot; 0: none
  const uint16_t* H;
  int d;
  const int32_t* rowsel;
  int64_t n_sel;
  const int32_t* ids;
  const float* g_c;
  float* dW;
  unsigned n_stats;                       // workgroups of ppo_stats; 0: none
  int nblk, n_roles;
  float entropy_coef;
  int64_t norm_rows;
  const double* blk_stats;                // NULL: from the rows
  Surrogate S;
  const float *logp_c, *ent_c;
  umas_loss_stats* stats;
  unsigned reduce_rows, reduce_pieces;    // workgroups of dh_reduce; 0: none
  DhSlices sl;
  int tiles_r, tiles_d;
  const uint16_t* W;
  const LiveInfo* info;
  const int32_t* blk_orig;
  uint16_t* dH;
  int64_t c0, rows;
  const float* sc;
};
__global__ void __launch_bounds__(256)
k_update_close(CloseArgs A) {
  unsigned i = blockIdx.x;
  if (i < A.onehot_groups * A.onehot_parts) {
    dw_onehot(i % A.onehot_groups, i / A.onehot_groups, A.onehot_parts, A.H, A.d, A.rowsel, A.n_sel, A.ids, A.g_c, A.dW);
    return;
  }
  i -= A.onehot_groups * A.onehot_parts;
  if (i < A.n_stats) {
    if (A.blk_stats) ppo_stats(i, A.nblk, A.n_roles, A.entropy_coef, A.norm_rows, A.blk_stats, A.stats);
    else ppo_stats_by_row(i, A.S, A.n_sel, A.entropy_coef, A.norm_rows, A.logp_c, A.ent_c, A.stats);
    return;
  }
  i -= A.n_stats;
  dh_reduce(i % A.reduce_rows, i / A.reduce_rows, A.sl, A.tiles_r, A.tiles_d, A.W, A.d, A.info, A.blk_orig, A.dH, A.rowsel, A.c0, A.rows,
            A.ids, A.g_c, A.sc);
}

// ------------------------------------------------------------------ host side
constexpr int64_t kF32ChunkRows = 4096;
constexpr double kF32MaxWork = 137438953472.0;   // 2^37 multiply-adds per product
// A chunk of more rows is no faster: 73 728 rows of 2048 in one chunk 108.6 ms, in two 105.8; 122 880 of 3584 in one 326 ms, in two
// 320.7, in three 315; 163 840 in two 432, in three 427.
constexpr int64_t kMaxChunkRows = 1 << 16;

int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

struct ScoreWs {
  float4* partial;   // [tiles_m][n_pad]
  float* logp_c;
  float* lse_c;
  float* ent_c;
};
size_t carve_score(Carver& c, ScoreWs& w, int64_t n_sel, int V, umas_dtype dt, bool compact) {
  const int64_t n_pad = round_up(n_sel > 0 ? n_sel : 1, Cfg::BN);
  const int64_t tiles_m = (V + Cfg::BM - 1) / Cfg::BM;
  w.partial = dt == UMAS_BF16 ? c.take<float4>(static_cast<size_t>(tiles_m) * n_pad) : nullptr;
  w.logp_c = w.lse_c = w.ent_c = nullptr;
  if (compact) {
    w.logp_c = c.take<float>(n_pad);
    w.lse_c = c.take<float>(n_pad);
    w.ent_c = c.take<float>(n_pad);
  }
  return c.off;
}

struct PpoWs {
  ScoreWs score;
  float* g_c;
  float* a_c;        // per selected row: coefficients of the backward's dense part
  float* kz_c;
  float* cref;       // keeping pass: per selected row, the reference of E and the row factor of dz = sc E
  float* sc;
  double* rest;      // float32 path, in place of these two: sum of the probabilities of the tokens not taken
  int32_t* flags;    // keeping pass: blocks of 256 selected rows whose dz must be recomputed
  int32_t* blk_live; // per block of 256 selected rows: some row has a gradient
  int32_t* blk_cidx; // its place among the live blocks of its chunk, -1 for a dead one
  int32_t* blk_orig; // per chunk: live block -> block of the chunk
  LiveInfo* live;    // of the chunk in work
  double* blk_stats;
  char* chunk;       // rest of the workspace: dZ (or E) [mcp, Vp], then the scaled copy of the chunk's rows of H
  size_t fixed_bytes;
};
// bytes one chunk of mc rows needs
size_t chunk_bytes(int64_t mc, int d, int V, umas_dtype dt) {
  if (dt == UMAS_F32) return align_up(static_cast<size_t>(mc) * V * sizeof(float));
  const int64_t Vp = round_up(V, 256), mcp = round_up(mc, 256);
  return align_up(static_cast<size_t>(mcp) * Vp * 2) + align_up(static_cast<size_t>(mcp) * round_up(d, 256) * 2);
}
// bytes one chunk of mc rows needs whose float32 logits are kept in place of the operand (entropy bonus)
size_t logit_chunk_bytes(int64_t mc, int d, int V) {
  return chunk_bytes(mc, d, V, UMAS_BF16) + static_cast<size_t>(round_up(mc, 256)) * round_up(V, 256) * 2;
}
// The float32 update keeps the logits (float64) of all its rows where that is no more than 1 GiB.  Storing and reading them costs the same
// at every hidden size, a second product costs by it: below 64 columns up to 128 MiB, which the memory-side cache holds together with
// dz, below 32 up to 32 MiB.  Update on new rows, computed twice / kept: 500 rows of 8 against 8000 (30 MiB) 179 / 180 us, 2000 (122) 278 /
// 298, 4000 of 16 against 4000 262 / 279, 1843 of 33 against 8001 359 / 346, 1000 of 40 against 16 000 446 / 458 (on the rows of the call
// before 448 / 427), 2500 of 32 against 8000 (153) 353 / 363, 300 of 64 against 40 000 790 / 789; on the rows of the call before, 12 000
// against 8000, d = 16 1121 / 1277, 32 1310 / 1404, 48 1517 / 1543, 64 1694 / 1639, 40 000 against 1000 d = 32 1384 / 1434, 64
// 1499 / 1513, 96 1727 / 1703.
size_t f32_logit_bytes(int64_t n_sel, int d, int V) {
  const double b = static_cast<double>(n_sel) * V * sizeof(double), most = d < 32 ? 33554432.0 : d < 64 ? 134217728.0 : 1073741824.0;
  return b <= most ? align_up(static_cast<size_t>(n_sel) * V * sizeof(double)) : 0;
}
// ... and, behind them, the statistics of parts of the rows that the update in few launches merges where it makes dz (one chunk of rows).
size_t f32_part_bytes(int64_t n_sel, int V) { return align_up(static_cast<size_t>(f32::part_plan(n_sel, V).splits) * n_sel * sizeof(f32::Stat)); }
bool f32_few_launches(int64_t n_sel, int d, int V, size_t room) {
  const size_t z = n_sel <= kF32ChunkRows ? f32_logit_bytes(n_sel, d, V) : 0;
  return z > 0 && chunk_bytes(n_sel, d, V, UMAS_F32) + z + f32_part_bytes(n_sel, V) <= room;
}
// partial sums of as many slices as are wanted
size_t full_part_bytes(int64_t n_sel, int64_t chunk_rows, int d, int V) {
  if (!slices_dh(n_sel, chunk_rows, d)) return 0;
  const int tiles_r = static_cast<int>(cdiv(chunk_rows, 256)), tiles_d = (d + 255) / 256;
  return dh_part_bytes(plan_dh(tiles_r, tiles_d, (V + 255) / 256, SIZE_MAX), tiles_r, tiles_d);
}
// The update with an entropy bonus keeps the logits of a chunk in float32 instead of computing them a second time where the
// workspace has room for chunks that are not small: the whole selection, or chunks whose dH tiles are whole ones (the same bits
// of dH as from larger workspaces).  0: it has not, the logits are computed twice.
// So they are for hidden sizes below kLogitWidth: a second product costs by the hidden size, the 10 bytes a logit that are stored and
// read more do not.  Update, computed twice / kept, 203, 700 and 3000 rows against 151 937: d = 256 211 / 220, 391 / 465, 1282 / 1622 us;
// 512 288 / 282, 578 / 613, 1985 / 2067; 640 355 / 336, 714 / 738, 2414 / 2459; 768 383 / 356, 765 / 763, 2610 / 2579; 896 452 / 386,
// 924 / 880, 3166 / 3011.
constexpr int kLogitWidth = 768;
// What the workspace is sized for.  A second chunk adds to dW, 0.3 to 0.5 ms at any size: in one and two chunks 8300 rows of 2048 14.15 and 14.43 ms,
// 10 590 (6 GiB) 17.77 and 18.16, 16 100 26.4 and 26.9, 24 000 39.4 and 39.7, 10 500 of 3584 28.9 and 29.3.  Beyond 6 GiB it is 2 % or less, which
// is not worth twice the memory.
constexpr size_t kLogitBytes = size_t{6} << 30;
int64_t logit_chunk_rows(int64_t n_sel, int d, int V, size_t room) {
  if (d < kLogitWidth) return 0;
  if (round_up(V, 256) / 256 > 8192) return 0;             // 32-bit offsets along a row of blocks
  if (dh_tiles(n_sel, d) < kDhSliceTiles) return logit_chunk_bytes(n_sel, d, V) + full_part_bytes(n_sel, n_sel, d, V) <= room ? n_sel : 0;
  const int64_t fit = std::min(static_cast<int64_t>(room / logit_chunk_bytes(256, d, V)) * 256, kMaxChunkRows);
  if (fit >= n_sel) return n_sel;
  if (fit == 0) return 0;
  const int64_t nchunk = (n_sel + fit - 1) / fit, mc = round_up((n_sel + nchunk - 1) / nchunk, 256);
  return dh_tiles(mc, d) >= kDhSliceTiles / 2 ? mc : 0;
}
size_t carve_ppo(Carver& c, PpoWs& w, int64_t n_sel, int d, int V, umas_dtype dt, int n_roles) {
  (void)d;                                      // the per-chunk buffers depend on d, the fixed part does not
  carve_score(c, w.score, n_sel, V, dt, true);
  const int64_t n_pad = round_up(n_sel > 0 ? n_sel : 1, Cfg::BN);
  w.g_c = c.take<float>(n_pad);
  w.a_c = c.take<float>(n_pad);
  w.kz_c = c.take<float>(n_pad);
  w.cref = w.sc = nullptr;
  w.rest = nullptr;
  if (dt == UMAS_F32) {
    w.rest = c.take<double>(n_pad);
  } else {
    w.cref = c.take<float>(n_pad);
    w.sc = c.take<float>(n_pad);
  }
  w.flags = c.take<int32_t>(static_cast<size_t>(cdiv(n_pad, kRowBlock)));
  w.blk_live = c.take<int32_t>(static_cast<size_t>(cdiv(n_pad, kRowBlock)));
  w.blk_cidx = c.take<int32_t>(static_cast<size_t>(cdiv(n_pad, kRowBlock)));
  w.blk_orig = c.take<int32_t>(static_cast<size_t>(cdiv(n_pad, kRowBlock)));
  w.live = c.take<LiveInfo>(1);
  w.blk_stats = c.take<double>(static_cast<size_t>(cdiv(n_pad, kRowBlock)) * (1 + n_roles) * kStat);
  w.chunk = c.base ? c.base + c.off : nullptr;
  w.fixed_bytes = c.off;
  return c.off;
}

umas_status check_model_args(const void* H, const void* W, umas_dtype dt, int64_t n_rows, int d, int V,
                             const int32_t* ids, const int32_t* rowsel, int64_t n_sel) {
  UMAS_REQUIRE(dt == UMAS_F32 || dt == UMAS_BF16, UMAS_EDTYPE, "dtype=%d is neither F32 nor BF16", static_cast<int>(dt));
  UMAS_REQUIRE(n_rows >= 0 && n_sel >= 0, UMAS_EINVAL, "negative row count");
  UMAS_REQUIRE(d >= 1 && V >= 1, UMAS_ESHAPE, "d=%d and V=%d must be positive", d, V);
  UMAS_REQUIRE(dt != UMAS_BF16 || d % 8 == 0, UMAS_ESHAPE, "bf16 needs d %% 8 == 0 (d=%d)", d);
  UMAS_REQUIRE(dt != UMAS_F32 || d <= 8192, UMAS_ESHAPE, "the float32 path supports d <= 8192 (d=%d)", d);
  // the float32 path sums in float64: small shapes only
  UMAS_REQUIRE(dt != UMAS_F32 || static_cast<double>(n_sel) * V * d <= kF32MaxWork, UMAS_ESHAPE,
               "the float32 path is for small shapes: n_sel * V * d = %.3g exceeds %.3g; use bf16",
               static_cast<double>(n_sel) * V * d, kF32MaxWork);
  UMAS_REQUIRE(dt != UMAS_BF16 || static_cast<uint64_t>(n_rows) * d * 2 < (1ull << 32), UMAS_ESHAPE,
               "bf16 H must be smaller than 4 GiB (32-bit buffer offsets): n_rows=%lld d=%d",
               static_cast<long long>(n_rows), d);
  UMAS_REQUIRE(dt != UMAS_BF16 || static_cast<uint64_t>(std::min(V, 256)) * d * 2 < (1ull << 32), UMAS_ESHAPE,
               "256 rows of a bf16 W must be smaller than 4 GiB (32-bit buffer offsets): V=%d d=%d", V, d);
  UMAS_REQUIRE(rowsel || n_sel == n_rows, UMAS_EINVAL, "rowsel is NULL but n_sel != n_rows");
  UMAS_REQUIRE(n_sel <= n_rows, UMAS_EINVAL, "n_sel=%lld exceeds n_rows=%lld", static_cast<long long>(n_sel),
               static_cast<long long>(n_rows));
  UMAS_REQUIRE((H && ids) || n_rows == 0, UMAS_EINVAL, "H and ids must not be NULL");
  UMAS_REQUIRE(W, UMAS_EINVAL, "W must not be NULL");
  UMAS_REQUIRE(reinterpret_cast<uintptr_t>(H) % 16 == 0 && reinterpret_cast<uintptr_t>(W) % 16 == 0, UMAS_EINVAL,
               "H and W must be 16-byte aligned");
  return UMAS_OK;
}

umas_status check_ws(void* ws, size_t have, size_t need) {
  UMAS_REQUIRE(ws && reinterpret_cast<uintptr_t>(ws) % kAlign == 0 && have >= need, UMAS_EWORKSPACE,
               "workspace must be 256-byte aligned and hold %zu bytes (got %zu)", need, have);
  return UMAS_OK;
}

// Four workgroups per compute unit, at most one wavefront per row: 203 rows of 3584 145 -> 29 us, 725 rows of 2048 88 ->
// 25 us, 39 000 rows (307 groups, three workgroups each) 203 -> 195 us; twice and four times as many are no faster.
dim3 onehot_grid(int64_t n_sel) {
  const unsigned groups = cdiv(n_sel, kOneHotRows);
  return dim3(groups, std::min(std::max(1024 / groups, 1u), static_cast<unsigned>(kOneHotRows / 4)));
}
int device_cus() {
  int dev = 0, n_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
    n_cu = 64;
  return n_cu;
}
template <int PPW, class... Args>
void launch_score_few_ppw(int ni, unsigned grid, hipStream_t st, Args... args) {
  if constexpr (PPW <= 4)
    if (ni > 2) { hipLaunchKernelGGL((k_score_few<4, PPW>), dim3(grid), dim3(kFewT), 0, st, args...); return; }
  if (ni <= 1) hipLaunchKernelGGL((k_score_few<1, PPW>), dim3(grid), dim3(kFewT), 0, st, args...);
  else hipLaunchKernelGGL((k_score_few<2, PPW>), dim3(grid), dim3(kFewT), 0, st, args...);
}
template <class... Args>
void launch_score_few(int ppw, Args... args) {
  switch (ppw) {
    case 1: return launch_score_few_ppw<1>(args...);
    case 2: return launch_score_few_ppw<2>(args...);
    case 3: return launch_score_few_ppw<3>(args...);
    case 4: return launch_score_few_ppw<4>(args...);
    case 5: return launch_score_few_ppw<5>(args...);
    case 6: return launch_score_few_ppw<6>(args...);
    case 7: return launch_score_few_ppw<7>(args...);
    default: return launch_score_few_ppw<8>(args...);
  }
}

// decided by the rows of the call, not of the chunk: a row's result does not depend on how the rows are chunked
template <class... Args>
void launch_finalize(int64_t rows, int64_t n_sel, hipStream_t st, Args... args) {
  if (n_sel < kFinSplitRows) hipLaunchKernelGGL(k_score_finalize<true>, dim3(cdiv(rows, 8)), dim3(256), 0, st, args...);
  else hipLaunchKernelGGL(k_score_finalize<false>, dim3(cdiv(rows, 32)), dim3(256), 0, st, args...);
}

// Row tiles that the logit kernels work through together (see tile_coords): an XCD reads all rows of H once for every four
// vocabulary tiles, all XCDs at about the same time, so a panel that stays in the memory-side cache (256 MB) comes from HBM once
// instead of nineteen times.  40 960 rows of 3584 (293 MB), score: all rows 33.4 ms, panels of at most 40 / 64 / 96 / 128 / 160
// MiB 31.5 / 30.6 / 30.7 / 30.5 / 30.7; 24 576 rows kept 20.6 -> 19.3 ms; 40 960 rows of 2048 (168 MB) 18.2 either way.
constexpr int64_t kPanelBytes = int64_t{128} << 20;
int row_panel(int tiles_n, int d) {
  const int most = std::max(static_cast<int>(kPanelBytes / (static_cast<int64_t>(Cfg::BN) * d * 2)) / kGN * kGN, kGN);
  const int panels = (tiles_n + most - 1) / most;
  return ((tiles_n + panels - 1) / panels + kGN - 1) / kGN * kGN;
}

// Tiles of every XCD that are cut in two (see score_tiles): those of the last round of compute units where it is at most half full.
int halved_tiles(int tiles_m, int tiles_n) {
  if (tiles_n > kGN) return 0;
  const int per_xcd = static_cast<int>(cdiv(static_cast<size_t>(tiles_m) * tiles_n, 8)), cus = std::max(device_cus() / 8, 1), rest = per_xcd % cus;
  return rest * 2 <= cus ? rest : 0;
}
dim3 score_grid(int tiles_m, int tiles_n, int panel, int halved) {
  return dim3(tile_grid<kGM, kGN>(tiles_m, tiles_n, panel, kTilesPerWg) + 8 * static_cast<unsigned>(halved));
}

// Forward scoring of the selected rows into compact arrays and/or scattered outputs.  float32: `room` holds statistics of
// parts of the vocabulary (no room: one workgroup per 32 rows walks all of it), rest_c goes with the compact arrays, z (may be
// NULL) takes the logits.
umas_status run_score(const void* H, const void* W, umas_dtype dt, int d, int V, const int32_t* ids,
                      const int32_t* rowsel, int64_t n_sel, const ScoreWs& w, void* room, size_t room_bytes, double* z, double* rest_c,
                      float* logp, float* lse, float* entropy, hipStream_t st) {
  if (n_sel == 0) return UMAS_OK;
  if (dt == UMAS_BF16) {
    int tiles_m = (V + Cfg::BM - 1) / Cfg::BM;
    const int tiles_n = static_cast<int>((n_sel + Cfg::BN - 1) / Cfg::BN);
    int64_t n_pad = round_up(n_sel, Cfg::BN);
    if (n_sel <= few_rows(d)) {
      // partials [workgroups][rows rounded to 16]: no more than the tiles' [V / 256][rows rounded to 256]
      const int ni = n_sel <= 16 ? 1 : n_sel <= 32 ? 2 : 4;
      n_pad = ni * 16;
      tiles_m = std::min(std::min(device_cus(), tiles_m * static_cast<int>(Cfg::BN / n_pad)), static_cast<int>(cdiv(V, 16)));
      launch_score_few(few_pieces(d), ni, tiles_m, st, static_cast<const uint16_t*>(W), static_cast<const uint16_t*>(H), d, V, rowsel,
                       static_cast<int>(n_sel), ids, w.partial, static_cast<int>(n_pad));
      UMAS_LAUNCHED("k_score_few");
    } else if (n_sel <= NarrowCfg::BN) {                     // ceil(V / 128) 128 <= ceil(V / 256) 256: the partials fit as well
      n_pad = NarrowCfg::BN;
      tiles_m = (V + NarrowCfg::BM - 1) / NarrowCfg::BM;
      hipLaunchKernelGGL(k_score_narrow, dim3(tile_grid<kGM, kGN>(tiles_m, 1, kGN, kTilesPerWg)), dim3(NarrowCfg::T), 0, st,
                         static_cast<const uint16_t*>(W), static_cast<const uint16_t*>(H), d, V, rowsel, n_sel, ids,
                         tiles_m, 1, kGN, w.partial, n_pad);
      UMAS_LAUNCHED("k_score_narrow");
    } else {
      const int panel = row_panel(tiles_n, d), halved = halved_tiles(tiles_m, tiles_n);
      hipLaunchKernelGGL(k_score_tiles, score_grid(tiles_m, tiles_n, panel, halved), dim3(Cfg::T), 0, st, static_cast<const uint16_t*>(W),
                         static_cast<const uint16_t*>(H), d, V, rowsel, n_sel, ids, tiles_m, tiles_n, panel, halved, w.partial, n_pad);
      UMAS_LAUNCHED("k_score_tiles");
    }
    launch_finalize(n_sel, n_sel, st, w.partial, tiles_m, n_pad, static_cast<int64_t>(0), n_sel, static_cast<const float*>(nullptr), rowsel, ids, V,
                    w.logp_c, w.lse_c, w.ent_c, logp, lse, entropy);
    UMAS_LAUNCHED("k_score_finalize");
  } else {
    return f32::score(static_cast<const float*>(W), static_cast<const float*>(H), d, V, rowsel, n_sel, ids, room, room_bytes,
                      f32::ScoreOut{z, rest_c, w.logp_c, w.lse_c, w.ent_c, logp, lse, entropy}, st);
  }
  return UMAS_OK;
}

}  // namespace
}  // namespace umas

using namespace umas;

extern "C" size_t umas_policy_logprobs_workspace_bytes(int64_t n_sel, int32_t d, int32_t V, umas_dtype dtype) {
  (void)d;
  if (n_sel < 0 || V < 1) return 0;
  Carver c(nullptr);
  ScoreWs w;
  const size_t b = carve_score(c, w, n_sel, V, dtype, false) + (dtype == UMAS_F32 ? align_up(f32::score_room(n_sel, V)) : 0);
  return b > 0 ? b : kAlign;
}

extern "C" umas_status umas_policy_logprobs(const void* H, const void* W, umas_dtype dtype, int64_t n_rows, int32_t d,
                                            int32_t V, const int32_t* ids, const int32_t* rowsel, int64_t n_sel,
                                            float* logp, float* lse, float* entropy, void* workspace,
                                            size_t workspace_bytes, void* hip_stream) {
  umas_status s = check_model_args(H, W, dtype, n_rows, d, V, ids, rowsel, n_sel);
  if (s != UMAS_OK) return s;
  UMAS_REQUIRE((logp && lse) || n_rows == 0, UMAS_EINVAL, "logp and lse must not be NULL");
  UMAS_REQUIRE(n_sel < (1LL << 31), UMAS_ESHAPE, "at most 2^31-1 selected rows");
  // float32 scores without any room as well
  s = check_ws(workspace, workspace_bytes, dtype == UMAS_F32 ? kAlign : umas_policy_logprobs_workspace_bytes(n_sel, d, V, dtype));
  if (s != UMAS_OK) return s;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  prof_mark(st);
  if (rowsel && n_rows > 0) {
    const size_t bytes = n_rows * sizeof(float);
    UMAS_HIP(clear_bytes(st, logp, bytes, lse, bytes, entropy, bytes));
  }
  Carver c(workspace);
  ScoreWs w;
  carve_score(c, w, n_sel, V, dtype, false);
  return run_score(H, W, dtype, d, V, ids, rowsel, n_sel, w, workspace, workspace_bytes, nullptr, nullptr, logp, lse, entropy, st);
}

// ------------------------------------------------------------------ scoring without any allocation
// The per-tile partials of the scoring pass live in a file-scope device array in place of a caller's workspace.
// Every GPU holds its own copy of the array at its own address, resolved once per device; host code only ever
// uses that resolved address.  Nothing in it has to start at zero: the tile kernel writes every partial that the
// merge kernel reads.
static __device__ __align__(256) unsigned char scratch[UMAS_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices];   // per device: address of `scratch` there, NULL until first used

umas_status static_scratch(void** out) {
  int dev = -1;
  UMAS_HIP(hipGetDevice(&dev));
  UMAS_REQUIRE(dev >= 0 && dev < kMaxDevices, UMAS_ESHAPE, "device %d outside [0,%d)", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    UMAS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    UMAS_REQUIRE(p, UMAS_EHIP, "hipGetSymbolAddress returned no address for the static scratch");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return UMAS_OK;
}
}  // namespace

extern "C" umas_status umas_policy_logprobs_static(const void* H, const void* W, umas_dtype dtype, int64_t n_rows,
                                                   int32_t d, int32_t V, const int32_t* ids, const int32_t* rowsel,
                                                   int64_t n_sel, float* logp, float* lse, float* entropy,
                                                   void* hip_stream) {
  umas_status s = check_model_args(H, W, dtype, n_rows, d, V, ids, rowsel, n_sel);
  if (s != UMAS_OK) return s;
  UMAS_REQUIRE((logp && lse) || n_rows == 0, UMAS_EINVAL, "logp and lse must not be NULL");
  UMAS_REQUIRE(n_sel < (1LL << 31), UMAS_ESHAPE, "at most 2^31-1 selected rows");
  const size_t need = dtype == UMAS_F32 ? 0 : umas_policy_logprobs_workspace_bytes(n_sel, d, V, dtype);   // float32 uses none
  UMAS_REQUIRE(need <= static_cast<size_t>(UMAS_STATIC_SCRATCH_BYTES), UMAS_EWORKSPACE,
               "%lld selected rows against a vocabulary of %d need %zu bytes of scratch, the static scratch holds %zu: "
               "score fewer rows per call or use umas_policy_logprobs with a workspace",
               static_cast<long long>(n_sel), V, need, static_cast<size_t>(UMAS_STATIC_SCRATCH_BYTES));
  void* ws = nullptr;
  s = static_scratch(&ws);
  if (s != UMAS_OK) return s;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  prof_mark(st);
  if (rowsel && n_rows > 0) {
    const size_t bytes = n_rows * sizeof(float);
    UMAS_HIP(clear_bytes(st, logp, bytes, lse, bytes, entropy, bytes));
  }
  Carver c(ws);
  ScoreWs w;
  carve_score(c, w, n_sel, V, dtype, false);
  return run_score(H, W, dtype, d, V, ids, rowsel, n_sel, w, nullptr, 0, nullptr, nullptr, logp, lse, entropy, st);
}

extern "C" size_t umas_ppo_loss_workspace_bytes_min(int64_t n_sel, int32_t d, int32_t V, umas_dtype dtype,
                                                    int32_t n_roles) {
  if (n_sel < 0 || d < 1 || V < 1 || n_roles < 0) return 0;
  Carver c(nullptr);
  PpoWs w;
  carve_ppo(c, w, n_sel, d, V, dtype, n_roles);
  const int64_t mc = n_sel < 256 ? (n_sel > 0 ? n_sel : 1) : 256;
  return c.off + chunk_bytes(mc, d, V, dtype);
}

namespace {
// The size at which an update runs in the fewest passes; `bonus`: with room for the logits that one with an entropy bonus keeps.
size_t full_ppo_bytes(int64_t n_sel, int d, int V, umas_dtype dtype, int n_roles, bool bonus) {
  if (n_sel < 0 || d < 1 || V < 1 || n_roles < 0) return 0;
  Carver c(nullptr);
  PpoWs w;
  carve_ppo(c, w, n_sel, d, V, dtype, n_roles);
  int64_t mc = n_sel > 0 ? n_sel : 1;
  const int64_t cap = dtype == UMAS_F32 ? kF32ChunkRows : kMaxChunkRows;
  if (mc > cap) {
    const int64_t nchunk = (mc + cap - 1) / cap;
    mc = round_up((mc + nchunk - 1) / nchunk, 256);
  }
  size_t chunk = chunk_bytes(mc, d, V, dtype);
  if (dtype == UMAS_F32) {                                                           // kept with any coefficient
    const size_t z = f32_logit_bytes(n_sel, d, V);
    return c.off + chunk + z + (z > 0 && n_sel <= kF32ChunkRows ? f32_part_bytes(n_sel, V) : 0);
  }
  const size_t parts = full_part_bytes(n_sel, mc, d, V);
  if (bonus) {
    // the logits of the whole selection, of half a chunk where they are many; no room that the call would not keep logits in
    const int64_t rows = mc >= n_sel && logit_chunk_bytes(mc, d, V) <= kLogitBytes ? mc : round_up((mc + 1) / 2, 256);
    const size_t with = std::max(chunk, logit_chunk_bytes(rows, d, V));
    if (logit_chunk_rows(n_sel, d, V, with + parts) > 0) chunk = with;
  }
  return c.off + chunk + parts;
}
}  // namespace

extern "C" size_t umas_ppo_loss_workspace_bytes(int64_t n_sel, int32_t d, int32_t V, umas_dtype dtype, int32_t n_roles) {
  return full_ppo_bytes(n_sel, d, V, dtype, n_roles, false);
}
extern "C" size_t umas_ppo_loss_workspace_bytes_entropy(int64_t n_sel, int32_t d, int32_t V, umas_dtype dtype, int32_t n_roles) {
  return full_ppo_bytes(n_sel, d, V, dtype, n_roles, true);
}

extern "C" umas_status umas_ppo_loss_fwd_bwd(const void* H, const void* W, umas_dtype dtype, int64_t n_rows, int32_t d,
                                             int32_t V, const int32_t* ids, const int32_t* rowsel, int64_t n_sel,
                                             const float* logp_old, const float* adv, const int32_t* tok_role,
                                             int32_t n_roles, float clip_eps, float entropy_coef, float dual_clip,
                                             int32_t accumulate_dW, int64_t norm_rows, const float* logp_ref,
                                             float kl_coef, umas_loss_stats* stats, float* logp_new, void* dH,
                                             float* dW, void* workspace, size_t workspace_bytes, void* hip_stream) {
  umas_status s = check_model_args(H, W, dtype, n_rows, d, V, ids, rowsel, n_sel);
  if (s != UMAS_OK) return s;
  UMAS_REQUIRE((adv && dH) || n_rows == 0, UMAS_EINVAL, "adv and dH must not be NULL");
  UMAS_REQUIRE(stats && dW, UMAS_EINVAL, "stats and dW must not be NULL");
  UMAS_REQUIRE(n_roles >= 0 && n_roles <= UMAS_MAX_ROLES, UMAS_ESHAPE, "n_roles=%d outside [0,%d]", n_roles, UMAS_MAX_ROLES);
  UMAS_REQUIRE(tok_role || n_roles == 0, UMAS_EINVAL, "tok_role is NULL but n_roles > 0");
  UMAS_REQUIRE(clip_eps > 0.f && clip_eps < 1.f, UMAS_EINVAL, "clip_eps=%g outside (0,1)", static_cast<double>(clip_eps));
  UMAS_REQUIRE(entropy_coef >= 0.f, UMAS_EINVAL, "entropy_coef=%g must not be negative", static_cast<double>(entropy_coef));
  UMAS_REQUIRE(dual_clip == 0.f || dual_clip > 1.f, UMAS_EINVAL, "dual_clip=%g must be 0 (off) or larger than 1",
               static_cast<double>(dual_clip));
  UMAS_REQUIRE(n_sel < (1LL << 31), UMAS_ESHAPE, "at most 2^31-1 selected rows");
  UMAS_REQUIRE(norm_rows == 0 || norm_rows >= n_sel, UMAS_EINVAL, "norm_rows=%lld must be 0 or at least n_sel=%lld",
               static_cast<long long>(norm_rows), static_cast<long long>(n_sel));
  UMAS_REQUIRE(kl_coef >= 0.f, UMAS_EINVAL, "kl_coef=%g must not be negative", static_cast<double>(kl_coef));
  UMAS_REQUIRE(kl_coef == 0.f || logp_ref || n_rows == 0, UMAS_EINVAL, "kl_coef > 0 needs logp_ref");
  s = check_ws(workspace, workspace_bytes, umas_ppo_loss_workspace_bytes_min(n_sel, d, V, dtype, n_roles));
  if (s != UMAS_OK) return s;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  prof_mark(st);
  const size_t esz = dtype == UMAS_BF16 ? 2 : 4;
  Carver c(workspace);
  PpoWs w;
  carve_ppo(c, w, n_sel, d, V, dtype, n_roles);

  if (dtype == UMAS_F32 && n_sel > 0 && f32_few_launches(n_sel, d, V, workspace_bytes - w.fixed_bytes)) {
    const int64_t norm = norm_rows > 0 ? norm_rows : n_sel;
    float* const dz = reinterpret_cast<float*>(w.chunk);
    const size_t z_at = chunk_bytes(n_sel, d, V, dtype), parts_at = z_at + f32_logit_bytes(n_sel, d, V);
    const f32::UpdateArgs U{static_cast<const float*>(W), static_cast<const float*>(H), d, n_sel, n_rows,
                            Surrogate{norm, rowsel, ids, V, logp_old, adv, tok_role, n_roles, clip_eps, dual_clip, logp_ref, kl_coef},
                            entropy_coef / static_cast<float>(norm), entropy_coef, norm_rows, w.score.logp_c, w.score.ent_c, logp_new,
                            reinterpret_cast<double*>(w.chunk + z_at), reinterpret_cast<f32::Stat*>(w.chunk + parts_at), dz,
                            static_cast<float*>(dH), dW, accumulate_dW ? 1 : 0, stats};
    return f32::update(U, st);
  }

  // Without an entropy bonus dz is a row factor times the softmax: the scoring pass keeps the numerators
  // and the logits are not computed a second time.
  const bool keep = dtype == UMAS_BF16 && entropy_coef == 0.f && n_sel > 0;
  // rows that are not selected, and (keeping path, see k_update_open) selected rows in blocks without any gradient,
  // are not visited by the backward
  if (!keep && rowsel && n_rows > 0) {
    UMAS_HIP(clear_bytes(st, logp_new, n_rows * sizeof(float), dH, static_cast<size_t>(n_rows) * d * esz));
  }
  if (!accumulate_dW && n_sel == 0) UMAS_HIP(clear_bytes(st, dW, static_cast<size_t>(V) * d * sizeof(float)));

  // chunks of selected rows sized to the workspace
  const size_t room = workspace_bytes - w.fixed_bytes;
  int64_t mc = n_sel > 0 ? n_sel : 1;
  const int64_t cap = dtype == UMAS_F32 ? kF32ChunkRows : kMaxChunkRows;
  if (mc > cap) mc = cap;
  if (mc > 256 && chunk_bytes(mc, d, V, dtype) > room)   // as many blocks of 256 rows as fit: their bytes are multiples of 256
    mc = std::max<int64_t>(static_cast<int64_t>(room / chunk_bytes(256, d, V, dtype)), 1) * 256;
  if (mc > 256) {   // balance the chunks
    const int64_t nchunk = (n_sel + mc - 1) / mc;
    const int64_t even = round_up((n_sel + nchunk - 1) / nchunk, 256);
    if (even < mc) mc = even;
  }
  UMAS_REQUIRE(chunk_bytes(mc < n_sel ? mc : (n_sel > 0 ? n_sel : 1), d, V, dtype) <= room, UMAS_EWORKSPACE,
               "workspace cannot hold one chunk of %lld rows", static_cast<long long>(mc));

  const int nblk = cdiv(n_sel > 0 ? n_sel : 1, kRowBlock);
  const size_t kPpoLds = (kRowBlock / kWave) * (1 + n_roles) * kStat * sizeof(double);
  const int64_t norm = norm_rows > 0 ? norm_rows : n_sel;   // rows the token mean is taken over
  const float k_ent = norm > 0 ? entropy_coef / static_cast<float>(norm) : 0.f;
  const Surrogate S{norm, rowsel, ids, V, logp_old, adv, tok_role, n_roles, clip_eps, dual_clip, logp_ref, kl_coef};
  const int64_t Vp = round_up(V, 256);
  const uint16_t* Wb = static_cast<const uint16_t*>(W);
  const uint16_t* Hb = static_cast<const uint16_t*>(H);

  // both gradient products of the chunk of `rows` rows from c0 on, and what the slices of dH leave; the partial sums lie
  // behind the chunk's operands or, once the scoring pass's own partials have been merged, in their place
  // (true: dW gets a launch of its own)
  auto dh_plan = [&](int64_t rows, size_t used, DhSlices* sl) {
    const size_t behind = room > used ? room - used : 0;
    const size_t front = static_cast<size_t>(reinterpret_cast<char*>(w.score.logp_c) - reinterpret_cast<char*>(w.score.partial));
    const GradPlan p = plan_gradients(n_sel, rows, d, V, slices_dh(n_sel, mc, d) ? std::max(behind, front) : 0);
    *sl = DhSlices{p.dh.slices, p.dh.voc_blks, behind > front ? reinterpret_cast<float*>(w.chunk + used) : reinterpret_cast<float*>(w.score.partial)};
    return p.dw_apart;
  };
  CloseArgs rest{};
  rest.H = Hb;
  rest.W = Wb;
  rest.d = d;
  rest.rowsel = rowsel;
  rest.n_sel = n_sel;
  rest.ids = ids;
  rest.g_c = w.g_c;
  rest.dW = dW;
  rest.n_stats = 1 + n_roles;
  rest.nblk = nblk;
  rest.n_roles = n_roles;
  rest.entropy_coef = entropy_coef;
  rest.norm_rows = norm_rows;
  rest.blk_stats = w.blk_stats;
  rest.S = S;
  rest.logp_c = w.score.logp_c;
  rest.ent_c = w.score.ent_c;
  rest.stats = stats;
  rest.info = w.live;
  rest.blk_orig = w.blk_orig;
  rest.dH = static_cast<uint16_t*>(dH);
  if (dtype == UMAS_BF16 && n_sel > 0) {
    const dim3 grid = onehot_grid(n_sel);
    rest.onehot_groups = grid.x;
    rest.onehot_parts = grid.y;
  }
  auto close = [&](const CloseArgs& C) -> umas_status {
    const unsigned grid = C.onehot_groups * C.onehot_parts + C.n_stats + C.reduce_rows * C.reduce_pieces;
    if (grid == 0) return UMAS_OK;
    hipLaunchKernelGGL(k_update_close, dim3(grid), dim3(256), 0, st, C);
    UMAS_LAUNCHED("k_update_close");
    return UMAS_OK;
  };
  auto gradients = [&](int64_t c0, int64_t rows, const DhSlices& sl, bool dw_apart, const uint16_t* op, int blk_pitch, const uint16_t* Hs, const float* sc) -> umas_status {
    const int64_t mcp = round_up(rows, 256);
    const int tiles_r = static_cast<int>(mcp / 256), tiles_v = static_cast<int>(Vp / 256), tiles_d = (d + 255) / 256;
    const unsigned grid = static_cast<unsigned>(round_up(device_cus(), 8));      // every XCD's sequence needs somebody
    hipLaunchKernelGGL(k_gemm_dh_dw, dim3(grid), dim3(Cfg::T), 0, st, op, blk_pitch, Vp, mcp, Wb, Hs, d, V, tiles_v,
                       tiles_d, sl, tiles_r, w.live, w.blk_orig, static_cast<uint16_t*>(dH), dW, (accumulate_dW || c0 > 0) ? 1 : 0,
                       rowsel, c0, rows, ids, w.g_c, sc);
    UMAS_LAUNCHED("k_gemm_dh_dw");
    if (dw_apart) {
      const int tiles_n = (d + ShortCfg::BN - 1) / ShortCfg::BN;
      hipLaunchKernelGGL(k_dw_short, dim3(static_cast<unsigned>(round_up(static_cast<int64_t>(tiles_v) * tiles_n, 8))), dim3(ShortCfg::T), 0, st, op, blk_pitch,
                         Vp, mcp, Hs, d, V, tiles_v, tiles_n, w.live, dW, (accumulate_dW || c0 > 0) ? 1 : 0);
      UMAS_LAUNCHED("k_dw_short");
    }
    CloseArgs C = rest;                                  // a chunk's slices are added up before the next one's are written
    if (c0 + rows < n_sel) C.onehot_groups = C.n_stats = 0;
    if (sl.n > 1) {
      C.reduce_rows = static_cast<unsigned>(mcp);
      C.reduce_pieces = cdiv(d, 1024);
      C.sl = sl;
      C.tiles_r = tiles_r;
      C.tiles_d = tiles_d;
      C.c0 = c0;
      C.rows = rows;
      C.sc = sc;
    }
    return close(C);
  };

  // With one the logits are kept instead where the workspace allows it.
  const int64_t mc_z = dtype == UMAS_BF16 && !keep && n_sel > 0 ? logit_chunk_rows(n_sel, d, V, room) : 0;
  if (mc_z > 0) mc = mc_z;
  auto ppo_rows = [&](int64_t c0, int64_t c1) -> umas_status {
    hipLaunchKernelGGL(k_ppo_rows, dim3(std::max(cdiv(c1 - c0, kRowBlock), 1u)), dim3(kRowBlock), kPpoLds, st, S, c0, c1, w.score.logp_c,
                       w.score.ent_c, k_ent, dtype == UMAS_BF16 ? 1 : 0, w.score.lse_c, w.g_c, w.a_c, w.kz_c, w.blk_stats);
    UMAS_LAUNCHED("k_ppo_rows");
    return UMAS_OK;
  };

  // float32: the logits lie behind the chunk's dz
  const size_t z_at = dtype == UMAS_F32 ? chunk_bytes(mc, d, V, dtype) : 0;
  double* const z_kept = dtype == UMAS_F32 && f32_logit_bytes(n_sel, d, V) > 0 && z_at + f32_logit_bytes(n_sel, d, V) <= room
                             ? reinterpret_cast<double*>(w.chunk + z_at) : nullptr;
  if (mc_z > 0) {
    // chunk by chunk, further down
  } else if (!keep) {
    // forward scoring and the surrogate
    s = run_score(H, W, dtype, d, V, ids, rowsel, n_sel, w.score, w.chunk, z_kept ? z_at : room, z_kept, w.rest, logp_new, nullptr, nullptr, st);
    if (s != UMAS_OK) return s;
    s = ppo_rows(0, n_sel);
    if (s != UMAS_OK) return s;
  } else {
    const int tiles_v = static_cast<int>(Vp / 256), tiles_d = (d + 255) / 256;
    auto live_args = [&](int64_t c0, int64_t rows, int slices, bool dw_apart) {
      return LiveArgs{static_cast<int>(c0 >> 8), static_cast<int>(round_up(rows, 256) / 256), rows, kl_coef != 0.f ? 1 : 0,   // a KL term gives every row a gradient
                      dw_apart ? 0 : tiles_v, tiles_d, Vp, slices, w.blk_live, w.blk_cidx, w.blk_orig, w.live};
    };
    OpenArgs O{Hb, Wb, d, V, rowsel, n_sel, ids, adv, nblk, w.blk_live, w.flags, w.cref, static_cast<uint32_t*>(dH),
               n_rows * static_cast<int64_t>(d) / 2, rowsel ? logp_new : nullptr, n_rows, 0, {}};
    if (mc >= n_sel && nblk <= kFewBlocks) {
      DhSlices sl;
      const bool dw_apart = dh_plan(n_sel, chunk_bytes(n_sel, d, V, dtype), &sl);
      O.nblk = O.pack = 1;
      O.live = live_args(0, n_sel, sl.n, dw_apart);
    }
    // (the statistics read the old log-probs and the advantages again once the new log-probs are written)
    auto apart = [&](const void* in) {
      const uintptr_t i = reinterpret_cast<uintptr_t>(in), o = reinterpret_cast<uintptr_t>(logp_new), bytes = static_cast<uintptr_t>(n_rows) * 4;
      return !in || !o || i + bytes <= o || o + bytes <= i;
    };
    const bool logp_new_apart = apart(logp_old) && apart(logp_ref) && apart(adv) && apart(tok_role) && apart(ids);
    // a wavefront per row up to 8192 workgroups; at least 1024 for the clearing
    hipLaunchKernelGGL(k_update_open, dim3(O.nblk + std::min<unsigned>(std::max<unsigned>(cdiv(n_sel, 4), 1024), 8192)), dim3(256), 0, st, O);
    UMAS_LAUNCHED("k_update_open");
    const bool narrow = n_sel <= NarrowCfg::BN;              // one chunk of one block
    const int64_t n_pad = round_up(n_sel, narrow ? NarrowCfg::BN : Cfg::BN);
    const int tiles_m = narrow ? static_cast<int>(Vp / NarrowCfg::BM) : tiles_v;   // of the scores: the partials are as large either way
    for (int64_t c0 = 0; c0 < n_sel; c0 += mc) {
      const int64_t rows = n_sel - c0 < mc ? n_sel - c0 : mc;
      const int64_t mcp = round_up(rows, 256);
      const int tiles_r = static_cast<int>(mcp / 256), panel = row_panel(tiles_r, d), halved = halved_tiles(tiles_v, tiles_r);
      uint16_t* E = reinterpret_cast<uint16_t*>(w.chunk);
      uint16_t* Hs = reinterpret_cast<uint16_t*>(w.chunk + align_up(static_cast<size_t>(mcp) * Vp * 2));
      DhSlices sl;
      const bool dw_apart = dh_plan(rows, chunk_bytes(rows, d, V, dtype), &sl);
      if (!O.pack) {
        hipLaunchKernelGGL(k_live_scan, dim3(1), dim3(512), 0, st, live_args(c0, rows, sl.n, dw_apart));
        UMAS_LAUNCHED("k_live_scan");
      }
      if (narrow)
        hipLaunchKernelGGL(k_score_keep_narrow, dim3(tile_grid<kGM, kGN>(tiles_m, 1, kGN, kTilesPerWg)), dim3(NarrowCfg::T), 0, st, Wb, Hb, d, V,
                           rowsel, rows, ids, tiles_m, w.score.partial, n_pad, w.cref, E, Vp, w.flags, w.blk_cidx);
      else
        hipLaunchKernelGGL(k_score_keep_tiles, score_grid(tiles_v, tiles_r, panel, halved), dim3(Cfg::T), 0, st, Wb, Hb, d, V, rowsel, c0, rows, ids,
                           tiles_v, tiles_r, panel, halved, w.score.partial, n_pad, w.cref, E, Vp, w.flags, w.blk_cidx);
      UMAS_LAUNCHED(narrow ? "k_score_keep_narrow" : "k_score_keep_tiles");
      const KeptRows K{Hb, d, V, E, tiles_v, w.cref, w.flags, w.blk_cidx, w.sc, Hs, mcp};
      if (O.pack && logp_new_apart) {
        const RowsArgs A{w.score.partial, tiles_m, n_pad, n_sel, S, w.score.logp_c, w.score.lse_c, w.score.ent_c, logp_new, w.g_c, w.a_c, w.kz_c, K};
        hipLaunchKernelGGL(k_rows_few, dim3(cdiv(n_sel, 8)), dim3(256), 0, st, A);
        UMAS_LAUNCHED("k_rows_few");
        rest.blk_stats = nullptr;
      } else {
        launch_finalize(rows, n_sel, st, w.score.partial, tiles_m, n_pad, c0, c0 + rows, w.cref, rowsel, ids, V, w.score.logp_c, w.score.lse_c,
                        w.score.ent_c, logp_new, static_cast<float*>(nullptr), static_cast<float*>(nullptr));
        UMAS_LAUNCHED("k_score_finalize");
        s = ppo_rows(c0, c0 + rows);
        if (s != UMAS_OK) return s;
        hipLaunchKernelGGL(k_keep_rows, dim3(cdiv(rows, 4)), dim3(256), 0, st, K, rowsel, c0, rows, ids, w.score.lse_c, w.a_c);
        UMAS_LAUNCHED("k_keep_rows");
      }
      // blocks of rows the scoring pass flagged (a logit far above the row's reference) get dz the long way
      hipLaunchKernelGGL(k_dz_flagged, dim3(kFlaggedGrid), dim3(Cfg::T), 0, st, Wb, Hb, d, V, rowsel, c0, rows, ids,
                         w.score.lse_c, w.a_c, w.kz_c, tiles_v, tiles_r, E, Vp, w.flags, w.blk_cidx);
      UMAS_LAUNCHED("k_dz_flagged");
      s = gradients(c0, rows, sl, dw_apart, E, 1, Hs, w.sc);
      if (s != UMAS_OK) return s;
    }
  }
  if (keep) return UMAS_OK;
  if (dtype == UMAS_F32 || n_sel == 0) {
    s = close(rest);                                     // only the statistics
    if (s != UMAS_OK || n_sel == 0) return s;
  }

  if (dtype == UMAS_F32) {
    float* dz = reinterpret_cast<float*>(w.chunk);
    for (int64_t c0 = 0; c0 < n_sel; c0 += mc) {
      const int64_t rows = n_sel - c0 < mc ? n_sel - c0 : mc;
      const float *Wf = static_cast<const float*>(W), *Hf = static_cast<const float*>(H);
      if (z_kept)
        hipLaunchKernelGGL(f32::k_dz_kept_f32, dim3(cdiv(V, 1024), static_cast<unsigned>(rows)), dim3(256), 0, st, z_kept, V, rowsel, c0, ids,
                           w.score.lse_c, w.rest, w.g_c, w.score.ent_c, w.kz_c, dz);
      else
        hipLaunchKernelGGL(f32::k_dz_f32, dim3(cdiv(V, f32::kVocBlock), cdiv(rows, f32::kTile)), dim3(f32::kWaves * kWave), 0, st, Wf, Hf, d, V,
                           rowsel, c0, rows, ids, w.score.lse_c, w.rest, w.g_c, w.score.ent_c, w.kz_c, dz);
      UMAS_LAUNCHED(z_kept ? "k_dz_kept_f32" : "k_dz_f32");
      f32::launch_gradients(f32::GradArgs{dz, Wf, Hf, d, V, rowsel, c0, static_cast<int>(rows), accumulate_dW || c0 > 0 ? 1 : 0,
                                          static_cast<float*>(dH), dW, 0, 0, 0}, f32::StatArgs{}, st);
      UMAS_LAUNCHED("k_dw_f32");                         // both products: one launch to a chunk
    }
    return UMAS_OK;
  }

  for (int64_t c0 = 0; c0 < n_sel; c0 += mc) {
    const int64_t rows = n_sel - c0 < mc ? n_sel - c0 : mc;
    const int64_t mcp = round_up(rows, 256);
    uint16_t* dZ = reinterpret_cast<uint16_t*>(w.chunk);
    const int tiles_v = static_cast<int>(Vp / 256), tiles_r = static_cast<int>(mcp / 256), tiles_d = (d + 255) / 256;
    const int blk_pitch = mc_z > 0 ? 2 : 1, panel = row_panel(tiles_r, d);
    if (mc_z > 0) {
      const int halved = halved_tiles(tiles_v, tiles_r);
      hipLaunchKernelGGL(k_score_logits, score_grid(tiles_v, tiles_r, panel, halved), dim3(Cfg::T), 0, st, Wb, Hb, d, V,
                         rowsel, c0, rows, ids, tiles_v, tiles_r, panel, halved, w.score.partial, round_up(n_sel, Cfg::BN),
                         reinterpret_cast<float*>(w.chunk), Vp);
      UMAS_LAUNCHED("k_score_logits");
      launch_finalize(rows, n_sel, st, w.score.partial, tiles_v, round_up(n_sel, Cfg::BN), c0, c0 + rows, static_cast<const float*>(nullptr), rowsel,
                      ids, V, w.score.logp_c, w.score.lse_c, w.score.ent_c, logp_new, static_cast<float*>(nullptr), static_cast<float*>(nullptr));
      UMAS_LAUNCHED("k_score_finalize");
      s = ppo_rows(c0, c0 + rows);
      if (s != UMAS_OK) return s;
      hipLaunchKernelGGL(k_dz_from_logits, dim3(static_cast<unsigned>(tiles_v * tiles_r)), dim3(kTurnWaves * kWave), 0, st,
                         reinterpret_cast<float*>(w.chunk), tiles_v, c0, rows, w.score.lse_c, w.a_c, w.kz_c);
      UMAS_LAUNCHED("k_dz_from_logits");
    } else {
      hipLaunchKernelGGL(k_dz_tiles, dim3(tile_grid<kGM, kGN>(tiles_v, tiles_r, panel, kTilesPerWg)), dim3(Cfg::T), 0, st, Wb, Hb, d, V, rowsel,
                         c0, rows, w.score.lse_c, w.a_c, w.kz_c, tiles_v, tiles_r, panel, dZ, Vp);
      UMAS_LAUNCHED("k_dz_tiles");
    }
    uint16_t* Hs = reinterpret_cast<uint16_t*>(w.chunk + align_up(static_cast<size_t>(mcp) * Vp * 2 * blk_pitch));
    hipLaunchKernelGGL(k_dz_rows, dim3(cdiv(rows, 4)), dim3(256), 0, st, Hb, d, V, rowsel, c0, rows, ids, dZ, static_cast<int64_t>(tiles_v),
                       blk_pitch, Hs, mcp);
    UMAS_LAUNCHED("k_dz_rows");
    // with an entropy bonus every row has a gradient: all blocks are live
    DhSlices sl;
    const bool dw_apart = dh_plan(rows, mc_z > 0 ? logit_chunk_bytes(rows, d, V) : chunk_bytes(rows, d, V, dtype), &sl);
    hipLaunchKernelGGL(k_live_scan, dim3(1), dim3(512), 0, st, LiveArgs{static_cast<int>(c0 >> 8), tiles_r, rows, 1, dw_apart ? 0 : tiles_v, tiles_d, Vp, sl.n,
                       w.blk_live, w.blk_cidx, w.blk_orig, w.live});
    UMAS_LAUNCHED("k_live_scan");
    s = gradients(c0, rows, sl, dw_apart, dZ, blk_pitch, Hs, nullptr);
    if (s != UMAS_OK) return s;
  }
  return UMAS_OK;
}
