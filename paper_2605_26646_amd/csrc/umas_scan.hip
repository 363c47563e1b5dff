// Generalised advantage estimation as a masked, segmented reverse scan.
//
// A_t = sum_l (gamma lam)^l delta_{t+l}, delta_t = r_t + gamma V(s_{t+1}) - V(s_t) (paragraph
// "Advantage computation and policy evaluation") is evaluated by its backward recurrence.
// Walking a segment from its last token to its first with the carried state (G, NV) =
// (advantage of the next valid token, value of the next valid token):
//   valid token   G' = gamma*lam*G + gamma*NV + (r - V),  NV' = V
//   masked token  state unchanged, outputs 0
//   segment end   state reset to (0, 0) before the segment's last token
//   turn boundary inside a trajectory segment: state scaled by gamma_turn^(step difference)
// Every one of these is an affine map of (G, NV) of the form
//   G' = a G + b NV + c,  NV' = e NV + f
// and such maps compose associatively, so inside a tile of 1024 tokens the recurrence is a parallel scan over maps:
// threads fold their own four tokens, wavefronts and the block combine the folds, and each thread replays its tokens
// from its incoming state.
//
// One pass over memory (17 bytes per token).  Segments are independent, so the stream is cut into ranges of about
// `chunk` tokens (chunk_tokens) at segment boundaries; a workgroup walks the tiles of one range from right to left and carries the
// state from tile to tile itself, the loads of the next two tiles in flight.  Ranges of ordinary segments need nothing
// from each other: one workgroup per range, in any order (k_gae_scan).
// Only a segment longer than kLongSegment tokens is cut inside.  A range whose right end lies inside such a segment
// is left to a second kernel (k_gae_scan_cut): it first folds all of its tiles into one map and publishes it (a
// second read of that range), composes the published maps of the ranges to its right up to the segment's end into its
// incoming state, and then replays, so a stream that is one giant segment is still spread over the whole device.
// That kernel's workgroups are persistent (range number j G + b from the right in round j of workgroup b) and few
// (one per compute unit at most, a fraction of what the device holds at once, so all of them run together): a range
// only ever waits for maps of ranges to its right, written by the first kernel or by a workgroup that is running,
// and publishing a map waits for nothing, so every wait ends.  When no segment is that long the second kernel finds
// nothing to do and leaves at once.  Few tokens (alone_tokens) are done without it.
#include <type_traits>

#include "umas_common.h"

namespace umas {
namespace {

constexpr int kThreads = 256;
constexpr int kIpt = 4;                          // tokens per thread: one 16-byte load per array, no transposition
constexpr int kTile = kThreads * kIpt;           // tokens per tile
constexpr int kChunkTiles = 8;                   // nominal tiles per range at most
// Nominal tokens per range: a range's tiles are done one after the other, so a stream that makes fewer than 512 ranges of
// eight tiles (4.2 million tokens) is cut finer, into 512 and more where it has as many tiles: two for every compute unit
// (49 152 tokens: 6 ranges of eight tiles 19 us, 48 of one 7 us; the call, waited for, 40 -> 28 us, 400 000 tokens 43 -> 33,
// 225 000 in segments that are cut 91 -> 60; 25 million tokens keep ranges of eight, 62 us).
// Finer ranges are 3 to 7 % faster where all turns are short (42 million tokens in turns of 256 110.5 and 108 us, of 1024 and 4096 154
// and 143), but the number of turns does not say that: of 30 000 tokens and twenty of 100 each 265 and 334 us, 6 million in turns of 15 000 and 128 30
// and 36; and runs of a trajectory may be longer than a range, which is then empty as often as not.
inline int64_t chunk_tokens(int64_t n_tokens) {
  const int64_t tiles = n_tokens / (static_cast<int64_t>(kTile) * 512);
  return (tiles < 1 ? 1 : tiles > kChunkTiles ? kChunkTiles : tiles) * kTile;
}
constexpr int64_t kLongSegment = 16 * kTile;     // a segment end farther away than this does not move a range's edge
// Up to so many tokens a workgroup whose range ends inside a long segment reads on to its end itself instead of leaving the range to
// a second launch, which costs 4 us also when there is nothing to do (turns of 400, 20 000 to 65 000 tokens 10.1 us in two launches that follow each
// other, 6.5 in one; 11 and 5.7 us of the host).  With one segment of all tokens, the longest way to read: 49 152 and 65 536 tokens 28.8
// and 29.9 us in two, 21.5 and 25.1 in one, with values 38.6 and 40.3, 31.5 and 40.3; with step discounts too 42.6 and 44.5, 40.8 and 52.5.
inline int64_t alone_tokens(bool decay) { return (decay ? 48 : 64) * kTile; }

enum : uint8_t { kFlagMask = 1, kFlagTurnEnd = 2, kFlagRunEnd = 4 };
constexpr int kFlagStepShift = 3, kFlagStepMany = 31;   // bits 3-7 of a turn end inside a run: steps to the next turn

struct Aff {
  float a, b, c, e, f;
};
__device__ __forceinline__ Aff aff_identity() { return Aff{1.f, 0.f, 0.f, 1.f, 0.f}; }
// the map "first, then second".  HV = false (no value estimates): NV stays 0, so only G' = a G + c is
// carried and b, e, f are never looked at.
template <bool HV>
__device__ __forceinline__ Aff then(const Aff& first, const Aff& second) {
  Aff r;
  r.a = second.a * first.a;
  if constexpr (HV) {
    r.b = second.a * first.b + second.b * first.e;
    r.c = second.a * first.c + second.b * first.f + second.c;
    r.e = second.e * first.e;
    r.f = second.e * first.f + second.f;
  } else {
    r.b = 0.f;
    r.c = second.a * first.c + second.c;
    r.e = 0.f;
    r.f = 0.f;
  }
  return r;
}
// Inclusive prefix over the wavefront, lane 0's map acting first: moves between lanes that go with the multiplication that uses them (row_shr 1,
// 2, 4, 8 inside the rows of 16 lanes, then the last lane of a row handed to the next row and lane 31 to the upper half); lanes
// without a source are not written.  The composition of "first" (moved) and "second" (own) in place, eight instructions a step against
// the twenty and five trips through LDS of shuffles.  A move reads a register two instructions after it was written at the earliest.
#define UMAS_SCAN_STEP(ctrl)                                                                                                        \
  if constexpr (HV) {                                                                                                               \
    float t;                                                                                                                        \
    asm("s_nop 1\n\tv_mov_b32 %5, %1\n\tv_fmac_f32_dpp %2, %2, %0 " ctrl "\n\tv_fmac_f32_dpp %2, %4, %1 " ctrl                      \
        "\n\tv_mul_f32_dpp %1, %3, %1 " ctrl "\n\tv_fmac_f32_dpp %1, %5, %0 " ctrl "\n\tv_fmac_f32_dpp %4, %4, %3 " ctrl               \
        "\n\tv_mul_f32_dpp %0, %0, %0 " ctrl "\n\tv_mul_f32_dpp %3, %3, %3 " ctrl                                                   \
        : "+v"(m.a), "+v"(m.b), "+v"(m.c), "+v"(m.e), "+v"(m.f), "=&v"(t));                                                         \
  } else {                                                                                                                          \
    asm("s_nop 1\n\tv_fmac_f32_dpp %1, %1, %0 " ctrl "\n\tv_mul_f32_dpp %0, %0, %0 " ctrl : "+v"(m.a), "+v"(m.c));                  \
  }
template <bool HV>
__device__ __forceinline__ void wave_prefix(Aff& m) {   // every lane of the wavefront takes part
  UMAS_SCAN_STEP("row_shr:1 row_mask:0xf bank_mask:0xf")
  UMAS_SCAN_STEP("row_shr:2 row_mask:0xf bank_mask:0xf")
  UMAS_SCAN_STEP("row_shr:4 row_mask:0xf bank_mask:0xf")
  UMAS_SCAN_STEP("row_shr:8 row_mask:0xf bank_mask:0xf")
  UMAS_SCAN_STEP("row_bcast:15 row_mask:0xa bank_mask:0xf")
  UMAS_SCAN_STEP("row_bcast:31 row_mask:0xc bank_mask:0xf")
  asm("s_nop 1" : "+v"(m.a), "+v"(m.b), "+v"(m.c), "+v"(m.e), "+v"(m.f));
}
#undef UMAS_SCAN_STEP
// the map of the lane below, identity in lane 0
template <bool HV>
__device__ __forceinline__ Aff lane_below(const Aff& m) {
  auto move = [](float old, float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), 0x138, 0xF, 0xF, false));   // wave_shr:1
  };
  Aff r = aff_identity();
  r.a = move(1.f, m.a);
  r.c = move(0.f, m.c);
  if constexpr (HV) {
    r.b = move(0.f, m.b);
    r.e = move(1.f, m.e);
    r.f = move(0.f, m.f);
  }
  return r;
}
// One range of the stream.  Ranges are numbered from the right end of the stream.
struct __attribute__((aligned(16))) Range {
  int64_t start, end;          // tokens [start, end); empty when start == end
  int32_t cut_right;           // `end` lies inside a long segment: the state entering the range comes from the right
  int32_t cut_left;            // `start` lies inside a long segment: the range to the left will ask for this one's map
  int64_t pad;
};
static_assert(sizeof(Range) == 32, "two 16-byte loads");

constexpr int kStateWords = 5;                     // a, b, c, e, f (without value estimates only a and c are used)
constexpr unsigned long long kReady = 1ull << 32;  // mark in the upper half of a published word

struct ScanParams {
  int64_t n_tokens;
  int64_t chunk;                    // nominal tokens per range
  uint32_t n_ranges;
  Range* ranges;                    // [n_ranges], written by k_gae_scan
  const int64_t* seg_off;           // [n_seg_entries + 1] ascending segment offsets, from 0 to n_tokens
  int n_seg_entries;
  unsigned long long* range_state;  // [n_ranges][kStateWords]: a published map, one float and its ready mark per 64-bit word
  const uint8_t* flags;        // per token: mask, last-of-turn, last-of-run
  const float* reward;
  const float* value;          // may be NULL
  const int32_t* tok_turn;     // only read when the step discount is on
  const int32_t* turn_step;    // only read when the step discount is on
  uint8_t seg_bit;             // kFlagTurnEnd or kFlagRunEnd: which flag ends a segment
  float gamma, lam, gamma_turn;
  float gl, gl4, gl3g;         // gamma lam as a float, its fourth power, its third times gamma (each rounded once)
};

// A record is published word by word; every word carries its own ready mark, so no ordering between the words
// is needed: a reader takes a record when all of its words are marked.  (Device-scope atomics, relaxed.)
__device__ __forceinline__ void publish_word(unsigned long long* p, float x) {
  __hip_atomic_store(p, kReady | static_cast<unsigned long long>(__float_as_uint(x)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool read_word(unsigned long long* p, float* x) {
  const unsigned long long w = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  *x = __uint_as_float(static_cast<uint32_t>(w));
  return (w >> 32) != 0;
}
template <bool HV>
__device__ __forceinline__ void publish(unsigned long long* rec, const Aff& m) {
  publish_word(rec + 0, m.a);
  publish_word(rec + 2, m.c);
  if constexpr (HV) {
    publish_word(rec + 1, m.b);
    publish_word(rec + 3, m.e);
    publish_word(rec + 4, m.f);
  }
}

// ------------------------------------------------------------------ ranges
// Smallest boundary (value of off[0..n]) that is >= x, for ascending off with off[0] = 0 and off[n] >= x.
// Wavefront-wide: every lane of the calling wavefront takes part and gets the same answer.
__device__ __forceinline__ int64_t boundary_at_or_after(const int64_t* __restrict__ off, int n, int64_t x) {
  if (x <= 0) return 0;
  return off[wave_last_le(off, n, x - 1) + 1];
}
// The same, looked for in the flags of 1024 tokens first: a search in the offsets is three or four trips to memory one behind the other, of
// lines all over them, and while all of memory is busy that is 6 us to find the eight tiles that a range takes 30 us for; the flags are
// the range's own or its neighbour's, and one trip (25 million tokens in turns of 256 72 -> 66.5 us, 19 million in runs of 192 51.5 -> 47; 42 million in
// runs of 5120 and more, where the offsets are searched as well, 165 either way).  0 < x < n_tokens.
__device__ __forceinline__ int64_t boundary_from(const ScanParams& P, int64_t x) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t first = x - 1, p = (first & ~int64_t{15}) + lane * 16;
  uint32_t w[4] = {0u, 0u, 0u, 0u};
  if (p + 16 <= P.n_tokens) {
    const uint4 v = *reinterpret_cast<const uint4*>(P.flags + p);
    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
  } else {
    for (int k = 0; k < 16 && p + k < P.n_tokens; ++k) w[k >> 2] |= static_cast<uint32_t>(P.flags[p + k]) << (8 * (k & 3));
  }
  int at = -1;                                                       // first flagged one of this lane's sixteen tokens
#pragma unroll
  for (int k = 3; k >= 0; --k) {
    const int skip = static_cast<int>(first - p) - 4 * k;            // bytes of the word in front of the first token
    const uint32_t hit = w[k] & (P.seg_bit * 0x01010101u) & (skip <= 0 ? ~0u : skip >= 4 ? 0u : ~0u << (8 * skip));
    at = hit ? 4 * k + (__ffs(static_cast<int>(hit)) - 1) / 8 : at;
  }
  const unsigned long long any = __ballot(at >= 0);
  if (!any) return boundary_at_or_after(P.seg_off, P.n_seg_entries, x);
  const int l = __ffsll(static_cast<long long>(any)) - 1;
  return (first & ~int64_t{15}) + l * 16 + __builtin_amdgcn_readlane(at, l) + 1;
}
// Where the range edge nominally at x really lies: at the next segment boundary unless that is farther than
// kLongSegment away, in which case the edge stays at x, inside the segment (*cut = 1).  *boundary: that boundary.
__device__ __forceinline__ int64_t range_edge(const ScanParams& P, int64_t x, int* cut, int64_t* boundary) {
  *cut = 0;
  *boundary = x <= 0 ? 0 : P.n_tokens;
  if (x <= 0 || x >= P.n_tokens) return *boundary;
  *boundary = boundary_from(P, x);
  if (*boundary - x < kLongSegment) return *boundary;
  *cut = 1;
  return x;
}
// ------------------------------------------------------------------ the scan
// The state that enters range q from the right, found by one wavefront: lane l looks at range q - 1 - l (ranges are
// numbered from the right), and the maps are composed up to the nearest range whose map is a constant, i.e. which
// holds the segment's end.  Only the records up to that range are waited for.
template <bool HV>
__device__ __forceinline__ void look_back(const ScanParams& P, uint32_t q, float* G_in, float* NV_in) {
  const int lane = threadIdx.x & (kWave - 1);
  Aff M = aff_identity();
  for (int64_t base = static_cast<int64_t>(q) - 1;; base -= kWave) {
    const int64_t k = base - lane;
    Aff A{0.f, 0.f, 0.f, 0.f, 0.f};                 // past the right end of the stream: the constant map to (0, 0)
    bool ready = true;
    int first = kWave;
    while (true) {
      if (k >= 0) {
        unsigned long long* rec = P.range_state + static_cast<size_t>(k) * kStateWords;
        ready = read_word(rec + 0, &A.a);
        ready = read_word(rec + 2, &A.c) && ready;
        if constexpr (HV) {
          ready = read_word(rec + 1, &A.b) && ready;
          ready = read_word(rec + 3, &A.e) && ready;
          ready = read_word(rec + 4, &A.f) && ready;
        }
      }
      const bool closed = ready && A.a == 0.f && (!HV || (A.b == 0.f && A.e == 0.f));   // a constant map: nothing further right matters
      const unsigned long long rdy = __ballot(ready), cls = __ballot(closed);
      const int n_ready = rdy == ~0ull ? kWave : __ffsll(static_cast<long long>(~rdy)) - 1;   // ready records in a row from lane 0
      first = cls ? __ffsll(static_cast<long long>(cls)) - 1 : kWave;
      if (first < n_ready || n_ready == kWave) break;
      __builtin_amdgcn_s_sleep(8);
    }
    const int upto = first < kWave ? first : kWave - 1;
    for (int j = 0; j <= upto; ++j) {
      Aff Aj;
      Aj.a = __shfl(A.a, j, kWave);
      Aj.c = __shfl(A.c, j, kWave);
      Aj.b = HV ? __shfl(A.b, j, kWave) : 0.f;
      Aj.e = HV ? __shfl(A.e, j, kWave) : 0.f;
      Aj.f = HV ? __shfl(A.f, j, kWave) : 0.f;
      M = then<HV>(Aj, M);                          // the farther range acts first
    }
    if (first < kWave) break;
  }
  *G_in = M.c;                                      // a constant map: its value
  *NV_in = HV ? M.f : 0.f;
}

// four consecutive tokens from p on, a multiple of four: 16 bytes per array, 4 bytes of flags; tokens past the end of the
// stream read as masked, without flags
struct Raw {
  float4 r4, v4;
  uint32_t w;
};
template <bool HV, bool PAST = false>
__device__ __forceinline__ void load_four(const ScanParams& P, const Range& R, int64_t p, Raw& x) {
  x.r4 = make_float4(0.f, 0.f, 0.f, 0.f);
  x.v4 = x.r4;
  x.w = 0;
  if (p + kIpt <= R.start || p >= R.end) return;    // none of these tokens belongs to the range: a neighbour reads them
  if (p + kIpt <= P.n_tokens) {
    x.r4 = *reinterpret_cast<const float4*>(P.reward + p);
    if constexpr (HV) x.v4 = PAST ? load_stream<float4>(P.value + p) : *reinterpret_cast<const float4*>(P.value + p);
    x.w = *reinterpret_cast<const uint32_t*>(P.flags + p);
  } else {
    float* rp = &x.r4.x;
    float* vp = &x.v4.x;
    for (int j = 0; j < kIpt; ++j)
      if (p + j < P.n_tokens) {
        rp[j] = P.reward[p + j];
        if constexpr (HV) vp[j] = P.value[p + j];
        x.w |= static_cast<uint32_t>(P.flags[p + j]) << (8 * j);
      }
  }
}

// Four consecutive tokens as the walks use them.
struct Four {
  float r[kIpt], v[kIpt];
  uint32_t w;                                       // the flags, 0 for tokens that belong to a neighbour: they change nothing
  float kap[kIpt];                                  // step discount applied before the token (1 = none)
};
// Discounts of 0 .. 30 steps: a power takes a hundred instructions, and where turns are short every wavefront has some in every tile (24 million
// tokens in turns of 300 104 -> 101 us).
constexpr int kKaps = kFlagStepMany;
template <bool DECAY>
__device__ __forceinline__ void fill_kaps(const ScanParams& P, float* s_kap) {   // a barrier follows
  if constexpr (DECAY)
    if (threadIdx.x < kKaps) s_kap[threadIdx.x] = powf(P.gamma_turn, static_cast<float>(threadIdx.x));
}
// 0xFF in the bytes of those of the four tokens from p0 on that lie in the range
__device__ __forceinline__ uint32_t own_bytes(const Range& R, int64_t p0) {
  const int64_t skip = R.start - p0, left = R.end - p0;
  const uint32_t from = skip <= 0 ? ~0u : skip >= kIpt ? 0u : ~0u << (8 * static_cast<int>(skip));
  return left >= kIpt ? from : left <= 0 ? 0u : from & ~(~0u << (8 * static_cast<int>(left)));
}
__device__ __forceinline__ bool has(uint32_t w, int k, uint32_t flag) { return (w >> (8 * k)) & flag; }
constexpr uint32_t kPlainFour = kFlagMask * 0x01010101u;   // four scored tokens, none of which ends anything
template <bool DECAY>
__device__ __forceinline__ Four four_tokens(const ScanParams& P, int64_t p0, const Raw& x, uint32_t w, const float* s_kap) {
  Four T{{x.r4.x, x.r4.y, x.r4.z, x.r4.w}, {x.v4.x, x.v4.y, x.v4.z, x.v4.w}, w, {1.f, 1.f, 1.f, 1.f}};
  if constexpr (DECAY) {
    if (w & (kFlagTurnEnd * 0x01010101u)) {
      uint32_t many = 0u;
#pragma unroll
      for (int k = 0; k < kIpt; ++k) {
        if (has(w, k, kFlagTurnEnd) && !has(w, k, P.seg_bit)) {   // a later turn of the same run follows: p + 1 exists
          const uint32_t ds = (w >> (8 * k + kFlagStepShift)) & kFlagStepMany;   // steps to the run's next turn; kFlagStepMany: more than fit
          if (ds < kFlagStepMany) T.kap[k] = s_kap[ds];
          else many |= 1u << k;
        }
      }
      while (many) {                                  // rare, and a hundred instructions each
        const int k = __ffs(static_cast<int>(many)) - 1;
        const int64_t p = p0 + k;
        const float kap = powf(P.gamma_turn, static_cast<float>(P.turn_step[P.tok_turn[p + 1]] - P.turn_step[P.tok_turn[p]]));
#pragma unroll
        for (int j = 0; j < kIpt; ++j) T.kap[j] = j == k ? kap : T.kap[j];
        many &= many - 1;
      }
    }
  }
  return T;
}
// What a run of plain tokens does not need to look at is the whole of its wavefront's: `plain` is the same in every lane.
// fold of the four tokens, right to left
template <bool HV, bool DECAY>
__device__ __forceinline__ Aff fold_four(const ScanParams& P, const Four& T, bool plain) {
  const float gl = P.gl;
  Aff m = aff_identity();
  if (plain) {
    float c = T.r[kIpt - 1] - T.v[kIpt - 1];
#pragma unroll
    for (int k = kIpt - 2; k >= 0; --k) c = fmaf(gl, c, HV ? fmaf(P.gamma, T.v[k + 1], T.r[k] - T.v[k]) : T.r[k]);
    m.a = P.gl4;
    m.b = HV ? P.gl3g : 0.f;
    m.c = c;
    m.e = 0.f;
    m.f = T.v[0];
    return m;
  }
#pragma unroll
  for (int k = kIpt - 1; k >= 0; --k) {
    const bool end = has(T.w, k, P.seg_bit), scored = has(T.w, k, kFlagMask);
    if constexpr (DECAY) { m.a *= T.kap[k]; m.b *= T.kap[k]; m.c *= T.kap[k]; m.e *= T.kap[k]; m.f *= T.kap[k]; }
    m.a = end ? 0.f : m.a;
    m.c = end ? 0.f : m.c;
    if constexpr (HV) {
      m.b = end ? 0.f : m.b;
      m.e = end ? 0.f : m.e;
      m.f = end ? 0.f : m.f;
    }
    const float d = HV ? T.r[k] - T.v[k] : T.r[k];
    m.c = scored ? fmaf(gl, m.c, HV ? fmaf(P.gamma, m.f, d) : d) : m.c;
    m.a = scored ? gl * m.a : m.a;
    if constexpr (HV) {
      m.b = scored ? fmaf(gl, m.b, P.gamma * m.e) : m.b;
      m.e = scored ? 0.f : m.e;
      m.f = scored ? T.v[k] : m.f;
    }
  }
  return m;
}

// One walk over the tiles of a range, right to left, thread 0 at a tile's right end.  REPLAY = false: fold only, returns the range's map in
// *total.  REPLAY = true: starts from the state (*G_io, *NV_io), writes advantages and returns, leaves the state at the
// range's left edge in (*G_io, *NV_io) (valid in the last thread).
// Bound by memory: 25 million tokens without values 66 -> 51 us (6.4 TB/s), of them with values and step discounts 97 -> 75; 42 million in runs of
// 10 240 with both 180 -> 172 behind the routing call, which leaves 250 MB of stores behind in the cache, on its own 170 -> 124
// (5.8 TB/s).  Before, every token's flags, place in the range and map were looked at by branches, the maps moved by shuffles, and
// a tile waited for the stores of the one before it; what a wavefront executes for its 256 tokens took longer than their 17 bytes.
// With PAST the values are read and both outputs stored past the caches (kPastTokens), which hold the rewards and flags that routing has left.
template <bool HV, bool DECAY, bool REPLAY, bool PAST>
__device__ __forceinline__ void walk_range(const ScanParams& P, const Range& R, float* __restrict__ adv, float* __restrict__ ret,
                                           Aff (*s_w)[kThreads / kWave], float (*s_carry)[2], const float* s_kap, float* G_io, float* NV_io, Aff* total) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  constexpr int nwave = kThreads / kWave;
  const float gl = P.gl;
  const int64_t t_hi = (R.end - 1) / kTile, t_lo = R.start / kTile;
  const int at = (kThreads - 1 - tid) * kIpt;
  Aff range_map = aff_identity();
  if (REPLAY && tid == 0) { s_carry[0][0] = *G_io; s_carry[0][1] = *NV_io; }
  int par = 0;
  float G = 0.f, NV = 0.f;
  // A tile in front of the range's last; one past its first is not read.  Always the same number of loads: what is waited for is known.
  auto fetch = [&](int64_t tile, Raw& x) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const int64_t t = tile < t_lo ? t_lo : tile;
    const int n = tile < t_lo ? 0 : kTile;            // tokens that can be read
    auto rsrc = [&](const void* p, int bytes) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000); };
    constexpr int kPolicy = REPLAY && PAST ? 2 : 0;   // 2: past the caches
    x.r4 = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rsrc(P.reward + t * kTile, n * 4), at * 4, 0, 0));
    x.v4 = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (HV) x.v4 = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rsrc(P.value + t * kTile, n * 4), at * 4, 0, kPolicy));
    x.w = __builtin_amdgcn_raw_buffer_load_b32(rsrc(P.flags + t * kTile, n), at, 0, 0);
  };
  auto step = [&](int64_t tile, const Raw& x, auto whole) {   // whole: all of the tile's tokens belong to the range
    constexpr bool kWhole = decltype(whole)::value;
    const int64_t p0 = tile * kTile + at;
    const uint32_t own = kWhole ? ~0u : own_bytes(R, p0), w = x.w & own;
    const bool plain = __all(w == kPlainFour);
    const Four T = four_tokens<DECAY>(P, p0, x, w, s_kap);
    Aff m = fold_four<HV, DECAY>(P, T, plain);
    wave_prefix<HV>(m);
    if (lane == kWave - 1) s_w[par][wave] = m;
    m = lane_below<HV>(m);
    __syncthreads();                                  // the one barrier of a tile
    if constexpr (!REPLAY) {
#pragma unroll
      for (int q = 0; q < nwave; ++q) range_map = then<HV>(range_map, s_w[par][q]);   // what lies further right acts first
    } else {
      Aff right = aff_identity();                   // the tile's own tokens first and the state last: one rounding at its size
#pragma unroll
      for (int q = 0; q < nwave - 1; ++q)
        if (q < wave) right = then<HV>(right, s_w[par][q]);
      m = then<HV>(right, m);
      const float g_in = s_carry[par][0], nv_in = HV ? s_carry[par][1] : 0.f;
      G = HV ? fmaf(m.a, g_in, fmaf(m.b, nv_in, m.c)) : fmaf(m.a, g_in, m.c);
      NV = HV ? fmaf(m.e, nv_in, m.f) : 0.f;
      float a[kIpt], b[kIpt];
      if (plain) {
#pragma unroll
        for (int k = kIpt - 1; k >= 0; --k) {
          G = fmaf(gl, G, HV ? fmaf(P.gamma, NV, T.r[k] - T.v[k]) : T.r[k]);
          NV = T.v[k];
          a[k] = G;
          b[k] = HV ? G + NV : G;
        }
      } else {
#pragma unroll
        for (int k = kIpt - 1; k >= 0; --k) {
          const bool end = has(w, k, P.seg_bit), scored = has(w, k, kFlagMask);
          if constexpr (DECAY) { G *= T.kap[k]; NV *= T.kap[k]; }
          G = end ? 0.f : G;
          if constexpr (HV) NV = end ? 0.f : NV;
          const float g = fmaf(gl, G, HV ? fmaf(P.gamma, NV, T.r[k] - T.v[k]) : T.r[k]);
          G = scored ? g : G;
          if constexpr (HV) NV = scored ? T.v[k] : NV;
          a[k] = scored ? g : 0.f;
          b[k] = scored ? (HV ? g + T.v[k] : g) : 0.f;
        }
      }
      if (tid == kThreads - 1) { s_carry[par ^ 1][0] = G; s_carry[par ^ 1][1] = NV; }   // state at the tile's left edge
      if (kWhole || own == ~0u) {
        const float4 a4 = make_float4(a[0], a[1], a[2], a[3]), b4 = make_float4(b[0], b[1], b[2], b[3]);
        if (PAST) {
          store_stream(adv + p0, a4);
          store_stream(ret + p0, b4);
        } else {
          *reinterpret_cast<float4*>(adv + p0) = a4;
          *reinterpret_cast<float4*>(ret + p0) = b4;
        }
      } else {
#pragma unroll
        for (int k = 0; k < kIpt; ++k)
          if (has(own, k, 1u)) { adv[p0 + k] = a[k]; ret[p0 + k] = b[k]; }
      }
    }
    par ^= 1;
  };
  using Whole = std::true_type;
  using Part = std::false_type;
  Raw x, even, odd;
  load_four<HV, REPLAY && PAST>(P, R, t_hi * kTile + at, x);
  fetch(t_hi - 1, even);
  fetch(t_hi - 2, odd);
  step(t_hi, x, Part());
  int64_t tile = t_hi - 1;
  const int64_t t_in = (R.start + kTile - 1) / kTile;   // first whole tile
  __builtin_amdgcn_s_waitcnt(0x0F70);                 // vmcnt(0): from here on it is known what is under way in the loop
  // (moved by instructions of its own, so that the next loads go to the registers that the last ones came to: the compiler would leave the
  // values there and move the new ones at the end of a turn, for which it waits)
  auto take = [&](const Raw& from) {
    auto move = [](float& to, float v) { asm volatile("v_mov_b32 %0, %1" : "=v"(to) : "v"(v) : "memory"); };
    move(x.r4.x, from.r4.x); move(x.r4.y, from.r4.y); move(x.r4.z, from.r4.z); move(x.r4.w, from.r4.w);
    if constexpr (HV) { move(x.v4.x, from.v4.x); move(x.v4.y, from.v4.y); move(x.v4.z, from.v4.z); move(x.v4.w, from.v4.w); }
    asm volatile("v_mov_b32 %0, %1" : "=v"(x.w) : "v"(from.w) : "memory");
  };
  for (; tile > t_in; tile -= 2) {
    take(even);
    fetch(tile - 2, even);
    step(tile, x, Whole());
    take(odd);
    fetch(tile - 3, odd);
    step(tile - 1, x, Whole());
  }
#pragma unroll 1
  for (; tile >= t_lo; --tile) {
    step(tile, even, Part());
    even = odd;
  }
  if constexpr (REPLAY) { *G_io = G; *NV_io = NV; } else { *total = range_map; }
}

// The map of the tokens R, which end a segment, for a workgroup that needs the state on their left: every wavefront folds a quarter of
// them, 1024 at a time, sixteen to a lane, and needs a barrier only at the end.  Every thread gets the map.  (Four to a lane make four
// times as many compositions across lanes: one segment of 65 536 tokens with values 59 us, 70 with step discounts.)
template <bool HV, bool DECAY>
__device__ __forceinline__ Aff fold_ahead(const ScanParams& P, const Range& R, Aff* s_w, const float* s_kap) {
  constexpr int nwave = kThreads / kWave, kFours = 4, kLane = kFours * kIpt, kStep = kWave * kLane;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, at = (kWave - 1 - lane) * kLane;   // lane 0 at the right end
  const int64_t first = R.start / kStep, n = (R.end - 1) / kStep + 1 - first, per = (n + nwave - 1) / nwave;
  const int64_t lo = first + wave * per, hi = lo + per < first + n ? lo + per : first + n;
  Aff map = aff_identity();
  Raw next[kFours];
  auto load = [&](int64_t t) {
#pragma unroll
    for (int i = 0; i < kFours; ++i) load_four<HV>(P, R, t * kStep + at + i * kIpt, next[i]);
  };
  if (hi > lo) load(hi - 1);
  for (int64_t t = hi - 1; t >= lo; --t) {
    Raw x[kFours];
#pragma unroll
    for (int i = 0; i < kFours; ++i) x[i] = next[i];
    if (t > lo) load(t - 1);
    Aff acc = aff_identity();
#pragma unroll
    for (int i = kFours - 1; i >= 0; --i) {
      const int64_t p0 = t * kStep + at + i * kIpt;
      const uint32_t w = x[i].w & own_bytes(R, p0);
      acc = then<HV>(acc, fold_four<HV, DECAY>(P, four_tokens<DECAY>(P, p0, x[i], w, s_kap), __all(w == kPlainFour)));
    }
    wave_prefix<HV>(acc);
    map = then<HV>(map, acc);                       // in the last lane
  }
  if (lane == kWave - 1) s_w[wave] = map;
  __syncthreads();
  Aff total = aff_identity();
  for (int w = nwave - 1; w >= 0; --w) total = then<HV>(total, s_w[w]);
  __syncthreads();
  return total;
}

// One workgroup per range.  It finds the range's edges (one wavefront each).  Unless the range is
// empty or its right end lies inside a long segment, it scans the range: nothing comes in from the right.  What the second kernel needs is
// left for it: the edges, the range's record cleared or published.  With ALONE there is no second kernel: a workgroup whose range ends inside a
// segment reads on to the segment's end itself, for its map.
template <bool HV, bool DECAY, bool ALONE, bool PAST>
__global__ void __launch_bounds__(kThreads)
k_gae_scan(ScanParams P, float* __restrict__ adv, float* __restrict__ ret) {
  __shared__ Aff s_w[2][kThreads / kWave];
  __shared__ float s_carry[2][2];
  __shared__ int64_t s_edge[2], s_end;
  __shared__ int s_cut[2];
  __shared__ float s_kap[kKaps];
  const int tid = threadIdx.x;
  fill_kaps<DECAY>(P, s_kap);
  const uint32_t q = blockIdx.x;                                                   // from the right
  const int64_t i = static_cast<int64_t>(P.n_ranges) - 1 - q;                      // from the left
  if (tid < 2 * kWave) {
    const int which = tid / kWave;                   // wavefront 0: left edge, wavefront 1: right edge
    int cut;
    int64_t boundary;
    const int64_t edge = range_edge(P, (i + which) * P.chunk, &cut, &boundary);
    if ((tid & (kWave - 1)) == 0) {
      s_edge[which] = edge;
      s_cut[which] = cut;
      if (which == 1) s_end = boundary;
    }
  }
  __syncthreads();
  Range R;
  R.start = s_edge[0];
  R.end = s_edge[1];
  R.cut_left = s_cut[0];
  R.cut_right = s_cut[1];
  R.pad = 0;
  float G = 0.f, NV = 0.f;
  if constexpr (ALONE) {
    if (R.start >= R.end) return;                   // the same for every thread, also below
    if (R.cut_right) {
      const Range ahead{R.end, s_end, 0, 0, 0};
      const Aff m = fold_ahead<HV, DECAY>(P, ahead, s_w[0], s_kap);
      G = m.c;                                      // a constant map: a segment ends there
      NV = HV ? m.f : 0.f;
    }
  } else {
    if (tid == 0) P.ranges[q] = R;
    if (tid < kStateWords) P.range_state[static_cast<size_t>(q) * kStateWords + tid] = 0ull;
    if (R.start >= R.end || R.cut_right) return;
  }
  Aff unused;
  walk_range<HV, DECAY, true, PAST>(P, R, adv, ret, s_w, s_carry, s_kap, &G, &NV, &unused);
  // a range that starts inside a long segment: what it hands to the left is a constant
  if (!ALONE && R.cut_left && tid == kThreads - 1)
    publish<HV>(P.range_state + static_cast<size_t>(q) * kStateWords, Aff{0.f, 0.f, G, 0.f, HV ? NV : 0.f});
}

// The ranges whose right end lies inside a long segment; persistent workgroups.
template <bool HV, bool DECAY, bool PAST>
__global__ void __launch_bounds__(kThreads)
k_gae_scan_cut(ScanParams P, float* __restrict__ adv, float* __restrict__ ret) {
  __shared__ Aff s_w[2][kThreads / kWave];
  __shared__ float s_carry[2][2];
  __shared__ float s_in[2];
  const int tid = threadIdx.x;
  // does any of this workgroup's ranges need it?  every thread looks at some of them, all loads at once
  int mine = 0;
  for (uint64_t q = blockIdx.x + static_cast<uint64_t>(tid) * gridDim.x; q < P.n_ranges; q += static_cast<uint64_t>(kThreads) * gridDim.x)
    mine |= P.ranges[q].cut_right;
  __shared__ float s_kap[kKaps];
  fill_kaps<DECAY>(P, s_kap);
  if (!__syncthreads_or(mine)) return;
  for (uint32_t q = blockIdx.x; q < P.n_ranges; q += gridDim.x) {
    const Range R = P.ranges[q];
    if (R.start >= R.end || !R.cut_right) continue; // the same for every thread
    // the range's own map first (published if the left end is cut too), then the state that the ranges to its right
    // hand over, then the replay
    float G = 0.f, NV = 0.f;
    Aff range_map;
    walk_range<HV, DECAY, false, PAST>(P, R, adv, ret, s_w, s_carry, s_kap, &G, &NV, &range_map);
    if (R.cut_left && tid == 0) publish<HV>(P.range_state + static_cast<size_t>(q) * kStateWords, range_map);
    if (tid < kWave) {
      float g_in, nv_in;
      look_back<HV>(P, q, &g_in, &nv_in);
      if (tid == 0) { s_in[0] = g_in; s_in[1] = nv_in; }
    }
    __syncthreads();                                // also: the LDS of the first walk is free
    G = s_in[0];
    NV = s_in[1];
    Aff unused;
    walk_range<HV, DECAY, true, PAST>(P, R, adv, ret, s_w, s_carry, s_kap, &G, &NV, &unused);
    __syncthreads();
  }
}

inline int64_t scan_ranges(int64_t n_tokens, int64_t chunk) { return (n_tokens + chunk - 1) / chunk; }
inline size_t scan_bytes(int64_t n_tokens, int64_t chunk) {   // ranges, records
  const size_t n = static_cast<size_t>(n_tokens > 0 ? scan_ranges(n_tokens, chunk) : 1);
  return align_up(n * sizeof(Range)) + align_up(n * kStateWords * sizeof(unsigned long long));
}

}  // namespace
}  // namespace umas

using namespace umas;

extern "C" size_t umas_advantages_workspace_bytes(int64_t n_tokens) {
  if (n_tokens < 0) return 0;
  return scan_bytes(n_tokens, chunk_tokens(n_tokens));
}

extern "C" umas_status umas_advantages(const umas_streams* s, int64_t n_tokens, int32_t n_turns,
                                       const float* value, float gamma, float lam, float gamma_turn,
                                       int32_t seg_mode, float* adv, float* ret, void* workspace,
                                       size_t workspace_bytes, void* hip_stream) {
  UMAS_REQUIRE(s, UMAS_EINVAL, "streams is NULL");
  UMAS_REQUIRE(n_tokens >= 0 && n_turns >= 0, UMAS_EINVAL, "negative size");
  UMAS_REQUIRE(seg_mode == UMAS_SEG_TURN || seg_mode == UMAS_SEG_TRAJ, UMAS_EINVAL, "seg_mode=%d is neither TURN nor TRAJ",
               seg_mode);
  UMAS_REQUIRE(s->tok_reward && s->tok_flags && s->turn_seg_off && s->traj_seg_off && s->tok_turn && s->turn_step,
               UMAS_EINVAL, "streams lacks tok_reward, tok_flags, turn_seg_off, traj_seg_off, tok_turn or turn_step");
  UMAS_REQUIRE((adv && ret) || n_tokens == 0, UMAS_EINVAL, "adv and ret must not be NULL");
  UMAS_REQUIRE(gamma == gamma && lam == lam && gamma_turn == gamma_turn, UMAS_EINVAL, "gamma, lam, gamma_turn must be numbers");
  UMAS_REQUIRE(reinterpret_cast<uintptr_t>(s->tok_reward) % 16 == 0 && reinterpret_cast<uintptr_t>(value) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(s->tok_flags) % 16 == 0 && reinterpret_cast<uintptr_t>(adv) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(ret) % 16 == 0,
               UMAS_EINVAL, "tok_reward, tok_flags, value, adv and ret must be 16-byte aligned");
  constexpr int64_t kMaxChunk = static_cast<int64_t>(kChunkTiles) * kTile;
  UMAS_REQUIRE(scan_ranges(n_tokens, kMaxChunk) < (1LL << 31), UMAS_ESHAPE, "at most 2^43 tokens");
  // a workspace for ranges of eight tiles will do: then they are no finer than it holds
  const size_t need = scan_bytes(n_tokens, kMaxChunk);
  UMAS_REQUIRE(workspace && reinterpret_cast<uintptr_t>(workspace) % kAlign == 0 && workspace_bytes >= need, UMAS_EWORKSPACE,
               "workspace must be 256-byte aligned and hold %zu bytes (got %zu)", need, workspace_bytes);
  if (n_tokens == 0) return UMAS_OK;
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  prof_mark(st);
  ScanParams P;
  P.n_tokens = n_tokens;
  P.chunk = chunk_tokens(n_tokens);
  while (scan_bytes(n_tokens, P.chunk) > workspace_bytes) P.chunk += kTile;
  const int64_t n_ranges = scan_ranges(n_tokens, P.chunk);
  P.n_ranges = static_cast<uint32_t>(n_ranges);
  Range* ranges = static_cast<Range*>(workspace);
  P.ranges = ranges;
  P.range_state = reinterpret_cast<unsigned long long*>(static_cast<char*>(workspace) + align_up(static_cast<size_t>(n_ranges) * sizeof(Range)));
  P.seg_off = seg_mode == UMAS_SEG_TURN ? s->turn_seg_off : s->traj_seg_off;
  P.n_seg_entries = n_turns;
  P.flags = s->tok_flags;
  P.reward = s->tok_reward;
  P.value = value;
  P.tok_turn = s->tok_turn;
  P.turn_step = s->turn_step;
  P.seg_bit = seg_mode == UMAS_SEG_TURN ? kFlagTurnEnd : kFlagRunEnd;
  P.gamma = gamma;
  P.lam = lam;
  P.gamma_turn = gamma_turn;
  P.gl = gamma * lam;
  const double gl = P.gl;
  P.gl4 = static_cast<float>(gl * gl * gl * gl);
  P.gl3g = static_cast<float>(gl * gl * gl * gamma);
  const bool decay = seg_mode == UMAS_SEG_TRAJ && gamma_turn != 1.0f;
  // (alone, workgroups read tokens that are others' to write the outputs of: not where these lie over the inputs)
  auto apart = [&](const float* out, const float* in) { return !in || out + n_tokens <= in || in + n_tokens <= out; };
  const bool alone = n_tokens <= alone_tokens(decay) && apart(adv, s->tok_reward) && apart(adv, value) && apart(ret, s->tok_reward) && apart(ret, value);
  const bool past = !alone && n_tokens >= kPastTokens;
  auto pick = [&](auto al, auto pa) -> void (*)(ScanParams, float*, float*) {
    constexpr bool A = decltype(al)::value, S = decltype(pa)::value;
    return value ? (decay ? k_gae_scan<true, true, A, S> : k_gae_scan<true, false, A, S>) : (decay ? k_gae_scan<false, true, A, S> : k_gae_scan<false, false, A, S>);
  };
  using Yes = std::true_type;
  using No = std::false_type;
  void (*kernel)(ScanParams, float*, float*) = alone ? pick(Yes(), No()) : past ? pick(No(), Yes()) : pick(No(), No());
  hipLaunchKernelGGL(kernel, dim3(P.n_ranges), dim3(kThreads), 0, st, P, adv, ret);
  UMAS_LAUNCHED("k_gae_scan");
  if (alone) return UMAS_OK;
  // The ranges cut inside long segments: persistent workgroups that wait for each other's maps.  At most one workgroup
  // per compute unit, far fewer than the device holds at once: whatever else is running, all of them get to run
  // together, so no workgroup waits for one that cannot start.
  auto pick_cut = [&](auto pa) -> void (*)(ScanParams, float*, float*) {
    constexpr bool S = decltype(pa)::value;
    return value ? (decay ? k_gae_scan_cut<true, true, S> : k_gae_scan_cut<true, false, S>) : (decay ? k_gae_scan_cut<false, true, S> : k_gae_scan_cut<false, false, S>);
  };
  void (*kernel_cut)(ScanParams, float*, float*) = past ? pick_cut(Yes()) : pick_cut(No());
  int dev = 0, n_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
    n_cu = 64;
  const unsigned nblk = static_cast<unsigned>(n_ranges < n_cu ? n_ranges : n_cu);
  hipLaunchKernelGGL(kernel_cut, dim3(nblk), dim3(kThreads), 0, st, P, adv, ret);
  UMAS_LAUNCHED("k_gae_scan_cut");
  return UMAS_OK;
}
