// Reward composition, group normalisation, routing through phi and reward placement.
//
// The thin graph arrives as host arrays (the controller's view: role ids, routing ids,
// reward metadata); it is validated on the host, staged to the device and every step after
// that runs in kernels: per-turn reward r_v = lam_node r_node + lam_turn r_turn + lam_traj
// r_traj (Section "Agent-Specific Reward Interface"), the stable partition of turns by
// phi(role) into model-local streams (Sections "Agent--LLM Mapping", "Model-Local Buffers")
// and the alignment of each turn's reward with its token sequence (paragraph "Batch
// construction").
//
// Small graphs take one launch (k_route_small).  The others take a copy of the thin arrays and three kernels (four with
// normalisation groups).  k_turn_plan does everything that is per turn: one thread walks
// one trajectory's turns (a trajectory's turns are consecutive, and everything a turn needs from its neighbours -
// whether it opens or closes the trajectory's run inside its model's stream, how many steps lie between it and the
// run's next turn - lies inside its trajectory), blocks of 256 trajectories publish their per-model totals and read
// everybody else's to place themselves.  k_tokens writes everything that is per token in one pass over the streams
// (22 bytes per token, the mask read once); k_rowsel compacts the positions of the scored tokens (the gathered mask
// read again, 4 bytes per scored token written).
#include <algorithm>
#include <vector>

#include "umas_common.h"

namespace umas {

namespace {

constexpr int kPlanThreads = 256;  // trajectories per chunk of the plan kernel
constexpr int kPlanPerCu = 2;      // its workgroups per compute unit at most (one with more than two models): a fraction of what
                                   // the device holds at once, so all of them are resident, also next to a second call's
constexpr int kCnt = 3;            // per model and chunk: turns, tokens, trajectory runs
constexpr int kPlanWords = UMAS_MAX_MODELS * kCnt;
constexpr int kTokThreads = 256;
constexpr int kTokPerThread = 4;   // consecutive tokens of one thread in one round
constexpr int kTokRounds = 4;      // rounds of a block, kTokThreads * kTokPerThread tokens apart
constexpr int kTokRound = kTokThreads * kTokPerThread;
constexpr int kTokBlock = kTokRound * kTokRounds;
constexpr unsigned long long kMark = 1ull << 63;          // ready mark of a published count

// What the token kernel needs to know about one turn segment of a model-local stream.
struct __attribute__((aligned(16))) SegMeta {
  int64_t src;         // global index of the segment's first token
  int32_t turn;
  int32_t role;
  float rho;           // composed reward of the turn
  int32_t end_flags;   // flag bits of the segment's last token besides the mask bit
  int64_t pad;
};
static_assert(sizeof(SegMeta) == 32, "two 16-byte loads");

struct RouteWs {
  // the thin arrays, staged from the host in one copy (everything up to traj_norm)
  int32_t* role_to_model;
  int32_t* traj_turn_off;
  uint8_t* turn_role;
  uint32_t* tok_off32;             // token offsets of the turns: 32 bits where all tokens are fewer than 2^32, ...
  int64_t* tok_off64;              // ... else 64
  int32_t* group_off;
  int32_t* group_members;          // not there where groups are in order: member i is trajectory i
  float* role_reward;
  float* turn_reward;
  float* traj_reward;
  float* weights;       // [3 * n_roles]: role, turn, traj
  unsigned long long* plan_part;   // [n_chunks][kPlanWords] per-chunk totals of the plan kernel; zeros come with the staged copy
  // written on the device
  float* traj_norm;     // [n_traj]
  SegMeta* seg_meta;    // [n_turns] per segment slot
  int32_t* blk_first;   // [nblk_tok] segment that holds the first token of each token block
  unsigned long long* tok_count;   // [nblk_tok + groups] scored tokens of the token kernel's blocks, then of its groups of blocks
};

// Blocks of the token kernel are grouped 2^shift to a group, about the square root of their number and at least 64.
inline int group_shift(size_t nbk) {
  int sh = 6;
  while ((size_t{1} << (2 * sh)) < nbk) ++sh;
  return sh;
}
inline int plan_chunks(int n_traj) { return static_cast<int>(cdiv(n_traj > 0 ? n_traj : 1, kPlanThreads)); }

// The thin arrays that a call has; what it has not takes no room and does not go over the bus (36 GB/s: 98 304 turns in 32 768 trajectories with one
// reward each 2.5 MB in 47 us; without the arrays that are not there, roles in a byte and offsets in 32 bits 0.8 MB in
// 20).
struct Thin {
  bool role_reward = true, turn_reward = true, traj_reward = true, weights = true, wide_offsets = true;
  int groups = -1;                 // -1: as many as trajectories
  bool members = true;
};
size_t carve(Carver& c, RouteWs& w, int n_roles, int n_traj, int n_turns, int64_t n_tokens, const Thin& has = Thin()) {
  const size_t nbk = cdiv(n_tokens > 0 ? n_tokens : 1, kTokBlock), offs = static_cast<size_t>(n_turns) + 1;
  w.role_to_model = c.take<int32_t>(n_roles);
  w.traj_turn_off = c.take<int32_t>(n_traj + 1);
  w.turn_role = c.take<uint8_t>(n_turns);
  w.tok_off32 = c.take<uint32_t>(has.wide_offsets ? 0 : offs);
  w.tok_off64 = c.take<int64_t>(has.wide_offsets ? offs : 0);
  w.group_off = c.take<int32_t>(has.groups < 0 ? n_traj + 2 : has.groups > 0 ? has.groups + 1 : 0);
  w.group_members = c.take<int32_t>(has.members ? n_traj : 0);
  w.role_reward = c.take<float>(has.role_reward ? static_cast<size_t>(n_traj) * n_roles : 0);
  w.turn_reward = c.take<float>(has.turn_reward ? n_turns : 0);
  w.traj_reward = c.take<float>(has.traj_reward ? n_traj : 0);
  w.weights = c.take<float>(has.weights ? 3 * n_roles : 0);
  w.plan_part = c.take<unsigned long long>(static_cast<size_t>(plan_chunks(n_traj)) * kPlanWords);
  w.traj_norm = c.take<float>(n_traj);
  w.seg_meta = c.take<SegMeta>(n_turns);
  w.blk_first = c.take<int32_t>(nbk);
  w.tok_count = c.take<unsigned long long>(nbk + (nbk >> group_shift(nbk)) + 1);
  return c.off;
}

// ------------------------------------------------------------------ kernels

// z-score of the trajectory rewards of one group, by one wavefront, float64 statistics.  Without `members` they are a .. e - 1.
__device__ __forceinline__ void normalise_group(const float* __restrict__ R, const int32_t* __restrict__ members, int a, int e, float eps,
                                                float* __restrict__ out) {
  const int lane = threadIdx.x & (kWave - 1);
  if (e == a) return;
  double s = 0.0;
  for (int i = a + lane; i < e; i += kWave) s += static_cast<double>(R[members ? members[i] : i]);
  const double mu = wave_sum(s) / static_cast<double>(e - a);
  double q = 0.0;
  for (int i = a + lane; i < e; i += kWave) {
    const double t = static_cast<double>(R[members ? members[i] : i]) - mu;
    q += t * t;
  }
  const double sigma = sqrt(wave_sum(q) / static_cast<double>(e - a));
  for (int i = a + lane; i < e; i += kWave) {
    const int b = members ? members[i] : i;
    out[b] = static_cast<float>((static_cast<double>(R[b]) - mu) / (sigma + static_cast<double>(eps)));
  }
}
__global__ void k_group_norm(const float* __restrict__ R, const int32_t* __restrict__ group_off,
                             const int32_t* __restrict__ members, int n_groups, float eps,
                             float* __restrict__ out) {
  const int g = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  if (g < n_groups) normalise_group(R, members, group_off[g], group_off[g + 1], eps, out);
}

// ------------------------------------------------------------------ the plan: everything per turn
struct PlanArgs {
  int n_traj, n_turns, n_roles, n_models, n_chunks;
  int64_t n_tokens, n_count;          // n_count: words of tok_count to clear
  const int32_t* __restrict__ traj_turn_off;
  const uint8_t* __restrict__ turn_role;
  const int32_t* __restrict__ role_to_model;
  const uint32_t* __restrict__ tok_off32;  // one of the two
  const int64_t* __restrict__ tok_off64;
  const float* __restrict__ role_reward;   // NULL level = 0
  const float* __restrict__ turn_reward;
  const float* __restrict__ traj_reward;   // already normalised when groups are given
  const float* __restrict__ w_role;        // NULL weight = 1
  const float* __restrict__ w_turn;
  const float* __restrict__ w_traj;
  unsigned long long* __restrict__ plan_part;
  SegMeta* __restrict__ seg_meta;
  int32_t* __restrict__ blk_first;
  unsigned long long* __restrict__ tok_count;
  // outputs
  int64_t* __restrict__ model_tok_off;
  int32_t* __restrict__ model_turn_off;
  int32_t* __restrict__ model_trajrun_off;
  int64_t* __restrict__ model_rowsel_off;
  int64_t* __restrict__ turn_seg_off;
  int32_t* __restrict__ seg_turn;
  int64_t* __restrict__ traj_seg_off;
  float* __restrict__ turn_scalar;
  int32_t* __restrict__ turn_step;
  __device__ __forceinline__ int64_t tok_off(int u) const { return tok_off32 ? static_cast<int64_t>(tok_off32[u]) : tok_off64[u]; }
};

// v[k] of a small per-model array with a run-time k, without indexing registers dynamically
template <typename T, int KM>
__device__ __forceinline__ T pick(const T (&v)[KM], int k) {
  T r = v[0];
#pragma unroll
  for (int i = 1; i < KM; ++i) r = k == i ? v[i] : r;
  return r;
}
template <typename T, int KM>
__device__ __forceinline__ void bump(T (&v)[KM], int k, T by) {
#pragma unroll
  for (int i = 0; i < KM; ++i) v[i] += k == i ? by : T(0);
}

// Per-model counts of one trajectory: turns, tokens, and whether the model has a run in it.
template <int KM>
struct TrajCounts {
  int64_t cnt[KM], tok[KM];
  uint32_t seen;
};
template <int KM, class Phi>
__device__ __forceinline__ void traj_counts(const PlanArgs& A, Phi phi, int b, TrajCounts<KM>& c) {
#pragma unroll
  for (int k = 0; k < KM; ++k) { c.cnt[k] = 0; c.tok[k] = 0; }
  c.seen = 0;
  if (b >= A.n_traj) return;
  const int t0 = A.traj_turn_off[b], t1 = A.traj_turn_off[b + 1];
  int64_t g0 = A.tok_off(t0);
  for (int u = t0; u < t1; ++u) {
    const int m = phi[A.turn_role[u]];
    const int64_t g1 = A.tok_off(u + 1);
    bump(c.cnt, m, int64_t{1});
    bump(c.tok, m, g1 - g0);
    c.seen |= 1u << m;
    g0 = g1;
  }
}

// One walk over the turns of trajectory b, whose first turn, token and run in every stream go to slot_at, tok_at and run_at: slots,
// offsets, runs, composed rewards and the record of every segment, which go to `sink`.  What a segment's last token says about its
// end - bit 1: last token of its turn; bit 2: also the last token of the trajectory's run (no later turn of the trajectory with
// tokens in this stream); bits 3-7: else the number of steps to the run's next turn with tokens (31 = more than 30: look it
// up) - is known only when that next turn comes by: the record is written as a run's end and its flags are written again then.
template <int KM, class Phi, class Sink>
__device__ __forceinline__ void walk_turns(const PlanArgs& A, Phi phi, int b, int64_t (&slot_at)[KM], int64_t (&tok_at)[KM],
                                           const int64_t (&run_at)[KM], Sink sink) {
  const int t0 = A.traj_turn_off[b], t1 = A.traj_turn_off[b + 1];
  const float rj = A.traj_reward ? A.traj_reward[b] : 0.0f;
  uint32_t seen = 0;
  int last_slot[KM], last_step[KM];   // the model's latest turn with tokens in this trajectory
#pragma unroll
  for (int k = 0; k < KM; ++k) { last_slot[k] = -1; last_step[k] = 0; }
  int64_t g0 = A.tok_off(t0);
  for (int u = t0; u < t1; ++u) {
    const int v = A.turn_role[u];
    const int m = phi[v];
    const int64_t g1 = A.tok_off(u + 1), len = g1 - g0;
    const int64_t slot = pick(slot_at, m), off = pick(tok_at, m);
    const int step = u - t0 + 1;
    bump(slot_at, m, int64_t{1});
    bump(tok_at, m, len);
    if (!((seen >> m) & 1u)) {                       // the trajectory's one run in stream m starts here
      sink.run(pick(run_at, m), off);
      seen |= 1u << m;
    }
    const float rr = A.role_reward ? A.role_reward[static_cast<size_t>(b) * A.n_roles + v] : 0.0f;
    const float rt = A.turn_reward ? A.turn_reward[u] : 0.0f;
    const float wr = A.w_role ? A.w_role[v] : 1.0f;
    const float wt = A.w_turn ? A.w_turn[v] : 1.0f;
    const float wj = A.w_traj ? A.w_traj[v] : 1.0f;
    // (node + turn) + traj with every product and sum rounded on its own: contraction into fused
    // multiply-adds is switched off for this expression so that the result is reproducible bit for bit
    float rho;
    {
#pragma clang fp contract(off)
      const float pr = wr * rr, pt = wt * rt, pj = wj * rj;
      const float s1 = pr + pt;
      rho = s1 + pj;
    }
    SegMeta M;
    M.src = g0;
    M.turn = u;
    M.role = v;
    M.rho = rho;
    M.end_flags = 2 | 4;
    M.pad = 0;
    sink.turn(slot, off, len, step, M);
    if (len > 0) {
      const int prev = pick(last_slot, m);
      if (prev >= 0) {
        const int ds = step - pick(last_step, m);
        sink.end_flags(prev, 2 | ((ds < 31 ? ds : 31) << 3));
      }
#pragma unroll
      for (int k = 0; k < KM; ++k) {
        last_slot[k] = m == k ? static_cast<int>(slot) : last_slot[k];
        last_step[k] = m == k ? step : last_step[k];
      }
    }
    g0 = g1;
  }
}
// What the plan says of a turn, in the outputs ...
__device__ __forceinline__ void publish_turn(const PlanArgs& A, int64_t slot, int64_t off, int step, const SegMeta& M) {
  A.seg_turn[slot] = M.turn;
  A.turn_seg_off[slot] = off;
  A.turn_scalar[M.turn] = M.rho;
  A.turn_step[M.turn] = step;
}
// ... and, for the token kernel, in the workspace: the records, the first segment of every token block.
struct PlanSink {
  const PlanArgs& A;
  __device__ __forceinline__ void run(int64_t r, int64_t off) const { A.traj_seg_off[r] = off; }
  __device__ __forceinline__ void turn(int64_t slot, int64_t off, int64_t len, int step, const SegMeta& M) const {
    publish_turn(A, slot, off, step, M);
    for (int64_t blk = (off + kTokBlock - 1) / kTokBlock; blk * kTokBlock < off + len; ++blk) A.blk_first[blk] = static_cast<int32_t>(slot);
    A.seg_meta[slot] = M;
  }
  __device__ __forceinline__ void end_flags(int slot, int32_t f) const { A.seg_meta[slot].end_flags = f; }
};

// KM: the smallest of 1, 2, 4, 8 that is at least the number of models (per-model state lives in registers).
template <int KM>
__global__ void __launch_bounds__(kPlanThreads, 2)
k_turn_plan(PlanArgs A) {
  __shared__ int64_t smem[32];
  __shared__ long long s_res[2][kPlanWords];         // [total | before this chunk][model, counter]
  __shared__ uint8_t s_phi[UMAS_MAX_ROLES];          // role -> model
  const int tid = threadIdx.x;
  const int K = A.n_models;
  if (tid < A.n_roles) s_phi[tid] = static_cast<uint8_t>(A.role_to_model[tid]);
  __syncthreads();

  // 1. every chunk of this workgroup: per-model totals of its 256 trajectories, published at once.  The counts of the
  // workgroup's first chunk (its only one unless there are more chunks than workgroups) stay in registers for step 2.
  TrajCounts<KM> first;
  for (int c = blockIdx.x; c < A.n_chunks; c += gridDim.x) {
    TrajCounts<KM> tc;
    traj_counts(A, s_phi, c * kPlanThreads + tid, tc);
    if (c == static_cast<int>(blockIdx.x)) first = tc;
    for (int k = 0; k < K; ++k) {
      const int64_t v[kCnt] = {pick(tc.cnt, k), pick(tc.tok, k), static_cast<int64_t>((tc.seen >> k) & 1u)};
#pragma unroll
      for (int j = 0; j < kCnt; ++j) {
        const int64_t total = block_sum<int64_t>(v[j], smem);
        if (tid == 0)
          __hip_atomic_store(A.plan_part + static_cast<size_t>(c) * kPlanWords + k * kCnt + j,
                             kMark | static_cast<unsigned long long>(total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }

  // housekeeping that waits for nobody: the token kernel's counts start at zero; with no tokens or no turns it does not run
  {
    const int64_t gtid = static_cast<int64_t>(blockIdx.x) * kPlanThreads + tid, gsize = static_cast<int64_t>(gridDim.x) * kPlanThreads;
    for (int64_t i = gtid; i < A.n_count; i += gsize) A.tok_count[i] = 0ull;
    if (gtid <= K) A.model_rowsel_off[gtid] = 0;
  }

  // 2. every chunk again: where its trajectories' turns go
  for (int c = blockIdx.x; c < A.n_chunks; c += gridDim.x) {
    // totals over all chunks and over the chunks before this one, for every (model, counter): thread t takes the
    // chunks t, t + 256, ..., all words of a chunk in flight together; a word is taken when its ready mark is set
    if (tid < 2 * kPlanWords) (&s_res[0][0])[tid] = 0;
    __syncthreads();
    {
      constexpr int kW = KM * kCnt;
      long long all[kW], before[kW];
#pragma unroll
      for (int j = 0; j < kW; ++j) { all[j] = 0; before[j] = 0; }
      for (int cc = tid; cc < A.n_chunks; cc += kPlanThreads) {
        unsigned long long* const src = A.plan_part + static_cast<size_t>(cc) * kPlanWords;
        unsigned long long w[kW];
#pragma unroll
        for (int j = 0; j < kW; ++j) w[j] = j < K * kCnt ? __hip_atomic_load(src + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kMark;
#pragma unroll
        for (int j = 0; j < kW; ++j) {
          while (!(w[j] & kMark)) {
            __builtin_amdgcn_s_sleep(2);
            w[j] = __hip_atomic_load(src + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          const long long v = static_cast<long long>(w[j] & ~kMark);
          all[j] += v;
          before[j] += cc < c ? v : 0;
        }
      }
#pragma unroll
      for (int j = 0; j < kW; ++j) {
        const long long ta = wave_sum(all[j]), tb = wave_sum(before[j]);
        if ((tid & (kWave - 1)) == 0) {
          atomicAdd(reinterpret_cast<unsigned long long*>(&s_res[0][j]), static_cast<unsigned long long>(ta));
          atomicAdd(reinterpret_cast<unsigned long long*>(&s_res[1][j]), static_cast<unsigned long long>(tb));
        }
      }
    }
    __syncthreads();
    // first slot, token offset and run of every stream: streams lie one after the other
    int64_t slot_at[KM], tok_at[KM], run_at[KM];
    {
      int64_t bs = 0, bt = 0, br = 0;
#pragma unroll
      for (int k = 0; k < KM; ++k) {
        slot_at[k] = bs; tok_at[k] = bt; run_at[k] = br;
        if (k < K) { bs += s_res[0][k * kCnt + 0]; bt += s_res[0][k * kCnt + 1]; br += s_res[0][k * kCnt + 2]; }
      }
      if (c == 0 && tid == 0) {
        for (int k = 0; k <= K; ++k) {
          A.model_turn_off[k] = static_cast<int32_t>(k < K ? pick(slot_at, k) : bs);
          A.model_tok_off[k] = k < K ? pick(tok_at, k) : bt;
          A.model_trajrun_off[k] = static_cast<int32_t>(k < K ? pick(run_at, k) : br);
        }
        A.turn_seg_off[A.n_turns] = A.n_tokens;
      }
      // entries of traj_seg_off past the runs read n_tokens
      const int64_t gtid = static_cast<int64_t>(c) * kPlanThreads + tid, gsize = static_cast<int64_t>(A.n_chunks) * kPlanThreads;
      for (int64_t i = br + gtid; i <= A.n_turns; i += gsize) A.traj_seg_off[i] = A.n_tokens;
#pragma unroll
      for (int k = 0; k < KM; ++k)
        if (k < K) { slot_at[k] += s_res[1][k * kCnt + 0]; tok_at[k] += s_res[1][k * kCnt + 1]; run_at[k] += s_res[1][k * kCnt + 2]; }
    }
    // ... plus what the trajectories before this thread's one inside the chunk hold
    const int b = c * kPlanThreads + tid;
    {
      TrajCounts<KM> tc;
      if (c == static_cast<int>(blockIdx.x)) tc = first;
      else traj_counts(A, s_phi, b, tc);
      for (int k = 0; k < K; ++k) {
        int64_t total;
        const int64_t e0 = block_excl_scan<int64_t>(pick(tc.cnt, k), smem, &total);
        const int64_t e1 = block_excl_scan<int64_t>(pick(tc.tok, k), smem, &total);
        const int64_t e2 = block_excl_scan<int64_t>(static_cast<int64_t>((tc.seen >> k) & 1u), smem, &total);
        bump(slot_at, k, e0);
        bump(tok_at, k, e1);
        bump(run_at, k, e2);
      }
    }
    if (b < A.n_traj) {
      walk_turns(A, s_phi, b, slot_at, tok_at, run_at, PlanSink{A});
    }
    __syncthreads();                                 // s_res is the next chunk's
  }
}

// ------------------------------------------------------------------ the tokens: everything per token
// Per token in model-local order: source index, turn, role, mask, flags, placed reward.  A block of 4096 tokens keeps
// the offsets and records of the segments that hold its tokens in LDS (up to kSegWin of them; a block of more and
// therefore very short segments takes a plain per-token path).  What a block cannot know from its own tokens is
// whether its last segment, if it goes on past the block, has another scored token further on, which decides if the
// segment's last scored token so far carries the reward: one wavefront reads ahead in the mask until it finds one or
// the segment ends.  The block also leaves its number of scored tokens for the compaction kernel, and adds it to the
// total of its group of blocks (about the square root of the number of blocks to a group).
constexpr int kSegWin = 256;
constexpr int kCompact = kTokBlock / kTokThreads;   // consecutive tokens of one thread when the scored positions are compacted
static_assert(kCompact == 16, "one 16-byte LDS read per thread");

struct TokArgs {
  int64_t n_tokens;
  int n_turns, n_models, place_mode, grp_shift;
  const int64_t* turn_seg_off;
  const SegMeta* seg_meta;
  const int32_t* blk_first;
  const uint8_t* mask_global;
  unsigned long long* blk_count;   // [blocks] scored tokens of the block
  unsigned long long* grp_count;   // [groups of 2^grp_shift blocks] scored tokens of the group, zero at the start
  int64_t* perm;
  int32_t* tok_turn;
  int32_t* tok_role;
  uint8_t* tok_mask;
  uint8_t* tok_flags;
  float* tok_reward;
};

// every non-zero byte becomes 1: (b | 0x80) - 1 keeps bit 7 exactly when b > 0, or-ed with b's own bit 7
__device__ __forceinline__ uint32_t bytes_to_01(uint32_t m4) {
  return ((((m4 | 0x80808080u) - 0x01010101u) | m4) >> 7) & 0x01010101u;
}
// mask bytes of four consecutive global tokens as one word (one load when the address allows it)
__device__ __forceinline__ uint32_t load_mask4(const uint8_t* __restrict__ mask, int64_t g0, bool base_aligned) {
  if (base_aligned && (g0 & 3) == 0) return *reinterpret_cast<const uint32_t*>(mask + g0);
  return static_cast<uint32_t>(mask[g0]) | (static_cast<uint32_t>(mask[g0 + 1]) << 8) |
         (static_cast<uint32_t>(mask[g0 + 2]) << 16) | (static_cast<uint32_t>(mask[g0 + 3]) << 24);
}
// One wavefront: does a segment, from its `skip`-th token on, hold a scored token?  (It lies at `src` and has len tokens.)
__device__ __forceinline__ bool scored_token_ahead(const TokArgs& A, int64_t src, int64_t len, int64_t skip) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t g = src + skip, n = len - skip;
  bool found = false;
  for (int64_t i0 = 0; i0 < n && !found; i0 += 8 * kWave) {   // eight bytes per lane, all in flight together
    uint32_t any = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int64_t i = i0 + lane * 8 + k;
      any |= i < n ? A.mask_global[g + i] : 0u;
    }
    found = __any(any != 0);
  }
  return found;
}

// The segments that hold a block's tokens, in LDS: offsets, the same relative to the block's first token, records, and the
// block-relative position of the segment's last scored token in this block (-1 at first).
struct SegWindow {
  const int64_t* off;
  const int32_t* loc;
  const SegMeta* meta;
  int32_t* lastv;
};
// largest j in [0, n] with loc[j] <= pl: the segment that holds the token
__device__ __forceinline__ int segment_of(const int32_t* loc, int n, int pl) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (loc[mid] <= pl) lo = mid; else hi = mid - 1;
  }
  return lo;
}
// This thread's four tokens from pl0 on: their masks as 0/1 bytes, the last scored token of every segment.  m4: the mask bytes when all
// four lie in segment lo (fast).  Every lane of the wavefront calls it.
__device__ __forceinline__ uint32_t four_masks(const TokArgs& A, const SegWindow& W, int64_t blk0, int ntok, int pl0, int lo, bool fast, uint32_t m4) {
  const int lane = threadIdx.x & (kWave - 1);
  uint32_t mk4 = 0;
  int cand = -1;                                    // this thread's last scored token of segment lo
  if (fast) {
    mk4 = bytes_to_01(m4);
    cand = mk4 ? pl0 + (31 - __clz(mk4)) / 8 : -1;
  }
  // when the whole wavefront sits in one segment, one update of the segment's last scored token does
  const int lo0 = __shfl(lo, 0, kWave);
  if (__all(fast && lo == lo0)) {
    const int best = wave_max(cand);
    if (lane == 0 && best >= 0) atomicMax(&W.lastv[lo], best);
  } else if (cand >= 0) {
    atomicMax(&W.lastv[lo], cand);
  }
  if (pl0 < ntok && !fast) {                        // a segment boundary or the stream's end inside the four tokens
    int s = lo;
    for (int k = 0; k < kTokPerThread; ++k) {
      const int pl = pl0 + k;
      if (pl >= ntok) break;
      while (W.loc[s + 1] <= pl) ++s;               // also steps over empty segments
      const uint32_t m = A.mask_global[W.meta[s].src + (blk0 + pl - W.off[s])] ? 1u : 0u;
      mk4 |= m << (8 * k);
      if (m) atomicMax(&W.lastv[s], pl);
    }
  }
  return mk4;
}
// The six outputs of the four tokens, once every thread has been through four_masks; pl0 < ntok.
// With PAST what the calls around the update do not read again (source index, turn, role) is stored past the caches, which leaves these to the
// mask, the flags and the rewards.  Such a store has to cover whole lines, also where a segment ends inside the wavefront's 256 tokens, and
// perm's in one instruction: two tokens to a lane, first of one half of the wavefront's tokens, then of the other (sixteen of
// every 32 bytes at a time, past the caches, are slower than plain stores: 25 million tokens 139 and 112 us, whole lines 103; 42 million
// 180 and 163, and what follows finds its inputs in the cache: KL penalty of 25 million 82 -> 71 us, second pass of the whitening 56 -> 51).
template <bool PAST>
__device__ __forceinline__ void store_four(const TokArgs& A, const SegWindow& W, int64_t blk0, int ntok, int pl0, int lo, bool fast, uint32_t mk4,
                                           bool ahead) {
  const int64_t p0 = blk0 + pl0;
  const int lane = threadIdx.x & (kWave - 1);
  // a segment's last scored token carries the reward, unless the segment goes on past the block and has another
  auto last_scored = [&](int s) { return W.loc[s + 1] <= kTokBlock || !ahead ? W.lastv[s] : -1; };
  auto reward = [&](int k, int lastv, float rho) {
    return ((mk4 >> (8 * k)) & 1u) && (A.place_mode == UMAS_PLACE_ALL || pl0 + k == lastv) ? rho : 0.f;
  };
  auto put_words = [&](uint32_t fg4, const float (&rw)[kTokPerThread]) {
    *reinterpret_cast<uint32_t*>(A.tok_mask + p0) = mk4;
    *reinterpret_cast<uint32_t*>(A.tok_flags + p0) = fg4;
    *reinterpret_cast<float4*>(A.tok_reward + p0) = make_float4(rw[0], rw[1], rw[2], rw[3]);
  };
  // the two tokens of a lane in half h of the wavefront's 256: whose lane's four they belong to, and the first one's place in the block
  auto from = [&](int h) { return h * (kWave / 2) + (lane >> 1); };
  auto pair = [&](int h) { return pl0 - lane * kTokPerThread + h * 2 * kWave + lane * 2; };
  int s = lo;
  if (PAST && __ballot(fast) == ~0ull) {            // all lanes are here and have four tokens of one segment
    const SegMeta M = W.meta[s];
    const int64_t g0 = M.src + (p0 - W.off[s]);
    const int lastv = last_scored(s);
    float rw[kTokPerThread];
#pragma unroll
    for (int k = 0; k < kTokPerThread; ++k) rw[k] = reward(k, lastv, M.rho);
    const uint32_t fg4 = pl0 + kTokPerThread == W.loc[s + 1] ? mk4 | static_cast<uint32_t>(M.end_flags) << 24 : mk4;
    const int64_t a = __shfl(static_cast<long long>(g0), from(0), kWave) + 2 * (lane & 1);
    const int64_t b = __shfl(static_cast<long long>(g0), from(1), kWave) + 2 * (lane & 1);
    store_stream(A.perm + blk0 + pair(0), make_longlong2(a, a + 1));
    store_stream(A.perm + blk0 + pair(1), make_longlong2(b, b + 1));
    store_stream(A.tok_turn + p0, make_int4(M.turn, M.turn, M.turn, M.turn));
    store_stream(A.tok_role + p0, make_int4(M.role, M.role, M.role, M.role));
    put_words(fg4, rw);
    asm volatile("");                               // keeps this end apart from the paths below: stores joined with theirs would be plain (a test reads the built code)
    return;
  }
  if (PAST && __ballot(pl0 + kTokPerThread <= ntok) == ~0ull) {   // four tokens, some lanes' of several segments
    int64_t g[kTokPerThread];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      int t = __shfl(lo, from(h), kWave);
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        while (W.loc[t + 1] <= pair(h) + k) ++t;
        g[h * 2 + k] = W.meta[t].src + (blk0 + pair(h) + k - W.off[t]);
      }
    }
    int32_t turn[kTokPerThread], role[kTokPerThread];
    float rw[kTokPerThread];
    uint32_t fg4 = mk4;
#pragma unroll
    for (int k = 0; k < kTokPerThread; ++k) {
      while (W.loc[s + 1] <= pl0 + k) ++s;
      const SegMeta M = W.meta[s];
      turn[k] = M.turn;
      role[k] = M.role;
      rw[k] = reward(k, last_scored(s), M.rho);
      if (pl0 + k + 1 == W.loc[s + 1]) fg4 |= static_cast<uint32_t>(M.end_flags) << (8 * k);
    }
    store_stream(A.perm + blk0 + pair(0), make_longlong2(g[0], g[1]));
    store_stream(A.perm + blk0 + pair(1), make_longlong2(g[2], g[3]));
    store_stream(A.tok_turn + p0, make_int4(turn[0], turn[1], turn[2], turn[3]));
    store_stream(A.tok_role + p0, make_int4(role[0], role[1], role[2], role[3]));
    put_words(fg4, rw);
    asm volatile("");
    return;
  }
  if (fast) {                                       // four tokens of one segment: no per-token bookkeeping
    const SegMeta M = W.meta[s];
    const int64_t g0 = M.src + (p0 - W.off[s]);
    const int lastv = last_scored(s);
    float rw[kTokPerThread];
#pragma unroll
    for (int k = 0; k < kTokPerThread; ++k) rw[k] = reward(k, lastv, M.rho);
    *reinterpret_cast<longlong2*>(A.perm + p0) = make_longlong2(g0, g0 + 1);
    *reinterpret_cast<longlong2*>(A.perm + p0 + 2) = make_longlong2(g0 + 2, g0 + 3);
    *reinterpret_cast<int4*>(A.tok_turn + p0) = make_int4(M.turn, M.turn, M.turn, M.turn);
    *reinterpret_cast<int4*>(A.tok_role + p0) = make_int4(M.role, M.role, M.role, M.role);
    put_words(pl0 + kTokPerThread == W.loc[s + 1] ? mk4 | static_cast<uint32_t>(M.end_flags) << 24 : mk4, rw);
    return;
  }
  for (int k = 0; k < kTokPerThread; ++k) {
    const int pl = pl0 + k;
    if (pl >= ntok) break;
    while (W.loc[s + 1] <= pl) ++s;
    const SegMeta M = W.meta[s];
    const uint32_t m = (mk4 >> (8 * k)) & 1u;
    A.perm[p0 + k] = M.src + (p0 + k - W.off[s]);
    A.tok_turn[p0 + k] = M.turn;
    A.tok_role[p0 + k] = M.role;
    A.tok_mask[p0 + k] = static_cast<uint8_t>(m);
    A.tok_flags[p0 + k] = static_cast<uint8_t>(m | (pl + 1 == W.loc[s + 1] ? M.end_flags : 0));
    A.tok_reward[p0 + k] = reward(k, last_scored(s), M.rho);
  }
}

// The plain path of a block with more than kSegWin segments: one token at a time, the segment found by a search in
// global memory.  First the masks (into s_mk) ...
__device__ __forceinline__ void many_segments_masks(const TokArgs& A, int64_t blk0, int ntok, int s_first, int s_last, uint8_t* s_mk) {
  for (int pl = threadIdx.x; pl < ntok; pl += kTokThreads) {
    const int64_t p = blk0 + pl;
    const int s = s_first + last_le(A.turn_seg_off + s_first, s_last - s_first, p);
    s_mk[pl] = A.mask_global[A.seg_meta[s].src + (p - A.turn_seg_off[s])] ? 1 : 0;
  }
}
// ... then the outputs.  A scored token carries the reward of its segment if no scored token follows it there: the
// gaps between scored tokens are disjoint, so all these searches together read the block's masks once.
__device__ __forceinline__ void many_segments_outputs(const TokArgs& A, int64_t blk0, int ntok, int s_first, int s_last, const uint8_t* s_mk,
                                                   bool ahead) {
  for (int pl = threadIdx.x; pl < ntok; pl += kTokThreads) {
    const int64_t p = blk0 + pl;
    const int s = s_first + last_le(A.turn_seg_off + s_first, s_last - s_first, p);
    const SegMeta M = A.seg_meta[s];
    const int64_t seg_a = A.turn_seg_off[s], seg_e = A.turn_seg_off[s + 1];
    const uint8_t m = s_mk[pl];
    float rw = 0.f;
    if (m) {
      bool carries = A.place_mode == UMAS_PLACE_ALL;
      if (!carries) {
        const int stop = seg_e - blk0 < ntok ? static_cast<int>(seg_e - blk0) : ntok;
        int q = pl + 1;
        while (q < stop && !s_mk[q]) ++q;
        carries = q == stop && (seg_e - blk0 <= ntok || !ahead);
      }
      rw = carries ? M.rho : 0.f;
    }
    A.perm[p] = M.src + (p - seg_a);
    A.tok_turn[p] = M.turn;
    A.tok_role[p] = M.role;
    A.tok_mask[p] = m;
    A.tok_flags[p] = static_cast<uint8_t>(m | (p == seg_e - 1 ? M.end_flags : 0));
    A.tok_reward[p] = rw;
  }
}

template <bool PAST>
__global__ void __launch_bounds__(kTokThreads)
k_tokens(TokArgs A) {
  __shared__ int64_t smem[32];
  __shared__ int64_t s_off[kSegWin + 1];
  __shared__ int32_t s_loc[kSegWin + 1];            // the same offsets relative to the block's first token, clamped
  __shared__ SegMeta s_meta[kSegWin];
  __shared__ int32_t s_lastv[kSegWin];              // block-relative position of the segment's last scored token in this block, -1
  __shared__ __attribute__((aligned(16))) uint8_t s_mk[kTokBlock];   // the block's masks, 0 or 1 (plain path)
  __shared__ int s_ahead;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  const int64_t blk0 = static_cast<int64_t>(blockIdx.x) * kTokBlock;
  const int64_t blk_end = blk0 + kTokBlock < A.n_tokens ? blk0 + kTokBlock : A.n_tokens;
  const int ntok = static_cast<int>(blk_end - blk0);
  const int s_first = A.blk_first[blockIdx.x];
  // segments s_first .. s_last hold the block's tokens (s_last = the segment of the next block's first token)
  const int s_last = blk_end < A.n_tokens ? A.blk_first[blockIdx.x + 1] : A.n_turns - 1;
  const int n_seg = s_last - s_first + 1;
  const bool windowed = n_seg <= kSegWin;
  const bool mask_aligned = (reinterpret_cast<uintptr_t>(A.mask_global) & 3) == 0;
  const SegWindow win{s_off, s_loc, s_meta, s_lastv};
  if (tid == 0) s_ahead = 0;
  *reinterpret_cast<uint4*>(s_mk + tid * kCompact) = make_uint4(0u, 0u, 0u, 0u);
  if (windowed) {
    for (int i = tid; i <= n_seg; i += kTokThreads) {
      const int64_t off = A.turn_seg_off[s_first + i];
      const int64_t rel = off - blk0;
      s_off[i] = off;
      s_loc[i] = static_cast<int32_t>(rel < -(1 << 30) ? -(1 << 30) : rel > (1 << 30) ? (1 << 30) : rel);
      if (i < n_seg) { s_meta[i] = A.seg_meta[s_first + i]; s_lastv[i] = -1; }
    }
  }
  __syncthreads();

  // ---- masks: into registers (windowed path) and LDS, the last scored token of every segment
  uint32_t mk_r[kTokRounds];                        // 0/1 bytes of this thread's four tokens in each round
  int lo_r[kTokRounds];                             // their first token's segment in the window; bit 30: all four lie in it
#pragma unroll
  for (int rd = 0; rd < kTokRounds; ++rd) { mk_r[rd] = 0; lo_r[rd] = 0; }
  if (windowed) {
    uint32_t m4_r[kTokRounds];
#pragma unroll
    for (int rd = 0; rd < kTokRounds; ++rd) {       // every load of the block goes out before anything waits for one
      const int pl0 = rd * kTokRound + tid * kTokPerThread;
      m4_r[rd] = 0;
      if (pl0 >= ntok) continue;
      const int lo = segment_of(s_loc, n_seg, pl0);
      const bool fast = pl0 + kTokPerThread <= s_loc[lo + 1];
      lo_r[rd] = lo | (fast ? 1 << 30 : 0);
      if (fast) m4_r[rd] = load_mask4(A.mask_global, s_meta[lo].src + (blk0 + pl0 - s_off[lo]), mask_aligned);
    }
#pragma unroll
    for (int rd = 0; rd < kTokRounds; ++rd) {
      const int pl0 = rd * kTokRound + tid * kTokPerThread;
      mk_r[rd] = four_masks(A, win, blk0, ntok, pl0, lo_r[rd] & ((1 << 30) - 1), (lo_r[rd] >> 30) != 0, m4_r[rd]);
    }
  } else {
    many_segments_masks(A, blk0, ntok, s_first, s_last, s_mk);
  }
  // the block's last segment, if it goes on past the block: is there a scored token further on?
  if (wave == 1 && A.place_mode == UMAS_PLACE_LAST && A.turn_seg_off[s_last + 1] > blk_end) {
    const int64_t a = A.turn_seg_off[s_last];
    const bool found = scored_token_ahead(A, A.seg_meta[s_last].src, A.turn_seg_off[s_last + 1] - a, blk_end - a);
    if (lane == 0) s_ahead = found ? 1 : 0;
  }
  __syncthreads();
  const bool ahead = s_ahead != 0;

  // ---- the block's count of scored tokens, for the compaction kernel: its own word and its group's total
  {
    int32_t c = 0;
    if (windowed) {
#pragma unroll
      for (int rd = 0; rd < kTokRounds; ++rd) c += __popc(mk_r[rd]);
    } else {
      const uint4 w = *reinterpret_cast<const uint4*>(s_mk + tid * kCompact);
      c = __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
    }
    const int32_t total = block_sum<int32_t>(c, reinterpret_cast<int32_t*>(smem));
    if (tid == 0) {
      A.blk_count[blockIdx.x] = static_cast<unsigned long long>(total);
      (void)__hip_atomic_fetch_add(A.grp_count + (blockIdx.x >> A.grp_shift), static_cast<unsigned long long>(total), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
    }
  }

  // ---- outputs per token
  if (windowed) {
#pragma unroll
    for (int rd = 0; rd < kTokRounds; ++rd) {
      const int pl0 = rd * kTokRound + tid * kTokPerThread;
      if (pl0 < ntok) store_four<PAST>(A, win, blk0, ntok, pl0, lo_r[rd] & ((1 << 30) - 1), (lo_r[rd] >> 30) != 0, mk_r[rd], ahead);
    }
  } else {
    many_segments_outputs(A, blk0, ntok, s_first, s_last, s_mk, ahead);
  }

}

// The compacted list of scored positions, per stream and stream-relative, from the masks in model-local order.  A
// block of 4096 tokens finds the number of scored tokens in front of it as the totals of the groups of blocks before
// its group plus the counts of the blocks before it in its group, all written by the token kernel.
struct SelArgs {
  int64_t n_tokens;
  int n_models, grp_shift;
  const uint8_t* tok_mask;
  const int64_t* model_tok_off;
  const unsigned long long* blk_count;
  const unsigned long long* grp_count;
  int32_t* rowsel;
  int64_t* model_rowsel_off;
};

constexpr int kSelMul = 2;                          // blocks of the token kernel to one block of the compaction kernel
constexpr int kSelBlock = kTokBlock * kSelMul;
constexpr int kSelPerThread = kSelBlock / kTokThreads;
constexpr int kSelWords = kSelPerThread / 4;

// Place of compacted entry i in LDS: eight bytes are left out after every 32 entries.  Where most tokens are scored, neighbouring threads
// write 32 entries apart, which would be four banks of the 64 for a whole wavefront (42 million tokens, all scored: 54 us, spread like
// this 37 to 44; 25 million of which 80 % are scored 25.5 and 23).
__host__ __device__ constexpr int sel_slot(int i) { return i + 4 * (i / 32); }
static_assert(kSelPerThread == 32, "what a thread writes where all its tokens are scored");

__global__ void __launch_bounds__(kTokThreads)
k_rowsel(SelArgs A) {
  __shared__ int64_t smem[32];
  __shared__ __attribute__((aligned(8))) uint16_t s_out[sel_slot(kSelBlock + 4)];   // the block's scored positions, block-relative, compacted
  __shared__ int64_t moff[UMAS_MAX_MODELS + 1];
  __shared__ int32_t s_mro[UMAS_MAX_MODELS + 1];    // scored tokens of the block in front of a stream that starts in it, -1
  const int tid = threadIdx.x;
  const int64_t blk0 = static_cast<int64_t>(blockIdx.x) * kSelBlock;
  const int64_t blk_end = blk0 + kSelBlock < A.n_tokens ? blk0 + kSelBlock : A.n_tokens;
  if (tid <= A.n_models) { moff[tid] = A.model_tok_off[tid]; s_mro[tid] = -1; }
  // what lies in front of the block
  int64_t part = 0;
  {
    const int64_t first = static_cast<int64_t>(blockIdx.x) * kSelMul;   // in blocks of the token kernel
    const int64_t grp = first >> A.grp_shift;
    for (int64_t g = tid; g < grp; g += kTokThreads) part += static_cast<int64_t>(A.grp_count[g]);
    for (int64_t k = (grp << A.grp_shift) + tid; k < first; k += kTokThreads) part += static_cast<int64_t>(A.blk_count[k]);
  }
  const int64_t p0 = blk0 + tid * kSelPerThread;
  uint32_t w4[kSelWords];
#pragma unroll
  for (int k = 0; k < kSelWords; ++k) w4[k] = 0u;
  if (p0 + kSelPerThread <= A.n_tokens) {
#pragma unroll
    for (int q = 0; q < kSelWords / 4; ++q) {
      const uint4 w = *reinterpret_cast<const uint4*>(A.tok_mask + p0 + 16 * q);
      w4[4 * q] = w.x; w4[4 * q + 1] = w.y; w4[4 * q + 2] = w.z; w4[4 * q + 3] = w.w;
    }
  } else {
    for (int k = 0; k < kSelPerThread; ++k)
      if (p0 + k < A.n_tokens) w4[k >> 2] |= static_cast<uint32_t>(A.tok_mask[p0 + k]) << (8 * (k & 3));
  }
  const int64_t prefix = block_sum<int64_t>(part, smem);
  int32_t c = 0;                                    // mask bytes are 0 or 1
#pragma unroll
  for (int k = 0; k < kSelWords; ++k) c += __popc(w4[k]);
  int32_t block_count;
  int o = block_excl_scan<int32_t>(c, reinterpret_cast<int32_t*>(smem), &block_count);
  // The entries leave single up to the first 16-byte boundary of rowsel, four to a store from there; they are staged
  // `pad` places further on so that every such group of four starts at an 8-byte boundary of s_out.
  int32_t* const dst = A.rowsel + prefix;
  const int to_boundary = static_cast<int>((4 - ((reinterpret_cast<uintptr_t>(dst) >> 2) & 3)) & 3);
  const int pad = (4 - to_boundary) & 3;
  // a stream may start inside the block: the scored tokens in front of its first token give its place in rowsel
  const int e = o;
#pragma unroll
  for (int k = 0; k < kSelPerThread; ++k)
    if ((w4[k >> 2] >> (8 * (k & 3))) & 1u) s_out[sel_slot(pad + o++)] = static_cast<uint16_t>(tid * kSelPerThread + k);
  for (int j = 0; j <= A.n_models; ++j) {
    const int64_t q = moff[j] - p0;
    if (q >= 0 && q < kSelPerThread && moff[j] < A.n_tokens) {
      int before = 0;
#pragma unroll
      for (int k = 0; k < kSelPerThread; ++k) before += k < q ? static_cast<int>((w4[k >> 2] >> (8 * (k & 3))) & 1u) : 0;
      s_mro[j] = e + before;
    }
  }
  __syncthreads();
  for (int j = tid; j <= A.n_models; j += kTokThreads)
    if (s_mro[j] >= 0) A.model_rowsel_off[j] = prefix + s_mro[j];
  int m0 = 0;                                        // the stream of the block's first token
  while (m0 < A.n_models && moff[m0 + 1] <= blk0) ++m0;
  auto entry = [&](int i) -> int32_t {               // compacted entry i of the block, stream-relative
    const int64_t p = blk0 + s_out[sel_slot(pad + i)];
    int m = m0;
    while (m < A.n_models && moff[m + 1] <= p) ++m;
    return static_cast<int32_t>(p - moff[m]);
  };
  const bool one_stream = moff[m0 + 1] >= blk_end;   // the usual case: every entry is relative to the same start
  const int32_t rel0 = static_cast<int32_t>(blk0 - moff[m0]);
  const int head = to_boundary < block_count ? to_boundary : block_count;
  const int n_vec = (block_count - head) / 4;
  if (tid < head) dst[tid] = entry(tid);
  for (int v = tid; v < n_vec; v += kTokThreads) {
    const int i = head + 4 * v;
    if (one_stream) {
      const uint2 q = *reinterpret_cast<const uint2*>(s_out + sel_slot(pad + i));
      *reinterpret_cast<int4*>(dst + i) = make_int4(rel0 + static_cast<int32_t>(q.x & 0xffffu), rel0 + static_cast<int32_t>(q.x >> 16),
                                                   rel0 + static_cast<int32_t>(q.y & 0xffffu), rel0 + static_cast<int32_t>(q.y >> 16));
    } else {
      *reinterpret_cast<int4*>(dst + i) = make_int4(entry(i), entry(i + 1), entry(i + 2), entry(i + 3));
    }
  }
  {
    const int i = head + 4 * n_vec + tid;
    if (i < block_count) dst[i] = entry(i);
  }
  if (blk_end == A.n_tokens && tid == 0)             // streams that start at the very end hold nothing
    for (int j = 0; j <= A.n_models; ++j)
      if (moff[j] >= A.n_tokens) A.model_rowsel_off[j] = prefix + block_count;
}

// ------------------------------------------------------------------ small graphs: everything in one launch
// A batch of up to 65 536 tokens is a matter of launches: copy, normalisation, plan, tokens and compaction one behind the other
// are 5 us each at the least, most of them a chain of loads that miss.  Here every workgroup reads the thin arrays from the pinned
// block itself (a few KB: one trip over the bus), makes the whole plan in LDS, and writes a block of 4096 tokens, four to a
// thread; what lies in front of the block is not asked of the others but counted in the mask.  The first workgroup writes the
// outputs per turn.  Copy, plan, tokens and compaction of 46 000 tokens in 115 turns: 39 us on the device, 12.7 in one launch; of 768
// tokens in 24 turns: 30 and 8.2 (the whole float32 step 92 -> 78).  At the limit of tokens, each call waited for: in 16 turns 54 and 45 us, in
// 512 72 and 56, in 500 of eight models and 25 groups 172 and 94.
constexpr int kSmallThreads = kTokBlock / kTokPerThread;
constexpr int kSmallTurns = 512;                   // LDS: 48 bytes a turn, 4 a trajectory and the thin arrays
constexpr size_t kSmallThin = 24 << 10;
constexpr int kSmallTraj = kSmallThreads;          // one thread each
constexpr int kSmallGroups = 128;                  // eight rounds of the workgroup's wavefronts
constexpr int kSmallTokens = 16 * kTokBlock;
constexpr size_t kSmallBus = 192 << 10;            // thin arrays times workgroups: 5 us at the rate of the bus
static_assert(kSmallThin + kSmallTurns * (sizeof(int64_t) + sizeof(SegMeta) + 2 * sizeof(int32_t)) + kSmallTraj * sizeof(float) + 2048 <= 64 << 10,
              "what a workgroup holds fits its LDS, 2 KB for sums and counts");

struct SmallArgs {
  PlanArgs plan;                                   // thin arrays: as if they lay in the workspace
  TokArgs tok;
  const char* ws;
  const char* thin;
  int thin16, n_groups;
  float norm_eps;
  const int32_t* group_off;
  const int32_t* group_members;
  int32_t* rowsel;
};

struct SmallSink {
  const PlanArgs& A;
  int64_t* off;
  int32_t* loc;
  SegMeta* meta;
  int64_t blk0;
  bool publish;
  __device__ __forceinline__ void run(int64_t r, int64_t o) const {
    if (publish) A.traj_seg_off[r] = o;
  }
  __device__ __forceinline__ void turn(int64_t slot, int64_t o, int64_t, int step, const SegMeta& M) const {
    off[slot] = o;
    loc[slot] = static_cast<int32_t>(o - blk0);
    meta[slot] = M;
    if (publish) publish_turn(A, slot, o, step, M);
  }
  __device__ __forceinline__ void end_flags(int slot, int32_t f) const { meta[slot].end_flags = f; }
};

template <int KM>
__global__ void __launch_bounds__(kSmallThreads)
k_route_small(SmallArgs A) {
  constexpr int nwave = kSmallThreads / kWave;
  __shared__ __attribute__((aligned(16))) char s_thin[kSmallThin];
  __shared__ int64_t s_off[kSmallTurns + 1];
  __shared__ int32_t s_loc[kSmallTurns + 1];
  __shared__ SegMeta s_meta[kSmallTurns];
  __shared__ int32_t s_lastv[kSmallTurns];
  __shared__ float s_norm[kSmallTraj];
  __shared__ int64_t s_sum[KM][nwave];
  __shared__ int32_t s_cnt[2][nwave];
  __shared__ int s_ahead;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int K = A.plan.n_models, U = A.plan.n_turns, B = A.plan.n_traj, N = static_cast<int>(A.plan.n_tokens);
  const int blk0 = blockIdx.x * kTokBlock, ntok = N - blk0 < kTokBlock ? N - blk0 : kTokBlock;
  // ---- the thin arrays
  {
    const uint4* const from = reinterpret_cast<const uint4*>(A.thin);
    for (int i = tid; i < A.thin16; i += kSmallThreads) reinterpret_cast<uint4*>(s_thin)[i] = from[i];
    for (int i = tid; i < U; i += kSmallThreads) s_lastv[i] = -1;
    if (tid == 0) s_ahead = 0;
  }
  __syncthreads();
  auto here = [&](auto* p) { return reinterpret_cast<decltype(p)>(s_thin + (reinterpret_cast<const char*>(p) - A.ws)); };
  PlanArgs L = A.plan;
  L.traj_turn_off = here(L.traj_turn_off);
  L.turn_role = here(L.turn_role);
  L.tok_off32 = here(L.tok_off32);
  const int32_t* const phi = here(L.role_to_model);
  if (L.role_reward) L.role_reward = here(L.role_reward);
  if (L.turn_reward) L.turn_reward = here(L.turn_reward);
  if (L.traj_reward) L.traj_reward = here(L.traj_reward);
  if (L.w_role) L.w_role = here(L.w_role);
  if (L.w_turn) L.w_turn = here(L.w_turn);
  if (L.w_traj) L.w_traj = here(L.w_traj);
  if (A.n_groups > 0) {
    const int32_t *const goff = here(A.group_off), *const members = A.group_members ? here(A.group_members) : nullptr;
    for (int g = wave; g < A.n_groups; g += nwave) normalise_group(L.traj_reward, members, goff[g], goff[g + 1], A.norm_eps, s_norm);
    L.traj_reward = s_norm;
    __syncthreads();
  }
  // ---- the plan: one thread per trajectory; turns, runs and tokens of a model in one word
  int64_t slot_at[KM], tok_at[KM], run_at[KM];
  int tok_start[KM];                                // first token of every stream
  {
    TrajCounts<KM> tc;
    traj_counts(L, phi, tid, tc);
    int64_t excl[KM];
#pragma unroll
    for (int k = 0; k < KM; ++k) {
      const int64_t v = tc.cnt[k] | static_cast<int64_t>((tc.seen >> k) & 1u) << 20 | tc.tok[k] << 40;
      const int64_t incl = wave_incl_scan(v);
      excl[k] = incl - v;
      if (lane == kWave - 1) s_sum[k][wave] = incl;
    }
    __syncthreads();
    constexpr int64_t kField = (1 << 20) - 1;
    int64_t bs = 0, bt = 0, br = 0;
    const int nw = (B + kWave - 1) / kWave;
    const bool first = blockIdx.x == 0 && tid == 0;
#pragma unroll
    for (int k = 0; k < KM; ++k) {
      int64_t total = 0, before = excl[k];
      for (int w = 0; w < nw; ++w) {
        const int64_t t = s_sum[k][w];
        total += t;
        before += w < wave ? t : 0;
      }
      if (first && k < K) {
        A.plan.model_turn_off[k] = static_cast<int32_t>(bs);
        A.plan.model_tok_off[k] = bt;
        A.plan.model_trajrun_off[k] = static_cast<int32_t>(br);
      }
      tok_start[k] = static_cast<int>(bt);
      slot_at[k] = bs + (before & kField);
      run_at[k] = br + ((before >> 20) & kField);
      tok_at[k] = bt + (before >> 40);
      bs += total & kField;
      br += (total >> 20) & kField;
      bt += total >> 40;
    }
    if (first) {
      A.plan.model_turn_off[K] = static_cast<int32_t>(bs);
      A.plan.model_tok_off[K] = bt;
      A.plan.model_trajrun_off[K] = static_cast<int32_t>(br);
      A.plan.turn_seg_off[U] = N;
    }
    if (blockIdx.x == 0)                            // entries of traj_seg_off past the runs read n_tokens
      for (int i = static_cast<int>(br) + tid; i <= U; i += kSmallThreads) A.plan.traj_seg_off[i] = N;
  }
  if (tid < B) walk_turns(L, phi, tid, slot_at, tok_at, run_at, SmallSink{A.plan, s_off, s_loc, s_meta, blk0, blockIdx.x == 0});
  if (tid == 0) {
    s_off[U] = N;
    s_loc[U] = N - blk0;
  }
  __syncthreads();
  // ---- the block's masks, and the number of scored tokens in front of it, sixteen tokens to a load
  const SegWindow win{s_off, s_loc, s_meta, s_lastv};
  const int pl0 = tid * kTokPerThread;
  int lo = 0;
  bool fast = false;
  uint32_t m4 = 0;
  if (pl0 < ntok) {
    lo = segment_of(s_loc, U, pl0);
    fast = pl0 + kTokPerThread <= s_loc[lo + 1];
    if (fast) m4 = load_mask4(A.tok.mask_global, s_meta[lo].src + (pl0 - s_loc[lo]), (reinterpret_cast<uintptr_t>(A.tok.mask_global) & 3) == 0);
  }
  int32_t before = 0;
  for (int p = tid * 16 - blk0; p < 0; p += kSmallThreads * 16) {   // block-relative; blk0 is a multiple of 16
    int s = segment_of(s_loc, U, p);
    const uint8_t* const at = A.tok.mask_global + s_meta[s].src + (p - s_loc[s]);
    if (p + 16 <= s_loc[s + 1]) {
      uint32_t w[4];
      __builtin_memcpy(w, at, 16);                  // at any address
      before += __popc(bytes_to_01(w[0])) + __popc(bytes_to_01(w[1])) + __popc(bytes_to_01(w[2])) + __popc(bytes_to_01(w[3]));
    } else {
      for (int k = 0; k < 16; ++k) {
        while (s_loc[s + 1] <= p + k) ++s;
        before += A.tok.mask_global[s_meta[s].src + (p + k - s_loc[s])] ? 1 : 0;
      }
    }
  }
  const uint32_t mk4 = four_masks(A.tok, win, blk0, ntok, pl0, lo, fast, m4);
  // the segment that goes on past the block, if one does: is there a scored token further on?
  if (wave == 1 && A.tok.place_mode == UMAS_PLACE_LAST && blk0 + ntok < N) {
    const int s = segment_of(s_loc, U, ntok);
    if (s_loc[s] < ntok) {
      const bool found = scored_token_ahead(A.tok, s_meta[s].src, s_loc[s + 1] - s_loc[s], ntok - s_loc[s]);
      if (lane == 0) s_ahead = found ? 1 : 0;
    }
  }
  const int32_t c = __popc(mk4);
  int32_t o = wave_incl_scan(c);
  before = wave_sum(before);
  if (lane == kWave - 1) {
    s_cnt[0][wave] = o;
    s_cnt[1][wave] = before;
  }
  __syncthreads();
  o -= c;
  int32_t end = 0;                                  // scored tokens up to the block's end
#pragma unroll
  for (int w = 0; w < nwave; ++w) {
    const int32_t t = s_cnt[0][w], b = s_cnt[1][w];
    o += b + (w < wave ? t : 0);
    end += b + t;
  }
  if (pl0 < ntok) {
    store_four<false>(A.tok, win, blk0, ntok, pl0, lo, fast, mk4, s_ahead != 0);
    // the scored positions, stream-relative, and where the streams that start here begin among them
#pragma unroll
    for (int k = 0; k < kTokPerThread; ++k) {
      const int p = blk0 + pl0 + k;
      int start = 0;
#pragma unroll
      for (int m = 0; m < KM; ++m) {
        if (m < K && tok_start[m] == p && p < N) A.plan.model_rowsel_off[m] = o;
        start = m < K && tok_start[m] <= p ? tok_start[m] : start;
      }
      if ((mk4 >> (8 * k)) & 1u) A.rowsel[o++] = p - start;
    }
  }
  if (blk0 + ntok == N && tid == 0) {               // streams that start at the very end hold nothing
#pragma unroll
    for (int m = 0; m < KM; ++m)
      if (m < K && tok_start[m] == N) A.plan.model_rowsel_off[m] = end;
    A.plan.model_rowsel_off[K] = end;
  }
}

// ------------------------------------------------------------------ host side
// The trajectories of every group that occurs, by group and ascending in it: members as a CSR with offsets off.  Groups that
// arrive in order (members next to each other) need no sorting and no list of members, group numbers that are not much larger than the number of
// trajectories are counted, a stable sort by comparison is left for the rest: 32 768 trajectories in order 617 -> 19 us, in any
// order 50.
void group_members(const int32_t* group, int n, std::vector<int32_t>* off, std::vector<int32_t>* mem) {
  off->reserve(static_cast<size_t>(n) + 1);
  off->push_back(0);
  if (std::is_sorted(group, group + n)) {
    for (int b = 1; b < n; ++b)
      if (group[b] != group[b - 1]) off->push_back(b);
  } else {
    mem->resize(n);
    const int32_t top = *std::max_element(group, group + n);
    if (top < 4 * static_cast<int64_t>(n) + 1024) {
      std::vector<int32_t> at(static_cast<size_t>(top) + 2, 0);
      for (int b = 0; b < n; ++b) ++at[static_cast<size_t>(group[b]) + 1];
      for (size_t k = 0; k <= static_cast<size_t>(top); ++k) {     // (top may be the largest int32)
        if (at[k + 1] > 0 && at[k] > 0) off->push_back(at[k]);
        at[k + 1] += at[k];
      }
      for (int b = 0; b < n; ++b) (*mem)[at[group[b]]++] = b;
    } else {
      for (int b = 0; b < n; ++b) (*mem)[b] = b;
      std::stable_sort(mem->begin(), mem->end(), [&](int32_t x, int32_t y) { return group[x] < group[y]; });
      for (int i = 1; i < n; ++i)
        if (group[(*mem)[i]] != group[(*mem)[i - 1]]) off->push_back(i);
    }
  }
  off->push_back(n);
}
// Whether every turn and predecessor is well-formed, without naming one that is not: a negative number is looked for among the offsets, their differences
// and the room to each limit, or'ed together (where an offset or entry is not negative itself, no difference overflows).  One turn after the other with an
// exit in every step took what registers the call that launches had left: 1.4 million turns with a predecessor each 3.58 ms, with a launch more
// in that call 3.75, like this 2.92; the call 4.16, 4.35 and 3.65, of 201 240 turns 360, 372 and 333 us.
__attribute__((noinline)) bool turns_well_formed(int n_turns, int n_roles, const int64_t* __restrict__ tok_off, const int32_t* __restrict__ role) {
  int64_t off = tok_off[n_turns];
  int32_t roles = 0;
  for (int u = 0; u < n_turns; ++u) off |= tok_off[u] | static_cast<int64_t>(static_cast<uint64_t>(tok_off[u + 1]) - static_cast<uint64_t>(tok_off[u]));
  for (int u = 0; u < n_turns; ++u) roles |= role[u] | static_cast<int32_t>(static_cast<uint32_t>(n_roles - 1) - static_cast<uint32_t>(role[u]));
  return off >= 0 && roles >= 0;
}
__attribute__((noinline)) bool predecessors_well_formed(int n_traj, int n_turns, const int32_t* __restrict__ traj_off, const int32_t* __restrict__ pred_off,
                                                        const int32_t* __restrict__ pred) {
  int32_t bad = pred_off[n_turns];
  for (int u = 0; u < n_turns; ++u) bad |= pred_off[u] | static_cast<int32_t>(static_cast<uint32_t>(pred_off[u + 1]) - static_cast<uint32_t>(pred_off[u]));
  if (bad < 0) return false;
  for (int b = 0; b < n_traj; ++b) {
    const uint32_t first = static_cast<uint32_t>(traj_off[b]);
    for (int u = traj_off[b]; u < traj_off[b + 1]; ++u)
      for (int e = pred_off[u]; e < pred_off[u + 1]; ++e)
        bad |= pred[e] | static_cast<int32_t>(static_cast<uint32_t>(pred[e]) - first) | static_cast<int32_t>(static_cast<uint32_t>(u - 1) - static_cast<uint32_t>(pred[e]));
  }
  return bad >= 0;
}
umas_status validate(const umas_graph* g, const umas_rewards* r, const umas_streams* o) {
  UMAS_REQUIRE(g && r && o, UMAS_EINVAL, "graph, rewards and out must not be NULL");
  UMAS_REQUIRE(g->n_roles >= 1 && g->n_roles <= UMAS_MAX_ROLES, UMAS_ESHAPE, "n_roles=%d outside [1,%d]",
               g->n_roles, UMAS_MAX_ROLES);
  UMAS_REQUIRE(g->n_models >= 1 && g->n_models <= UMAS_MAX_MODELS, UMAS_ESHAPE, "n_models=%d outside [1,%d]",
               g->n_models, UMAS_MAX_MODELS);
  UMAS_REQUIRE(g->n_traj >= 0 && g->n_turns >= 0 && g->n_tokens >= 0, UMAS_EINVAL, "negative size");
  UMAS_REQUIRE(g->role_to_model && g->traj_turn_off && g->turn_tok_off && (g->turn_role || g->n_turns == 0),
               UMAS_EINVAL, "role_to_model, traj_turn_off, turn_role, turn_tok_off must not be NULL");
  for (int v = 0; v < g->n_roles; ++v)
    UMAS_REQUIRE(g->role_to_model[v] >= 0 && g->role_to_model[v] < g->n_models, UMAS_EINVAL,
                 "role_to_model[%d]=%d is not a model in [0,%d)", v, g->role_to_model[v], g->n_models);
  UMAS_REQUIRE(g->traj_turn_off[0] == 0 && g->traj_turn_off[g->n_traj] == g->n_turns, UMAS_EINVAL,
               "traj_turn_off must run from 0 to n_turns");
  for (int b = 0; b < g->n_traj; ++b)
    UMAS_REQUIRE(g->traj_turn_off[b] <= g->traj_turn_off[b + 1], UMAS_EINVAL, "traj_turn_off decreases at %d", b);
  UMAS_REQUIRE(g->turn_tok_off[0] == 0 && g->turn_tok_off[g->n_turns] == g->n_tokens, UMAS_EINVAL,
               "turn_tok_off must run from 0 to n_tokens");
  if (!turns_well_formed(g->n_turns, g->n_roles, g->turn_tok_off, g->turn_role))
    for (int u = 0; u < g->n_turns; ++u) {
      UMAS_REQUIRE(g->turn_tok_off[u] <= g->turn_tok_off[u + 1], UMAS_EINVAL, "turn_tok_off decreases at %d", u);
      UMAS_REQUIRE(g->turn_role[u] >= 0 && g->turn_role[u] < g->n_roles, UMAS_EINVAL,
                   "turn_role[%d]=%d is not a role in [0,%d)", u, g->turn_role[u], g->n_roles);
    }
  // rowsel holds positions relative to the stream's start as int32
  if (g->n_tokens > INT32_MAX) {
    int64_t stream_tokens[UMAS_MAX_MODELS] = {};
    for (int u = 0; u < g->n_turns; ++u) stream_tokens[g->role_to_model[g->turn_role[u]]] += g->turn_tok_off[u + 1] - g->turn_tok_off[u];
    for (int m = 0; m < g->n_models; ++m)
      UMAS_REQUIRE(stream_tokens[m] <= INT32_MAX, UMAS_ESHAPE, "the stream of model %d would hold %lld tokens, more than 2^31 - 1", m,
                   static_cast<long long>(stream_tokens[m]));
  }
  if (g->turn_pred_off) {
    UMAS_REQUIRE(g->turn_pred || g->turn_pred_off[g->n_turns] == 0, UMAS_EINVAL, "turn_pred is NULL");
    UMAS_REQUIRE(g->turn_pred_off[0] == 0, UMAS_EINVAL, "turn_pred_off must start at 0");
    if (!predecessors_well_formed(g->n_traj, g->n_turns, g->traj_turn_off, g->turn_pred_off, g->turn_pred)) {
      for (int u = 0; u < g->n_turns; ++u)
        UMAS_REQUIRE(g->turn_pred_off[u] <= g->turn_pred_off[u + 1], UMAS_EINVAL, "turn_pred_off decreases at %d", u);
      for (int u = 0, b = 0; u < g->n_turns; ++u) {
        while (g->traj_turn_off[b + 1] <= u) ++b;
        for (int e = g->turn_pred_off[u]; e < g->turn_pred_off[u + 1]; ++e)
          UMAS_REQUIRE(g->turn_pred[e] >= g->traj_turn_off[b] && g->turn_pred[e] < u, UMAS_EINVAL,
                       "predecessor %d of turn %d is not an earlier turn of the same trajectory", g->turn_pred[e], u);
      }
    }
  }
  if (g->traj_group)
    for (int b = 0; b < g->n_traj; ++b)
      UMAS_REQUIRE(g->traj_group[b] >= 0, UMAS_EINVAL, "traj_group[%d] is negative", b);
  UMAS_REQUIRE(r->place_mode == UMAS_PLACE_LAST || r->place_mode == UMAS_PLACE_ALL, UMAS_EINVAL,
               "place_mode=%d is neither LAST nor ALL", r->place_mode);
  UMAS_REQUIRE(r->norm_eps > 0.0f, UMAS_EINVAL, "norm_eps must be positive");
  UMAS_REQUIRE(o->model_tok_off && o->perm && o->tok_turn && o->tok_role && o->tok_mask && o->tok_reward &&
                   o->turn_seg_off && o->seg_turn && o->model_turn_off && o->traj_seg_off &&
                   o->model_trajrun_off && o->rowsel && o->model_rowsel_off && o->turn_scalar && o->turn_step &&
                   o->tok_flags,
               UMAS_EINVAL, "every pointer of the output streams must be set");
  // the token kernel writes four tokens of every per-token array in one store
  auto aligned16 = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
  UMAS_REQUIRE(aligned16(o->perm) && aligned16(o->tok_turn) && aligned16(o->tok_role) && aligned16(o->tok_mask) &&
                   aligned16(o->tok_flags) && aligned16(o->tok_reward),
               UMAS_EINVAL, "perm, tok_turn, tok_role, tok_mask, tok_flags and tok_reward must be 16-byte aligned");
  return UMAS_OK;
}


}  // namespace
}  // namespace umas

using namespace umas;

extern "C" size_t umas_assign_workspace_bytes(const umas_graph* g) {
  if (!g || g->n_roles < 0 || g->n_traj < 0 || g->n_turns < 0 || g->n_tokens < 0) return 0;
  Carver c(nullptr);
  RouteWs w;
  return carve(c, w, g->n_roles, g->n_traj, g->n_turns, g->n_tokens);
}

extern "C" umas_status umas_assign_token_rewards(const umas_graph* g, const umas_rewards* r,
                                                 const uint8_t* tok_mask_global, const umas_streams* o,
                                                 void* workspace, size_t workspace_bytes, void* hip_stream) {
  umas_status vs = validate(g, r, o);
  if (vs != UMAS_OK) return vs;
  UMAS_REQUIRE(tok_mask_global || g->n_tokens == 0, UMAS_EINVAL, "tok_mask_global is NULL");
  const size_t need = umas_assign_workspace_bytes(g);
  UMAS_REQUIRE(workspace && reinterpret_cast<uintptr_t>(workspace) % kAlign == 0 && workspace_bytes >= need,
               UMAS_EWORKSPACE, "workspace must be 256-byte aligned and hold %zu bytes (got %zu)", need,
               workspace_bytes);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  prof_mark(st);
  const int R = g->n_roles, K = g->n_models, B = g->n_traj, U = g->n_turns;
  const int64_t N = g->n_tokens;
  // members of each normalisation group, as a CSR over the groups that occur
  Thin has;
  has.role_reward = r->role_reward; has.turn_reward = r->turn_reward; has.traj_reward = r->traj_reward;
  has.weights = r->w_role || r->w_turn || r->w_traj;
  has.wide_offsets = N >> 32 != 0;
  int n_groups = 0;
  std::vector<int32_t> goff, gmem;
  if (g->traj_group && r->traj_reward && B > 0) {
    group_members(g->traj_group, B, &goff, &gmem);
    n_groups = static_cast<int>(goff.size()) - 1;
  }
  has.groups = n_groups;
  has.members = !gmem.empty();
  Carver c(workspace);
  RouteWs w;
  carve(c, w, R, B, U, N, has);

  // The thin arrays are the first arrays of the workspace, up to traj_norm: they are gathered at the same offsets in a
  // block of pinned host memory, from where one kernel takes them over the bus, together with the zeros that the plan
  // kernel's per-chunk totals start from.  The host arrays have been read when the call returns; the host does not
  // wait for the stream.
  char* const ws_base = static_cast<char*>(workspace);
  const size_t staged_bytes = static_cast<size_t>(reinterpret_cast<char*>(w.traj_norm) - ws_base);
  const int n_chunks = plan_chunks(B);
  ThinStage stage;
  vs = stage.begin(staged_bytes, st);
  if (vs != UMAS_OK) return vs;
  auto put = [&](const void* dst, const void* src, size_t bytes) {
    stage.put(static_cast<size_t>(static_cast<const char*>(dst) - ws_base), src, bytes);
  };
  put(w.role_to_model, g->role_to_model, sizeof(int32_t) * R);
  put(w.traj_turn_off, g->traj_turn_off, sizeof(int32_t) * (static_cast<size_t>(B) + 1));
  {
    // Pointers of their own that do not overlap: a store of bytes may change anything, also where the graph says that its arrays lie, and then
    // the host takes one turn at a time (2.4 million turns of 16 tokens 5.7 ms a call with its scan, 4.9 like this; 250 000 565 and 486 us).
    char* const block = stage.at(0);
    const int32_t* __restrict__ const turn_role = g->turn_role;
    const int64_t* __restrict__ const turn_tok_off = g->turn_tok_off;
    uint8_t* __restrict__ const role = reinterpret_cast<uint8_t*>(block + (reinterpret_cast<char*>(w.turn_role) - ws_base));
    for (int u = 0; u < U; ++u) role[u] = static_cast<uint8_t>(turn_role[u]);
    static_assert(UMAS_MAX_ROLES <= 256, "a role is a byte");
    uint32_t* __restrict__ const off = reinterpret_cast<uint32_t*>(block + (reinterpret_cast<char*>(w.tok_off32) - ws_base));
    if (has.wide_offsets) put(w.tok_off64, turn_tok_off, sizeof(int64_t) * (static_cast<size_t>(U) + 1));
    else
      for (int u = 0; u <= U; ++u) off[u] = static_cast<uint32_t>(turn_tok_off[u]);
  }
  put(w.role_reward, r->role_reward, sizeof(float) * static_cast<size_t>(B) * R);
  put(w.turn_reward, r->turn_reward, sizeof(float) * U);
  put(w.traj_reward, r->traj_reward, sizeof(float) * B);
  if (has.weights) {
    put(w.weights, r->w_role, sizeof(float) * R);
    put(w.weights + R, r->w_turn, sizeof(float) * R);
    put(w.weights + 2 * R, r->w_traj, sizeof(float) * R);
  }
  if (n_groups > 0) {
    put(w.group_off, goff.data(), sizeof(int32_t) * goff.size());
    put(w.group_members, gmem.data(), sizeof(int32_t) * gmem.size());
  }
  const int64_t nbk = cdiv(N > 0 ? N : 1, kTokBlock);
  PlanArgs P;
  P.n_traj = B; P.n_turns = U; P.n_roles = R; P.n_models = K; P.n_chunks = n_chunks;
  const int gsh = group_shift(nbk);
  P.n_tokens = N; P.n_count = nbk + (nbk >> gsh) + 1;
  P.traj_turn_off = w.traj_turn_off; P.turn_role = w.turn_role; P.role_to_model = w.role_to_model;
  P.tok_off32 = has.wide_offsets ? nullptr : w.tok_off32; P.tok_off64 = w.tok_off64;
  P.role_reward = r->role_reward ? w.role_reward : nullptr;
  P.turn_reward = r->turn_reward ? w.turn_reward : nullptr;
  P.traj_reward = r->traj_reward ? w.traj_reward : nullptr;
  P.w_role = r->w_role ? w.weights : nullptr;
  P.w_turn = r->w_turn ? w.weights + R : nullptr;
  P.w_traj = r->w_traj ? w.weights + 2 * R : nullptr;
  P.plan_part = w.plan_part; P.seg_meta = w.seg_meta; P.blk_first = w.blk_first;
  P.tok_count = w.tok_count;
  P.model_tok_off = o->model_tok_off; P.model_turn_off = o->model_turn_off; P.model_trajrun_off = o->model_trajrun_off;
  P.model_rowsel_off = o->model_rowsel_off; P.turn_seg_off = o->turn_seg_off; P.seg_turn = o->seg_turn;
  P.traj_seg_off = o->traj_seg_off; P.turn_scalar = o->turn_scalar; P.turn_step = o->turn_step;
  TokArgs T;
  T.n_tokens = N; T.n_turns = U; T.n_models = K; T.place_mode = r->place_mode; T.grp_shift = gsh;
  T.turn_seg_off = o->turn_seg_off; T.seg_meta = w.seg_meta; T.blk_first = w.blk_first; T.mask_global = tok_mask_global;
  T.blk_count = w.tok_count; T.grp_count = w.tok_count + nbk;
  T.perm = o->perm; T.tok_turn = o->tok_turn; T.tok_role = o->tok_role; T.tok_mask = o->tok_mask;
  T.tok_flags = o->tok_flags; T.tok_reward = o->tok_reward;

  // everything in one launch where the plan fits a workgroup and the thin arrays are little to read for every one of them
  const size_t thin = static_cast<size_t>(reinterpret_cast<char*>(w.plan_part) - ws_base);
  if (N > 0 && N <= kSmallTokens && U <= kSmallTurns && B <= kSmallTraj && n_groups <= kSmallGroups && thin <= kSmallThin &&
      thin * static_cast<size_t>(nbk) <= kSmallBus) {
    SmallArgs A;
    A.plan = P; A.tok = T; A.ws = ws_base; A.thin16 = static_cast<int>(thin / 16); A.n_groups = n_groups; A.norm_eps = r->norm_eps;
    A.group_off = w.group_off; A.group_members = has.members ? w.group_members : nullptr; A.rowsel = o->rowsel;
    A.thin = stage.lend();
    const dim3 grid(static_cast<unsigned>(nbk)), threads(kSmallThreads);
    if (K <= 1) hipLaunchKernelGGL(k_route_small<1>, grid, threads, 0, st, A);
    else if (K <= 2) hipLaunchKernelGGL(k_route_small<2>, grid, threads, 0, st, A);
    else if (K <= 4) hipLaunchKernelGGL(k_route_small<4>, grid, threads, 0, st, A);
    else hipLaunchKernelGGL(k_route_small<UMAS_MAX_MODELS>, grid, threads, 0, st, A);
    vs = stage.launched(st, hipGetLastError());
    if (vs == UMAS_OK && g_prof_on) prof_kernel("k_route_small", st);
    return vs;
  }

  stage.zero(static_cast<size_t>(reinterpret_cast<char*>(w.plan_part) - ws_base),
             sizeof(unsigned long long) * static_cast<size_t>(n_chunks) * kPlanWords);
  vs = stage.flush(workspace, staged_bytes, st);
  if (vs != UMAS_OK) return vs;
  prof_mark(st);

  if (n_groups > 0) {
    hipLaunchKernelGGL(k_group_norm, dim3(cdiv(n_groups, 4)), dim3(256), 0, st, w.traj_reward, w.group_off,
                       has.members ? w.group_members : nullptr, n_groups, r->norm_eps, w.traj_norm);
    UMAS_LAUNCHED("k_group_norm");
    P.traj_reward = w.traj_norm;
  }
  // workgroups of the plan kernel wait for one another's totals: no more of them than the device holds at once
  int dev = 0, n_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
    n_cu = 64;
  const dim3 plan_grid(std::min(n_chunks, (K <= 2 ? kPlanPerCu : 1) * n_cu));
  if (K <= 1) hipLaunchKernelGGL(k_turn_plan<1>, plan_grid, dim3(kPlanThreads), 0, st, P);
  else if (K <= 2) hipLaunchKernelGGL(k_turn_plan<2>, plan_grid, dim3(kPlanThreads), 0, st, P);
  else if (K <= 4) hipLaunchKernelGGL(k_turn_plan<4>, plan_grid, dim3(kPlanThreads), 0, st, P);
  else hipLaunchKernelGGL(k_turn_plan<UMAS_MAX_MODELS>, plan_grid, dim3(kPlanThreads), 0, st, P);
  UMAS_LAUNCHED("k_turn_plan");
  if (U > 0 && N > 0) {
    // Turns of 16 tokens and less on average leave most blocks one token at a time and plain stores (kSegWin).  The instance that knows nothing else needs 38
    // registers, the other 68, of which seven workgroups fit a compute unit and not eight: a last round of them more at many sizes, and no other path to make
    // up for it.  Routing and scan with it and without, turns of 16: 10 million tokens 347 and 342 us, 25 million 671 and 750, 30 million 826 and 892, 40 million 1117 and
    // 1202; of 17 and more the other way round (40 million in turns of 17 603, before 792).  (Held to the 64 registers of eight it spills 12 bytes: 10 million
    // tokens in turns of 256 120 and 115 us.)
    const bool one_by_one = N < (kTokBlock / kSegWin + 1) * static_cast<int64_t>(U);
    if (N >= kPastTokens && !one_by_one) hipLaunchKernelGGL(k_tokens<true>, dim3(static_cast<unsigned>(nbk)), dim3(kTokThreads), 0, st, T);
    else hipLaunchKernelGGL(k_tokens<false>, dim3(static_cast<unsigned>(nbk)), dim3(kTokThreads), 0, st, T);
    UMAS_LAUNCHED("k_tokens");
    SelArgs S;
    S.n_tokens = N; S.n_models = K; S.grp_shift = gsh;
    S.tok_mask = o->tok_mask; S.model_tok_off = o->model_tok_off; S.blk_count = w.tok_count; S.grp_count = w.tok_count + nbk;
    S.rowsel = o->rowsel; S.model_rowsel_off = o->model_rowsel_off;
    hipLaunchKernelGGL(k_rowsel, dim3(cdiv(N, kSelBlock)), dim3(kTokThreads), 0, st, S);
    UMAS_LAUNCHED("k_rowsel");
  }
  return UMAS_OK;
}
