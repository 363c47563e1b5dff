// Ready-batch construction: a model-local buffer becomes a batch ready for the update by dropping
// incomplete trajectories, shuffling, and cutting what is left into minibatches that match the worker
// group's configuration (Section "Model-Local Buffers", B_i -> D_i^ready).
//
// The shuffle is an input (a permutation of the trajectories).  The kept trajectories, in shuffled
// order, are cut into n_minibatch contiguous parts whose sizes differ by at most one; for every model
// and minibatch the scored rows of its trajectories are listed trajectory by trajectory in shuffled
// order, rows of one trajectory in stream order.  All of it is index work on the streams that
// umas_assign_token_rewards wrote: a trajectory's turns are contiguous inside a stream (one "trajectory
// run"), so a run's rows are one slice of rowsel, and minibatches are built by moving slices.
#include <algorithm>
#include <type_traits>
#include <vector>

#include "umas_common.h"

namespace umas {
namespace {

constexpr int kScanItems = 8;
constexpr int kScanTile = 256 * kScanItems;       // entries one workgroup scans at a time
constexpr int kPerCu = 2;                         // workgroups per compute unit of the kernels that wait for one another
constexpr unsigned long long kMark = 1ull << 63;  // ready mark of a published sum

// Sum of the published words part[0 .. n): every thread takes some, a word is taken when its ready mark is set;
// also returns, in *before, the sum of the words part[0 .. upto).  Result in every thread.  Waiting is safe because
// every workgroup publishes all of its words before it reads any, and all workgroups of the grid are resident.
__device__ __forceinline__ int64_t sum_published(unsigned long long* part, int n, int upto, int64_t* smem, int64_t* before) {
  int64_t all = 0, bef = 0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    unsigned long long w;
    while (!((w = __hip_atomic_load(part + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) & kMark)) __builtin_amdgcn_s_sleep(2);
    const int64_t v = static_cast<int64_t>(w & ~kMark);
    all += v;
    bef += i < upto ? v : 0;
  }
  *before = block_sum<int64_t>(bef, smem);
  return block_sum<int64_t>(all, smem);
}

// rank[b] = position of trajectory b among the kept trajectories in shuffled order, or -1; *n_kept = their number.
// Tiles of kScanTile positions of the shuffle; a workgroup publishes the kept count of each of its tiles, then places
// each of them behind the tiles before it.  Also clears what the later kernels add to or wait for: zero_a, zero_b.
__global__ void __launch_bounds__(256)
k_kept_ranks(int n_traj, int ntile, const int32_t* __restrict__ order, const uint8_t* __restrict__ keep,
             unsigned long long* part, int32_t* __restrict__ rank, int64_t* __restrict__ n_kept,
             int64_t* __restrict__ zero_a, int64_t n_zero_a, unsigned long long* __restrict__ zero_b, int64_t n_zero_b) {
  __shared__ int64_t smem[32];
  const int tid = threadIdx.x;
  auto flags_of = [&](int t, int32_t (&b)[kScanItems], int (&f)[kScanItems]) {
    int sum = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      const int q = t * kScanTile + tid * kScanItems + k;
      b[k] = q < n_traj ? (order ? order[q] : q) : -1;
    }
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      f[k] = b[k] >= 0 && (!keep || keep[b[k]]) ? 1 : 0;
      sum += f[k];
    }
    return sum;
  };
  for (int t = blockIdx.x; t < ntile; t += gridDim.x) {
    int32_t b[kScanItems];
    int f[kScanItems];
    const int64_t total = block_sum<int64_t>(flags_of(t, b, f), smem);
    if (tid == 0) __hip_atomic_store(part + t, kMark | static_cast<unsigned long long>(total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  {
    const int64_t gtid = static_cast<int64_t>(blockIdx.x) * blockDim.x + tid, gsize = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = gtid; i < n_zero_a; i += gsize) zero_a[i] = 0;
    for (int64_t i = gtid; i < n_zero_b; i += gsize) zero_b[i] = 0ull;
  }
  for (int t = blockIdx.x; t < ntile; t += gridDim.x) {
    int64_t before;
    const int64_t all = sum_published(part, ntile, t, smem, &before);
    if (t == 0 && tid == 0) *n_kept = all;
    int32_t b[kScanItems];
    int f[kScanItems];
    const int mine = flags_of(t, b, f);
    int32_t total;
    int32_t pos = static_cast<int32_t>(before) + block_excl_scan<int32_t>(mine, reinterpret_cast<int32_t*>(smem), &total);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      if (b[k] >= 0) rank[b[k]] = f[k] ? pos : -1;
      pos += f[k];
    }
  }
}

// First place in rs[0 .. n) that holds at least x, for strictly ascending positions below len: the places of scored tokens in a stream.  A
// probe at g that misses x by e leaves at most |e| places (one position each at least), and the stream's density says where
// among them: three or four probes where masks are alike everywhere, halving after kGuesses where they are not.
constexpr int kGuesses = 8;
__device__ __forceinline__ int64_t first_row_from(const int32_t* __restrict__ rs, int64_t n, int64_t len, int64_t x) {
  int64_t lo = x - (len - n), hi = x < n ? x : n;   // all but len - n positions are there
  lo = lo > 0 ? lo : 0;
  const float density = static_cast<float>(n) / static_cast<float>(len);
  int64_t g = static_cast<int64_t>(static_cast<float>(x) * density);
  for (int k = 0; lo < hi; ++k) {
    g = k >= kGuesses ? (lo + hi) >> 1 : g < lo ? lo : g >= hi ? hi - 1 : g;
    const int64_t e = x - rs[g];
    if (e > 0) {
      lo = g + 1;
      hi = g + e < hi ? g + e : hi;
    } else {
      lo = g + e > lo ? g + e : lo;
      hi = g;
    }
    g += static_cast<int64_t>(static_cast<float>(e) * density);
  }
  return lo;
}
// The trajectory of turn u: last b with off[b] <= u, by the same kind of guesses.
__device__ __forceinline__ int trajectory_of(const int32_t* __restrict__ off, int n_traj, int n_turns, int u) {
  int lo = 0, hi = n_traj;
  const float density = static_cast<float>(n_traj) / static_cast<float>(n_turns);
  int g = static_cast<int>((static_cast<float>(u) + 0.5f) * density);
  for (int k = 0; lo < hi; ++k) {
    // g: a guess at b; off[b] <= u < off[b + 1], two loads of one line
    g = k >= kGuesses ? (lo + hi + 1) >> 1 : g < lo ? lo : g > hi ? hi : g;
    const int here = off[g], next = g < n_traj ? off[g + 1] : INT32_MAX;
    if (here > u) hi = g - 1;
    else if (next > u) return g;
    else lo = g + 1;
    const float e = static_cast<float>(u - here) * density;
    g += static_cast<int>(here > u ? e - 1.f : e + 1.f);
  }
  return lo;
}
// Per trajectory run: its model, trajectory and the slice of rowsel that holds its scored rows; written
// at (model, rank of the trajectory) when the trajectory is kept.  A run's rows end where the next run's of its stream start: a workgroup looks
// for 256 starts and has 255 runs.  (Two binary searches for start and end, the trajectory a third, all advancing in one loop: 25 trips to memory,
// 25.8 us for 32 768 runs and 20 million rows, now 13.2; wider searches were slower, there are as many more scattered loads.)
constexpr int kRunThreads = 256;
__global__ void __launch_bounds__(kRunThreads)
k_run_slices(int n_turns, int n_traj, int n_models, const int64_t* __restrict__ traj_seg_off,
             const int32_t* __restrict__ model_trajrun_off, const int64_t* __restrict__ model_tok_off,
             const int64_t* __restrict__ model_rowsel_off, const int32_t* __restrict__ rowsel,
             const int32_t* __restrict__ tok_turn, const int32_t* __restrict__ traj_turn_off,
             const int32_t* __restrict__ rank, int64_t* __restrict__ cnt_mq, int64_t* __restrict__ src_mq) {
  __shared__ int64_t s_pos[kRunThreads];
  const int j = blockIdx.x * (kRunThreads - 1) + threadIdx.x, n_runs = min(n_turns, model_trajrun_off[n_models]);
  int m = 0;
  int64_t start = 0, row = 0;
  if (j < n_runs) {
    start = traj_seg_off[j];
    while (m + 1 < n_models && model_trajrun_off[m + 1] <= j) ++m;
    const int64_t ra = model_rowsel_off[m], t0 = model_tok_off[m];
    row = ra + first_row_from(rowsel + ra, model_rowsel_off[m + 1] - ra, model_tok_off[m + 1] - t0, start - t0);
    s_pos[threadIdx.x] = row;
  }
  __syncthreads();
  if (j >= n_runs || threadIdx.x == kRunThreads - 1 || traj_seg_off[j + 1] <= start) return;
  const int q = rank[trajectory_of(traj_turn_off, n_traj, n_turns, tok_turn[start])];
  if (q < 0) return;
  const int64_t end = j + 1 < model_trajrun_off[m + 1] ? s_pos[threadIdx.x + 1] : model_rowsel_off[m + 1];
  cnt_mq[static_cast<size_t>(m) * n_traj + q] = end - row;
  src_mq[static_cast<size_t>(m) * n_traj + q] = row;
}

// In-place exclusive prefix sums of the rows of data[n_models][n_traj] (the rows of every model by kept rank), the
// rows' totals, and mb_off[m][k] = rows before minibatch k of model m: minibatch k starts at the first kept
// trajectory q with q * n_minibatch / n_kept >= k, i.e. q = ceil(k n_kept / n_minibatch).  Tiles of kScanTile
// entries of a row; a workgroup publishes the sum of each of its tiles, then places each of them behind the tiles
// before it in its row and the rows before that.
__global__ void __launch_bounds__(256)
k_mb_scan(int n_models, int n_traj, int ntile, int n_minibatch, int balance_rows, const int64_t* __restrict__ n_kept_p,
          int64_t* __restrict__ data, unsigned long long* part, int64_t* __restrict__ totals, int64_t* __restrict__ mb_off) {
  __shared__ int64_t smem[32];
  __shared__ int64_t s_scan[kScanTile];
  const int tid = threadIdx.x;
  const int n_all = n_models * ntile;
  for (int t = blockIdx.x; t < n_all; t += gridDim.x) {
    const int64_t* row = data + static_cast<size_t>(t / ntile) * n_traj;
    const int base = (t % ntile) * kScanTile + tid * kScanItems;
    int64_t sum = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) sum += base + k < n_traj ? row[base + k] : 0;
    const int64_t total = block_sum<int64_t>(sum, smem);
    if (tid == 0) __hip_atomic_store(part + t, kMark | static_cast<unsigned long long>(total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const int64_t n_kept = *n_kept_p;
  for (int t = blockIdx.x; t < n_all; t += gridDim.x) {
    const int m = t / ntile, tile0 = (t % ntile) * kScanTile;
    int64_t before_row, in_row_before;
    const int64_t row_total = sum_published(part + static_cast<size_t>(m) * ntile, ntile, t % ntile, smem, &in_row_before);
    (void)sum_published(part, m * ntile, m * ntile, smem, &before_row);   // the rows of the models before m
    int64_t* row = data + static_cast<size_t>(m) * n_traj;
    const int base = tile0 + tid * kScanItems;
    int64_t v[kScanItems];
    int64_t sum = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      v[k] = base + k < n_traj ? row[base + k] : 0;
      sum += v[k];
    }
    int64_t total;
    int64_t r = in_row_before + block_excl_scan<int64_t>(sum, smem, &total);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      if (base + k < n_traj) row[base + k] = r;
      s_scan[tid * kScanItems + k] = r;
      r += v[k];
    }
    __syncthreads();
    if (t % ntile == 0 && tid == 0) totals[m] = row_total;
    for (int k = tid; k <= n_minibatch; k += blockDim.x) {
      int64_t* out = mb_off + static_cast<size_t>(m) * (n_minibatch + 1) + k;
      if (balance_rows) {
        // cut by rows: part k starts at the first trajectory whose first row is at or behind ceil(k T / M); the tile
        // whose prefix sums first reach the threshold writes it (the first tile when the threshold is 0)
        const int64_t thr = (static_cast<int64_t>(k) * row_total + n_minibatch - 1) / n_minibatch;
        const int len = n_traj - tile0 < kScanTile ? n_traj - tile0 : kScanTile;   // entries of the tile that exist
        if (thr <= in_row_before ? tile0 == 0 : thr <= in_row_before + total) {
          int lo = 0, hi = len;                          // first entry of the tile at or above the threshold, len if none
          while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (s_scan[mid] < thr) lo = mid + 1; else hi = mid;
          }
          *out = before_row + (lo < len ? s_scan[lo] : in_row_before + total);
        }
        continue;
      }
      const int64_t q = (static_cast<int64_t>(k) * n_kept + n_minibatch - 1) / n_minibatch;
      if (k == n_minibatch || q >= n_kept) {
        if (t % ntile == 0) *out = before_row + row_total;
      } else if (q >= tile0 && q < tile0 + kScanTile) {
        *out = before_row + s_scan[q - tile0];
      }
    }
    __syncthreads();                                // s_scan and smem are the next tile's
  }
}

// One wavefront per (model, kept trajectory): its rowsel slice goes to its place in mb_rowsel, 16 bytes at a time from the first 16-byte boundary there
// on (at any 4-byte boundary of rowsel).  A slice is a few hundred entries, so a wavefront's time is its chain of loads: what says where
// the slice lies is asked for together, whether the trajectory was kept or not, and so are a slice's whole vectors and its ends; slices of up to a
// wavefront's entries have only ends.  36 million tokens in trajectories of 101, 202, 280, 420, 616 and 2800 scored ones, 4 bytes at a time 69,
// 55.5, 48.5, 43.7, 40.3 and 40.5 us, 16 bytes and the ends with trips of their own 74, 49.5, 41.3, 35.3, 33.9 and 35.6, now 61.6, 41.7, 36, 35,
// 34.8 and 36.2; 18 million in trajectories of 50 54.5, 62 and 48.5; 4 million of 11 47, 54.6 and 39.7.
__global__ void __launch_bounds__(256)
k_mb_copy(int n_models, int n_traj, const int64_t* __restrict__ n_kept_p, const int64_t* __restrict__ scan_mq,
          const int64_t* __restrict__ src_mq, const int64_t* __restrict__ totals, const int32_t* __restrict__ rowsel,
          int32_t* __restrict__ mb_rowsel) {
  typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
  typedef int32_t i32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
  const int lane = threadIdx.x & (kWave - 1);
  int64_t q = static_cast<int64_t>(blockIdx.x) * (blockDim.x / kWave) + __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  if (q >= static_cast<int64_t>(n_models) * n_traj) return;
  const size_t at = static_cast<size_t>(q);
  int m = 0;
  int64_t base = 0;
  for (; q >= n_traj; q -= n_traj) base += totals[m++];
  const int64_t n_kept = *n_kept_p, first = scan_mq[at], next = q + 1 < n_traj ? scan_mq[at + 1] : totals[m];
  const int32_t* const src = rowsel + src_mq[at];
  if (q >= n_kept) return;
  const int64_t len = next - first;
  int32_t* const dst = mb_rowsel + base + first;
  if (len <= kWave) {
    if (lane < len) dst[lane] = src[lane];
    return;
  }
  const int64_t off = static_cast<int64_t>((16 - (reinterpret_cast<uintptr_t>(dst) & 15)) & 15) / 4, head = off < len ? off : len;
  const int64_t n4 = (len - head) / 4, tail = head + n4 * 4;
  int32_t first_entry = 0, last_entry = 0;                   // up to three in front of the whole vectors, up to three behind
  if (lane < head) first_entry = src[lane];
  if (tail + lane < len) last_entry = src[tail + lane];
  const i32x4_a4* const src4 = reinterpret_cast<const i32x4_a4*>(src + head);
  i32x4* const dst4 = reinterpret_cast<i32x4*>(dst + head);
  for (int64_t i0 = lane; i0 < n4; i0 += 4 * kWave) {        // four loads in flight per lane
    i32x4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (i0 + k * kWave < n4) v[k] = src4[i0 + k * kWave];
    if (i0 == lane) {                                        // (a slice has 15 vectors here at least)
      if (lane < head) dst[lane] = first_entry;
      if (tail + lane < len) dst[tail + lane] = last_entry;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (i0 + k * kWave < n4) dst4[i0 + k * kWave] = v[k];
  }
}

// Parts under a budget of scored rows, one wavefront per model: starting from the model's first row, a part ends at
// the last trajectory boundary within max_rows rows of its start, or, when not even the first trajectory fits, behind
// that trajectory.  scan_mq holds the model's rows before each kept trajectory (kept rank order), so a boundary is found
// by one wavefront-wide search per part (one trip to memory where trajectories are alike: 9 parts of 32 768 trajectories 13.7 us, now 10.3); every part holds at least one row, so the walk ends after at most as many
// steps as the model has rows.  Entries of the offsets past the last part repeat the model's end.
constexpr int kPackThreads = 1024;
__global__ void __launch_bounds__(kPackThreads)
k_mb_pack(int n_traj, int64_t max_rows, const int64_t* __restrict__ n_kept_p, const int64_t* __restrict__ scan_mq,
          const int64_t* __restrict__ totals, int64_t* __restrict__ mb_off, int32_t* __restrict__ n_parts) {
  __shared__ int s_parts;
  const int m = blockIdx.x, tid = threadIdx.x;
  const int n_kept = static_cast<int>(*n_kept_p);
  const int64_t* row = scan_mq + static_cast<size_t>(m) * n_traj;
  const int64_t total = totals[m];
  int64_t base = 0;
  for (int mm = 0; mm < m; ++mm) base += totals[mm];
  int64_t* out = mb_off + static_cast<size_t>(m) * (static_cast<size_t>(n_traj) + 1);
  if (tid < kWave) {                                 // the walk is one wavefront's; the others help with the tail afterwards
    if (tid == 0) out[0] = base;
    int k = 0;
    int64_t at = 0;                                  // first row of the open part, relative to the model's first
    int j0 = 0;                                      // a kept trajectory with row[j0] == at
    const double per_row = static_cast<double>(n_kept) / static_cast<double>(total);   // trajectories
    while (at < total) {                             // n_kept >= 1 here
      const int64_t limit = at + max_rows;
      int64_t end = total;
      if (total > limit) {
        // largest j with row[j] <= limit: first among 256 entries around where it lies if trajectories are alike, no further back
        // than j0 (one trip; row[j0] = at <= limit), then, if it is not one of them, by the general search on its side of them
        const double guess = static_cast<double>(j0) + static_cast<double>(max_rows) * per_row - 2 * kWave;
        const int b0 = guess > j0 ? guess < n_kept ? static_cast<int>(guess) : n_kept - 1 : j0;
        int64_t v[4];
        int c = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = b0 + tid + q * kWave < n_kept ? row[b0 + tid + q * kWave] : INT64_MAX;
#pragma unroll
        for (int q = 0; q < 4; ++q) c += __popcll(__ballot(v[q] <= limit));
        int j;
        if (c > 0 && c < 4 * kWave) {
          j = b0 + c - 1;
          const int64_t mine = (c - 1) >> 6 == 0 ? v[0] : (c - 1) >> 6 == 1 ? v[1] : (c - 1) >> 6 == 2 ? v[2] : v[3];
          end = __shfl(mine, (c - 1) & (kWave - 1), kWave);
        } else {
          const int from = c == 0 ? j0 : b0 + 4 * kWave - 1, upto = c == 0 ? b0 : n_kept - 1;   // row[from] <= limit either way
          j = from + wave_last_le(row + from, upto - from, limit);
          end = row[j];
        }
        if (end == at) {                             // the trajectory at the part's start is over the budget by itself
          ++j;
          end = j < n_kept ? row[j] : total;
        }
        j0 = j;
      }
      ++k;
      if (tid == 0) out[k] = base + end;
      at = end;
    }
    if (tid == 0) { n_parts[m] = k; s_parts = k; }
  }
  __syncthreads();
  for (int64_t i = s_parts + 1 + tid; i <= n_traj; i += kPackThreads) out[i] = base + total;
}

// ------------------------------------------------------------------ small batches: everything in one launch
// Up to 256 trajectories the five kernels above and the copy in front of them are launches of 4 to 9 us each, on the device and on the
// host, for a few KB of index work.  Here every workgroup reads the thin arrays from the pinned block itself, makes ranks, slices
// and prefix sums in LDS, and moves its share of the slices, several wavefronts to a slice; the first one writes the offsets instead.
// 32 trajectories, 28 000 rows, packed: 33 us in six launches, 9.3 in one (10 with the thin arrays waited for first), and 26 and 8.5 us of the host.
constexpr int kSmallThreads = 1024;
constexpr int kSmallTraj = 256;
constexpr int kSmallSlices = 1024;                  // models times trajectories
constexpr int kSmallTurns = 1024;                   // runs are no more than turns; at least one lane searches for each
constexpr size_t kSmallThin = 4 * 1024;
constexpr unsigned kSmallMovers = 16;               // workgroups that move slices, and as many more as make a wavefront for each
static_assert(kSmallTraj * 9 + 4 + 3 * kAlign <= kSmallThin && kSmallThin <= 16 * kSmallThreads, "offsets, order and flags, 16 bytes a thread");

struct SmallArgs {
  const char* thin;
  int thin16, at_order, at_keep;                    // byte offsets in the block, -1: none; traj_turn_off is at 0
  int n_turns, n_traj, n_models, n_minibatch, balance_rows;
  int64_t max_rows;                                 // packed parts when n_parts is given
  const int64_t* traj_seg_off;
  const int32_t* model_trajrun_off;
  const int64_t* model_tok_off;
  const int64_t* model_rowsel_off;
  const int32_t* rowsel;
  const int32_t* tok_turn;
  int32_t* mb_rowsel;
  int64_t* mb_off;
  int32_t* n_parts;
};

// First place in rs[0 .. n) that holds at least x, by G lanes next to each other that probe G places a round.  (Guesses like first_row_from's, a run to a
// thread, take more rounds than this with sixteen lanes has: 12.0 us against 9.3.)
template <int G>
__device__ __forceinline__ int64_t first_at_least(const int32_t* __restrict__ rs, int64_t n, int64_t x) {
  const int lane = threadIdx.x & (kWave - 1), mine = lane & (G - 1), shift = lane - mine;
  int64_t lo = 0, hi = n;
  while (lo < hi) {                                 // the same for the G lanes
    auto probe = [&](int i) { return lo + (hi - lo) * (i + 1) / (G + 1); };
    const unsigned long long below = __ballot(rs[probe(mine)] < x);
    const int c = __popcll((below >> shift) & ((1ull << G) - 1));   // the first c probes hold less
    const int64_t next_hi = c < G ? probe(c) : hi;
    lo = c > 0 ? probe(c - 1) + 1 : lo;
    hi = next_hi;
  }
  return lo;
}

__global__ void __launch_bounds__(kSmallThreads)
k_ready_small(SmallArgs A) {
  constexpr int nwave = kSmallThreads / kWave;
  __shared__ __attribute__((aligned(16))) char s_thin[kSmallThin];
  __shared__ int64_t s_tok[UMAS_MAX_MODELS + 1], s_sel[UMAS_MAX_MODELS + 1];   // where the streams' tokens and scored rows start
  __shared__ int32_t s_run[UMAS_MAX_MODELS + 1];    // ... and their runs
  __shared__ int32_t s_rank[kSmallTraj];
  __shared__ int64_t s_pos[kSmallTurns];            // first row of every run
  __shared__ int64_t s_row[kSmallSlices + 1];       // rows of every (model, kept trajectory), then the rows before it
  __shared__ int64_t s_src[kSmallSlices];
  __shared__ int64_t s_wave[nwave];
  __shared__ int s_kept[kSmallTraj / kWave];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int B = A.n_traj, K = A.n_models, n_mq = K * B;
  // the thin arrays are on their way over the bus while the runs are searched, which needs none of them; the last wavefronts ask for
  // them, for whose loads come back in order and few runs leave these nothing to search
  const int t16 = kSmallThreads - 1 - tid;
  uint4 thin = make_uint4(0u, 0u, 0u, 0u);
  if (t16 < A.thin16) thin = reinterpret_cast<const uint4*>(A.thin)[t16];
  if (tid <= K) {
    s_tok[tid] = A.model_tok_off[tid];
    s_sel[tid] = A.model_rowsel_off[tid];
    s_run[tid] = A.model_trajrun_off[tid];
  }
  if (tid < n_mq) s_row[tid] = 0;
  __syncthreads();
  // ---- first rows of the runs: as many lanes to a run as there are
  const int n_runs = s_run[K] < A.n_turns ? s_run[K] : A.n_turns;
  auto model_of_run = [&](int j) {
    int m = 0;
    while (m + 1 < K && s_run[m + 1] <= j) ++m;
    return m;
  };
  auto search = [&](auto lanes) {
    constexpr int G = decltype(lanes)::value;
    const int j = tid / G;
    if (j >= n_runs) return;
    const int m = model_of_run(j);
    const int64_t ra = s_sel[m];
    const int64_t lo = first_at_least<G>(A.rowsel + ra, s_sel[m + 1] - ra, A.traj_seg_off[j] - s_tok[m]);
    if ((tid & (G - 1)) == 0) s_pos[j] = ra + lo;
  };
  if (n_runs <= kSmallThreads / 16) search(std::integral_constant<int, 16>());
  else if (n_runs <= kSmallThreads / 4) search(std::integral_constant<int, 4>());
  else search(std::integral_constant<int, 1>());
  int64_t start = 0, end = 0;                       // this thread's run
  int turn = 0;
  if (tid < n_runs) {
    start = A.traj_seg_off[tid];
    end = A.traj_seg_off[tid + 1];
    if (end > start) turn = A.tok_turn[start];
  }
  if (t16 < A.thin16) reinterpret_cast<uint4*>(s_thin)[t16] = thin;
  __syncthreads();
  const int32_t* const tto = reinterpret_cast<const int32_t*>(s_thin);
  // ---- ranks of the kept trajectories in shuffled order
  int b = -1;
  bool kept = false;
  int pos = 0;
  if (wave < kSmallTraj / kWave) {
    if (tid < B) {
      b = A.at_order >= 0 ? reinterpret_cast<const int32_t*>(s_thin + A.at_order)[tid] : tid;
      kept = A.at_keep < 0 || reinterpret_cast<const uint8_t*>(s_thin + A.at_keep)[b] != 0;
    }
    const unsigned long long k = __ballot(kept);
    pos = __popcll(k & ((1ull << lane) - 1));
    if (lane == 0) s_kept[wave] = __popcll(k);
  }
  __syncthreads();
  int n_kept = 0;
  for (int w = 0; w < kSmallTraj / kWave; ++w) {
    pos += w < wave ? s_kept[w] : 0;
    n_kept += s_kept[w];
  }
  if (b >= 0) s_rank[b] = kept ? pos : -1;
  __syncthreads();
  // ---- the slice of every run whose trajectory is kept
  if (end > start) {
    const int m = model_of_run(tid);
    const int q = s_rank[last_le(tto, B, turn)];
    if (q >= 0) {
      s_row[m * B + q] = (tid + 1 < s_run[m + 1] ? s_pos[tid + 1] : s_sel[m + 1]) - s_pos[tid];
      s_src[m * B + q] = s_pos[tid];
    }
  }
  __syncthreads();
  // ---- the rows before every slice; entries past the kept ones hold nothing
  {
    const int64_t v = tid < n_mq ? s_row[tid] : 0;
    int64_t before = wave_incl_scan(v);
    if (lane == kWave - 1) s_wave[wave] = before;
    __syncthreads();
    before -= v;
    int64_t total = 0;
#pragma unroll
    for (int w = 0; w < nwave; ++w) {
      before += w < wave ? s_wave[w] : 0;
      total += s_wave[w];
    }
    if (tid < n_mq) s_row[tid] = before;
    if (tid == 0) s_row[n_mq] = total;
    __syncthreads();
  }
  if (blockIdx.x > 0) {                             // move slices
    const int movers = (static_cast<int>(gridDim.x) - 1) * nwave, per = movers / n_mq > 1 ? movers / n_mq : 1;
    const int w = (static_cast<int>(blockIdx.x) - 1) * nwave + wave;
    for (int at = w / per; at < n_mq; at += movers / per) {
      const int64_t dst = s_row[at], len = s_row[at + 1] - dst;
      if (len <= 0) continue;
      const int64_t src = s_src[at];
      for (int64_t i0 = (w % per) * (4 * kWave) + lane; i0 < len; i0 += per * (4 * kWave)) {   // four loads in flight per lane
        int32_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = i0 + k * kWave < len ? A.rowsel[src + i0 + k * kWave] : 0;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (i0 + k * kWave < len) A.mb_rowsel[dst + i0 + k * kWave] = v[k];
      }
    }
    return;
  }
  if (A.n_parts) {                                  // parts under a row budget, a wavefront per model (see k_mb_pack)
    if (wave >= K) return;
    const int64_t* const row = s_row + wave * B;    // row[B]: the model's end
    const int64_t end = row[B];
    int64_t* const out = A.mb_off + static_cast<size_t>(wave) * (static_cast<size_t>(B) + 1);
    if (lane == 0) out[0] = row[0];
    int k = 0;
    for (int64_t at = row[0]; at < end;) {
      int64_t to = end;
      if (end - at > A.max_rows) {
        int j = wave_last_le(row, n_kept - 1, at + A.max_rows);   // row[0] <= at
        if (row[j] == at) ++j;                      // the trajectory at the part's start is over the budget by itself
        to = j < n_kept ? row[j] : end;
      }
      ++k;
      if (lane == 0) out[k] = to;
      at = to;
    }
    if (lane == 0) A.n_parts[wave] = k;
    for (int i = k + 1 + lane; i <= B; i += kWave) out[i] = end;
    return;
  }
  const int64_t M = A.n_minibatch;
  for (int64_t i = tid; i < K * (M + 1); i += kSmallThreads) {
    const int64_t m = i / (M + 1), k = i % (M + 1);
    const int64_t* const row = s_row + m * B;
    const int64_t first = row[0], total = row[B] - first;
    int64_t q;
    if (A.balance_rows) {                           // the first trajectory whose first row is at or behind ceil(k T / M)
      const int64_t thr = first + (k * total + M - 1) / M;
      int lo = 0, hi = B;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (row[mid] < thr) lo = mid + 1; else hi = mid;
      }
      q = lo;
    } else {                                        // ceil(k n_kept / M)
      q = (k * n_kept + M - 1) / M;
      if (k == M || q >= n_kept) q = B;
    }
    A.mb_off[i] = row[q];
  }
}

struct BatchWs {
  int32_t* traj_turn_off;
  int32_t* order;
  uint8_t* keep;
  unsigned long long* part_q;   // [tiles] kept counts of the tiles of the shuffle; zeros come with the staged copy
  int32_t* rank;
  int64_t* n_kept;
  unsigned long long* part_mq;  // [n_models][tiles] sums of the tiles of cnt_mq
  int64_t* cnt_mq;   // [n_models][n_traj], scanned in place
  int64_t* src_mq;   // [n_models][n_traj]
  int64_t* totals;   // [n_models]
  int64_t* one_off;  // [n_models][2] the scan kernel's offsets when the parts are cut by k_mb_pack
};
inline int scan_tiles(int n_traj) { return static_cast<int>(cdiv(n_traj > 0 ? n_traj : 1, kScanTile)); }
size_t carve_batch(Carver& c, BatchWs& w, int n_traj, int n_models) {
  w.traj_turn_off = c.take<int32_t>(static_cast<size_t>(n_traj) + 1);
  w.order = c.take<int32_t>(n_traj);
  w.keep = c.take<uint8_t>(n_traj);
  w.part_q = c.take<unsigned long long>(scan_tiles(n_traj));
  w.rank = c.take<int32_t>(n_traj);
  w.n_kept = c.take<int64_t>(1);
  w.part_mq = c.take<unsigned long long>(static_cast<size_t>(n_models) * scan_tiles(n_traj));
  w.cnt_mq = c.take<int64_t>(static_cast<size_t>(n_models) * n_traj);
  w.src_mq = c.take<int64_t>(static_cast<size_t>(n_models) * n_traj);
  w.totals = c.take<int64_t>(n_models);
  w.one_off = c.take<int64_t>(2 * static_cast<size_t>(n_models));
  return c.off;
}

}  // namespace
}  // namespace umas

using namespace umas;

extern "C" size_t umas_ready_batch_workspace_bytes(int32_t n_traj, int32_t n_models) {
  if (n_traj < 0 || n_models < 1) return 0;
  Carver c(nullptr);
  BatchWs w;
  return carve_batch(c, w, n_traj, n_models);
}

namespace {
umas_status ready_batch(const umas_streams* s, int32_t n_models, int32_t n_turns, const int32_t* traj_turn_off, int32_t n_traj,
                        const uint8_t* traj_keep, const int32_t* traj_order, int32_t n_minibatch, int balance_rows,
                        int64_t max_rows, int32_t* n_parts, int32_t* mb_rowsel, int64_t* mb_off, void* workspace,
                        size_t workspace_bytes, void* hip_stream) {
  const bool packed = n_parts != nullptr;           // parts under a row budget instead of n_minibatch parts
  UMAS_REQUIRE(!packed || max_rows >= 1, UMAS_EINVAL, "max_rows=%lld must be at least 1", static_cast<long long>(max_rows));
  if (max_rows > (int64_t{1} << 62)) max_rows = int64_t{1} << 62;   // more than any batch holds; keeps start + budget inside int64
  UMAS_REQUIRE(s && s->traj_seg_off && s->model_trajrun_off && s->model_tok_off && s->model_rowsel_off && s->rowsel && s->tok_turn,
               UMAS_EINVAL, "streams lacks traj_seg_off, model_trajrun_off, model_tok_off, model_rowsel_off, rowsel or tok_turn");
  UMAS_REQUIRE(n_models >= 1 && n_models <= UMAS_MAX_MODELS, UMAS_ESHAPE, "n_models=%d outside [1,%d]", n_models, UMAS_MAX_MODELS);
  UMAS_REQUIRE(n_traj >= 0 && n_turns >= 0, UMAS_EINVAL, "negative size");
  UMAS_REQUIRE(n_minibatch >= 1, UMAS_EINVAL, "n_minibatch=%d must be at least 1", n_minibatch);
  UMAS_REQUIRE(traj_turn_off && mb_off && (mb_rowsel || n_turns == 0), UMAS_EINVAL, "traj_turn_off, mb_rowsel and mb_off must not be NULL");
  UMAS_REQUIRE(traj_turn_off[0] == 0 && traj_turn_off[n_traj] == n_turns, UMAS_EINVAL, "traj_turn_off must run from 0 to n_turns");
  for (int b = 0; b < n_traj; ++b)
    UMAS_REQUIRE(traj_turn_off[b] <= traj_turn_off[b + 1], UMAS_EINVAL, "traj_turn_off decreases at %d", b);
  if (traj_order) {                                  // a permutation of the trajectories
    std::vector<uint8_t> seen(static_cast<size_t>(n_traj), 0);
    for (int q = 0; q < n_traj; ++q) {
      const int b = traj_order[q];
      UMAS_REQUIRE(b >= 0 && b < n_traj && !seen[b], UMAS_EINVAL, "traj_order is not a permutation (entry %d = %d)", q, b);
      seen[b] = 1;
    }
  }
  const size_t need = umas_ready_batch_workspace_bytes(n_traj, n_models);
  UMAS_REQUIRE(workspace && reinterpret_cast<uintptr_t>(workspace) % kAlign == 0 && workspace_bytes >= need, UMAS_EWORKSPACE,
               "workspace must be 256-byte aligned and hold %zu bytes (got %zu)", need, workspace_bytes);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  prof_mark(st);
  Carver c(workspace);
  BatchWs w;
  carve_batch(c, w, n_traj, n_models);
  // the thin arrays (the first arrays of the workspace, up to rank) go through pinned staging memory, from where one
  // kernel takes them over the bus, together with the zeros that the first kernel's tile counts start from: they have been
  // read when the call returns, and the host does not wait for the stream
  char* const ws_base = static_cast<char*>(workspace);
  const size_t staged_bytes = static_cast<size_t>(reinterpret_cast<char*>(w.rank) - ws_base);
  const int ntile = scan_tiles(n_traj);
  ThinStage stage;
  umas_status vs = stage.begin(staged_bytes, st);
  if (vs != UMAS_OK) return vs;
  stage.put(static_cast<size_t>(reinterpret_cast<char*>(w.traj_turn_off) - ws_base), traj_turn_off, (static_cast<size_t>(n_traj) + 1) * sizeof(int32_t));
  stage.put(static_cast<size_t>(reinterpret_cast<char*>(w.order) - ws_base), traj_order, static_cast<size_t>(n_traj) * sizeof(int32_t));
  stage.put(static_cast<size_t>(reinterpret_cast<char*>(w.keep) - ws_base), traj_keep, static_cast<size_t>(n_traj));
  const int64_t n_mq = static_cast<int64_t>(n_models) * n_traj;
  if (n_turns > 0 && n_turns <= kSmallTurns && n_traj <= kSmallTraj && n_mq <= kSmallSlices) {
    SmallArgs A;
    A.thin16 = static_cast<int>((reinterpret_cast<char*>(w.part_q) - ws_base) / 16);
    A.at_order = traj_order ? static_cast<int>(reinterpret_cast<char*>(w.order) - ws_base) : -1;
    A.at_keep = traj_keep ? static_cast<int>(reinterpret_cast<char*>(w.keep) - ws_base) : -1;
    A.n_turns = n_turns; A.n_traj = n_traj; A.n_models = n_models; A.n_minibatch = n_minibatch; A.balance_rows = balance_rows;
    A.max_rows = max_rows;
    A.traj_seg_off = s->traj_seg_off; A.model_trajrun_off = s->model_trajrun_off; A.model_tok_off = s->model_tok_off;
    A.model_rowsel_off = s->model_rowsel_off; A.rowsel = s->rowsel; A.tok_turn = s->tok_turn;
    A.mb_rowsel = mb_rowsel; A.mb_off = mb_off; A.n_parts = n_parts;
    const unsigned grid = 1 + std::max(kSmallMovers, cdiv(static_cast<size_t>(n_mq), kSmallThreads / kWave));
    A.thin = stage.lend();
    hipLaunchKernelGGL(k_ready_small, dim3(grid), dim3(kSmallThreads), 0, st, A);
    vs = stage.launched(st, hipGetLastError());
    if (vs == UMAS_OK && g_prof_on) prof_kernel("k_ready_small", st);
    return vs;
  }
  stage.zero(static_cast<size_t>(reinterpret_cast<char*>(w.part_q) - ws_base), static_cast<size_t>(ntile) * sizeof(unsigned long long));
  vs = stage.flush(workspace, staged_bytes, st);
  if (vs != UMAS_OK) return vs;
  prof_mark(st);

  // workgroups of the two scanning kernels wait for one another's sums: no more of them than the device holds at once
  int dev = 0, n_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
    n_cu = 64;
  const int32_t* d_order = traj_order ? w.order : nullptr;
  const uint8_t* d_keep = traj_keep ? w.keep : nullptr;
  hipLaunchKernelGGL(k_kept_ranks, dim3(std::min(ntile, kPerCu * n_cu)), dim3(256), 0, st, n_traj, ntile, d_order, d_keep, w.part_q,
                     w.rank, w.n_kept, w.cnt_mq, n_mq, w.part_mq, static_cast<int64_t>(n_models) * ntile);
  UMAS_LAUNCHED("k_kept_ranks");
  if (n_turns > 0 && n_traj > 0) {
    hipLaunchKernelGGL(k_run_slices, dim3(cdiv(n_turns, kRunThreads - 1)), dim3(kRunThreads), 0, st, n_turns, n_traj, n_models, s->traj_seg_off,
                       s->model_trajrun_off, s->model_tok_off, s->model_rowsel_off, s->rowsel, s->tok_turn, w.traj_turn_off,
                       w.rank, w.cnt_mq, w.src_mq);
    UMAS_LAUNCHED("k_run_slices");
  }
  hipLaunchKernelGGL(k_mb_scan, dim3(std::min(n_models * ntile, kPerCu * n_cu)), dim3(256), 0, st, n_models, n_traj, ntile,
                     packed ? 1 : n_minibatch, balance_rows, w.n_kept, w.cnt_mq, w.part_mq, w.totals, packed ? w.one_off : mb_off);
  UMAS_LAUNCHED("k_mb_scan");
  if (packed) {
    hipLaunchKernelGGL(k_mb_pack, dim3(n_models), dim3(kPackThreads), 0, st, n_traj, max_rows, w.n_kept, w.cnt_mq, w.totals, mb_off, n_parts);
    UMAS_LAUNCHED("k_mb_pack");
  }
  if (n_mq > 0) {
    hipLaunchKernelGGL(k_mb_copy, dim3(cdiv(n_mq, 4)), dim3(256), 0, st, n_models, n_traj, w.n_kept, w.cnt_mq, w.src_mq,
                       w.totals, s->rowsel, mb_rowsel);
    UMAS_LAUNCHED("k_mb_copy");
  }
  return UMAS_OK;
}
}  // namespace

extern "C" umas_status umas_ready_batch(const umas_streams* s, int32_t n_models, int32_t n_turns,
                                        const int32_t* traj_turn_off, int32_t n_traj, const uint8_t* traj_keep,
                                        const int32_t* traj_order, int32_t n_minibatch, int32_t* mb_rowsel,
                                        int64_t* mb_off, void* workspace, size_t workspace_bytes, void* hip_stream) {
  return ready_batch(s, n_models, n_turns, traj_turn_off, n_traj, traj_keep, traj_order, n_minibatch, 0, 0, nullptr, mb_rowsel, mb_off,
                     workspace, workspace_bytes, hip_stream);
}

extern "C" umas_status umas_ready_batch_balanced(const umas_streams* s, int32_t n_models, int32_t n_turns,
                                                 const int32_t* traj_turn_off, int32_t n_traj, const uint8_t* traj_keep,
                                                 const int32_t* traj_order, int32_t n_minibatch, int32_t* mb_rowsel,
                                                 int64_t* mb_off, void* workspace, size_t workspace_bytes, void* hip_stream) {
  return ready_batch(s, n_models, n_turns, traj_turn_off, n_traj, traj_keep, traj_order, n_minibatch, 1, 0, nullptr, mb_rowsel, mb_off,
                     workspace, workspace_bytes, hip_stream);
}

extern "C" umas_status umas_ready_batch_packed(const umas_streams* s, int32_t n_models, int32_t n_turns,
                                               const int32_t* traj_turn_off, int32_t n_traj, const uint8_t* traj_keep,
                                               const int32_t* traj_order, int64_t max_rows, int32_t* mb_rowsel,
                                               int64_t* mb_off, int32_t* n_parts, void* workspace, size_t workspace_bytes,
                                               void* hip_stream) {
  UMAS_REQUIRE(n_parts, UMAS_EINVAL, "n_parts must not be NULL");
  return ready_batch(s, n_models, n_turns, traj_turn_off, n_traj, traj_keep, traj_order, 1, 0, max_rows, n_parts, mb_rowsel, mb_off,
                     workspace, workspace_bytes, hip_stream);
}
