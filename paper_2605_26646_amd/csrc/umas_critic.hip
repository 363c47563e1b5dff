// Critic: value head V = w . h + b on the selected rows, clipped value loss and its backward.
//
// The worker groups of Section "PPO-Style Training Loop" compute value estimates next to the
// log-probs and update "actor and critic" from the ready batch.  The paper prints no value loss; the
// clipped form used with PPO is taken:
//   Vc = clip(V, V_old - eps, V_old + eps);  L = 1/2 max((V - R)^2, (Vc - R)^2);  loss = mean L
//   g = dloss/dV = (V - R) / S where the unclipped term is the larger one (ties included), else 0
//   dH_i = g_i w,  dw = sum_i g_i h_i,  db = sum_i g_i
// The whole step is one pass over H: one wavefront per row keeps the row in registers, forms the dot
// product and the row's g, writes dH and adds g h to its dw accumulators; the next row is already in
// flight.  dH leaves past the caches: nothing here reads it, and the rows of H that the value pass has just read stay in the
// memory-side cache (values and update, 39 224 rows of 2048 125 -> 119 us on new rows, 112 -> 99 on the rows of the pass
// before; 60 000 float32 rows of 1024 177 -> 153).  Who reads dH next does not pay for it: with a kernel behind them that multiplies dH by H,
// 1000 rows of 2048 30.4 and 30.4 us, 6000 49 and 48, 39 224 221 and 204, 100 000 543 and 522; with a product of dH by 512 columns
// 47 and 47, 61.5 and 62, 219 and 209, 505 and 497.  A workgroup's partial sums meet in LDS, the workgroups' in one small kernel,
// both in a fixed order, so results do not depend on scheduling.
#include <type_traits>

#include <algorithm>

#include "umas_common.h"

namespace umas {
namespace {

constexpr int kVT = 256;                 // threads per workgroup
constexpr int kVWaves = kVT / kWave;
constexpr int kMaxKV = 16;               // 16-byte column vectors per lane: d <= 64 * 16 * (8 bf16 | 4 float)
constexpr unsigned kMaxGrid = 1024;      // workgroups of the row kernel at most (the launch takes no more than are resident at once)
// Rows of 768 bytes to 2 KB, two vectors a lane: three workgroups to a compute unit, those that clear among them.  640 of rows and 128 that clear against 1024 and 128, four
// and a half, values and update: 12 000 rows of 512 bf16 columns 27.9 and 26.7 us, 40 000 45.5 and 42.1, 18 000 of 896 38.6 and 36.7, 40 000 58.8
// and 56, 40 000 of 1024 62.4 and 59.7, 70 000 92.4 and 88.7, 40 000 float32 rows of 256 45.8 and 42, of 512 60.2 and 59.1 (with
// one row in flight 40 000 of 896 57, of 1024 61.2); 640 and 64, 96, 192, 256 for 40 000 of 896 61.2, 55.8, 60.2 and 59.8.  Shorter
// rows are bound by what a wavefront does for one, not by memory: the update of all of 250 000 of 256 columns 73.4 us with 768, 68.3 with 1024, of 384 73.8
// and 76.7.
constexpr unsigned kShortRowsGrid = 768;
constexpr int kVStat = 4;                // (sum L, clipped rows, sum V, rows)
__host__ __device__ constexpr int part_pitch(int d) { return (d + 1 + 15) / 16 * 16; }   // floats of a partial row: dw, then db

__device__ __forceinline__ uint16_t f2bf(float x) { return __builtin_bit_cast(uint16_t, static_cast<__bf16>(x)); }

// Sums over a row and over rows: float for bf16 inputs (every product is exact in float), float64 for float32
// inputs, whose bar is 1e-5 and whose speed does not matter (a float sum of d float32 products loses up to
// d 2^-24 of the sum of their magnitudes, which the difference V - R then magnifies).
template <typename T> using AccT = std::conditional_t<std::is_same<T, float>::value, double, float>;

// 16 bytes of a row as floats: 8 bf16 or 4 float
template <typename T> struct Vec;
template <> struct Vec<uint16_t> {
  static constexpr int N = 8;
  __device__ static void load(const uint16_t* p, float (&x)[8]) { unpack(*reinterpret_cast<const uint4*>(p), x); }
  __device__ static void unpack(const uint4& v, float (&x)[8]) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = __uint_as_float(w[i] << 16);
      x[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
  }
  __device__ static uint4 pack(const float (&x)[8]) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = static_cast<uint32_t>(f2bf(x[2 * i])) | (static_cast<uint32_t>(f2bf(x[2 * i + 1])) << 16);
    return make_uint4(w[0], w[1], w[2], w[3]);
  }
};
template <> struct Vec<float> {
  static constexpr int N = 4;
  __device__ static void load(const float* p, float (&x)[4]) { unpack(*reinterpret_cast<const uint4*>(p), x); }
  __device__ static void unpack(const uint4& v, float (&x)[4]) {
    x[0] = __uint_as_float(v.x); x[1] = __uint_as_float(v.y); x[2] = __uint_as_float(v.z); x[3] = __uint_as_float(v.w);
  }
  __device__ static uint4 pack(const float (&x)[4]) {
    return make_uint4(__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3]));
  }
};

__global__ void k_zero_u32(uint32_t* __restrict__ p, int64_t n) {
  int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (; i < n; i += stride) p[i] = 0u;
}
// What a call defines on rows that are not selected, in the launch that works on the others: some workgroups take a share of the rows each,
// read the whole selection (it stays in L2; eight loads of a thread under way) into a bit per row of their share, and hand the rows without one to `clear`, all threads of the
// workgroup together, up to 64 rows at a time, as a mask of the rows from `first` on.  Values and update, with launches of their own to clear,
// to mark a byte per row and to clear the rows without one, and like this: 1000 rows of 2048 25 and 20 us, 6000 34 and 28, 39 224 100 and 93 (on new
// rows 119 and 111), 100 000 of 1024 123 and 113, 400 000 of 512 401 and 395.  (One entry at a time, with 64-bit places, the selection took 60 us
// for 400 000 rows; marks by all workgroups and a queue of the rows to clear lost 80 us to atomics on one word.)
constexpr int kMapRows = 16384;            // rows of a workgroup at most
template <class F>
__device__ __forceinline__ void unselected_rows(int wg, int n_wg, int n_rows, const int32_t* __restrict__ rowsel, int64_t n_sel, uint32_t* s_map,
                                                F clear) {
  const int share = (n_rows + n_wg - 1) / n_wg, r0 = wg * share, n = min(share, n_rows - r0);   // share <= kMapRows (clear_grid)
  if (n <= 0) return;
  for (int i = threadIdx.x; i < kMapRows / 32; i += kVT) s_map[i] = 0u;
  __syncthreads();
  auto place = [&](int32_t row) { return static_cast<uint32_t>(row) - static_cast<uint32_t>(r0); };   // in the share: below n
  auto mark = [&](uint32_t i) {
    if (i < static_cast<uint32_t>(n)) atomicOr(s_map + (i >> 5), 1u << (i & 31));
  };
  const int64_t head = (4 - ((reinterpret_cast<uintptr_t>(rowsel) >> 2) & 3)) & 3;   // up to the first 16-byte boundary
  const int64_t n4 = n_sel > head ? (n_sel - head) / 4 : 0;
  const int4* const sel4 = reinterpret_cast<const int4*>(rowsel + head);
  for (int64_t i = threadIdx.x; i < n4; i += 8 * kVT) {
    int4 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = i + k * kVT < n4 ? sel4[i + k * kVT] : make_int4(-1, -1, -1, -1);
#pragma unroll
    for (int k = 0; k < 8; ++k) {                              // nearly always all of the wavefront's lie outside: three instructions an entry
      const uint32_t a = place(v[k].x), b = place(v[k].y), c = place(v[k].z), e = place(v[k].w), least = min(min(a, b), min(c, e));
      if (least < static_cast<uint32_t>(n)) { mark(a); mark(b); mark(c); mark(e); }
    }
  }
  const int64_t tail = head + 4 * n4 + threadIdx.x - 4;
  if (threadIdx.x < 4) {
    if (threadIdx.x < head && threadIdx.x < n_sel) mark(place(rowsel[threadIdx.x]));
  } else if (threadIdx.x < 8 && tail < n_sel) {
    mark(place(rowsel[tail]));
  }
  __syncthreads();
  for (int j = 0; j < n; j += kWave) {
    unsigned long long rest = ~(s_map[j >> 5] | static_cast<unsigned long long>(s_map[(j >> 5) + 1]) << 32);
    if (n - j < kWave) rest &= (1ull << (n - j)) - 1;
    if (rest) clear(static_cast<int64_t>(r0) + j, rest);
  }
}
// What an update defines on them; either may be NULL.
template <typename T>
struct ClearRows {
  float* value_new;
  T* dH;
  int nvec;
  __device__ __forceinline__ void operator()(int64_t first, unsigned long long rest) const {
    const int lane = threadIdx.x & (kWave - 1);
    if (value_new && threadIdx.x < kWave && (rest >> lane) & 1) value_new[first + lane] = 0.f;
    if (!dH) return;
    for (; rest; rest &= rest - 1) {
      T* const p = dH + (first + __ffsll(static_cast<long long>(rest)) - 1) * nvec * Vec<T>::N;
      for (int i = threadIdx.x; i < nvec; i += kVT) store_stream(p + i * Vec<T>::N, make_uint4(0u, 0u, 0u, 0u));
    }
  }
};
// Workgroups for it: enough that clearing takes no longer than the rows, few enough that most of the device does rows.  Every one of them
// reads the whole selection, so that the rows it is for are limited; beyond, launches go over all rows first.  Short rows leave
// nothing to read it behind (values and update in launches and along: 20 000 rows of 16 bytes 29.4 and 25.0 us, 30 000 30.2 and 31.2, 200 000 116
// and 138, 800 000 412 and 527; of 512 bytes 200 000 149 and 157; of 768 bytes 400 000 360 and 356, of 1 KB 800 000 794 and 785); rows of two to
// four KB hold fewer workgroups at once, which 64 of them delay by more than the launches (100 000 of 2176 bytes 187 and 185.5 us,
// 200 000 342 and 344, 380 000 628 and 636; of 4 KB 100 000 263 and 258, 380 000 966 and 984); behind the rows it costs longer ones nothing
// (268 000 of 6.9 KB 1472 and 1455).  Rows of up to 2 KB, two vectors a lane, have room for 128 (kShortRowsGrid): with 64 the rows, loaded two ahead, are done
// first and wait for the selection to be read and the stores behind it (64 and 128, values and update: 40 000 rows of 1 KB 46.7 and 42.1 us, of
// 1408 bytes 54.7 and 50.5, 70 000 float32 ones of 1 KB 70.8 and 59.3, 15 000 of 2 KB 31.1 and 31.2).  Longer rows give up what the
// clearing takes: 64 and 128, 39 224 of 4 KB 98 and 101, 100 000 of 2176 bytes 157 and 161.
constexpr unsigned kClearWgs = 64;
unsigned clear_grid(const int32_t* rowsel, int64_t n_rows, int64_t row_bytes) {
  static_assert(1 << 20 <= kClearWgs * kMapRows, "every share fits its map");
  const int64_t most = row_bytes < 768 ? 1 << 15 : row_bytes <= 1024 || row_bytes > 4096 ? 1 << 20 : 1 << 17;
  return rowsel && n_rows <= most ? std::min(row_bytes <= 2048 ? 2 * kClearWgs : kClearWgs, cdiv(static_cast<size_t>(n_rows), 128)) : 0;
}
// Those of an update: value_new[n] (may be NULL) and n16 16-byte words of `big` are cleared.
__global__ void __launch_bounds__(256)
k_value_open(uint32_t* __restrict__ value_new, int64_t n, uint4* __restrict__ big, int64_t n16) {
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x, stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = i0; i < n16; i += stride) store_stream(big + i, make_uint4(0u, 0u, 0u, 0u));
  if (value_new)
    for (int64_t i = i0; i < n; i += stride) value_new[i] = 0u;
}
// Large selections: dH is cleared only where the row kernel does not write it.  A byte per row says which rows are selected
// (in the memory of the partial sums, which come later); clearing all of dH first would write the selected rows twice.
__global__ void __launch_bounds__(256)
k_value_mark(const int32_t* __restrict__ rowsel, int64_t n_sel, int64_t n_rows, uint8_t* __restrict__ map) {
  const int64_t n = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (n >= n_sel) return;
  const int64_t row = rowsel[n];
  if (row >= 0 && row < n_rows) map[row] = 1;
}
constexpr int kClearRows = 64;             // rows of one workgroup: one ballot of a wavefront
__global__ void __launch_bounds__(256)
k_value_clear_rest(const uint8_t* __restrict__ map, int64_t n_rows, int row16, uint4* __restrict__ dH) {
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * kClearRows;
  const int64_t mine = r0 + (threadIdx.x & (kWave - 1));
  // every wavefront looks at the same rows and takes its share of each unselected one
  for (unsigned long long rest = __ballot(mine < n_rows && map[mine] == 0); rest; rest &= rest - 1) {
    uint4* p = dH + (r0 + __ffsll(static_cast<long long>(rest)) - 1) * row16;
    for (int i = threadIdx.x; i < row16; i += 256) store_stream(p + i, make_uint4(0u, 0u, 0u, 0u));
  }
}
// Below this many bytes of selected rows the two launches more cost as much as they save.
constexpr int64_t kMarkBytes = int64_t{48} << 20;

// Forward only: one wavefront per selected row, behind n_clear workgroups for the others.
template <typename T, bool SELECT>
__global__ void __launch_bounds__(kVT)
k_value_fwd(const T* __restrict__ H, const T* __restrict__ w, float bias, int d, const int32_t* __restrict__ rowsel,
            int64_t n_sel, int n_rows, int n_clear, float* __restrict__ value) {
  const int lane = threadIdx.x & (kWave - 1);
  if constexpr (SELECT) {
    if (static_cast<int>(blockIdx.x) < n_clear) {
      __shared__ uint32_t s_map[kMapRows / 32];
      unselected_rows(blockIdx.x, n_clear, n_rows, rowsel, n_sel, s_map, ClearRows<T>{value, nullptr, 0});
      return;
    }
  }
  const int64_t n = static_cast<int64_t>(blockIdx.x - n_clear) * kVWaves + threadIdx.x / kWave;
  if (n >= n_sel) return;
  const int64_t row = rowsel ? rowsel[n] : n;
  const T* h = H + row * d;
  AccT<T> acc = 0;
  for (int c = lane * Vec<T>::N; c < d; c += kWave * Vec<T>::N) {
    float x[Vec<T>::N], y[Vec<T>::N];
    Vec<T>::load(h + c, x);
    Vec<T>::load(w + c, y);
#pragma unroll
    for (int i = 0; i < Vec<T>::N; ++i) acc = fma(static_cast<AccT<T>>(x[i]), static_cast<AccT<T>>(y[i]), acc);
  }
  acc = wave_sum(acc);
  if (lane == 0) value[row] = static_cast<float>(acc + static_cast<AccT<T>>(bias));
}

__device__ __forceinline__ void add_stats(double* a, double loss, double clipped, double v, double rows) {
  atomicAdd(a + 0, loss);
  atomicAdd(a + 1, clipped);
  atomicAdd(a + 2, v);
  atomicAdd(a + 3, rows);
}
// Loss and backward, one wavefront per row.  Lane l owns the 16-byte column vectors l, l + 64, ... (KV of them):
// it keeps its part of w, of the current row and of the next row (prefetched) in registers, and its part of
// dw in float accumulators over all rows of the wavefront.  No barrier in the row loop.  With SELECT n_clear workgroups, from
// the clear_at-th on, do the rows that are not selected.  With ADD dH is added to, in a kernel of its own: both loops in one share a register
// budget (up to 860 bytes of scratch a lane, 10 000 rows of 8192 174 us, added to 246; apart and with the statistics below 125 and 170).  Four
// bf16 vectors a lane are held to the 168 registers of three wavefronts to a SIMD; float ones, with float64 sums, spill there (250 000 rows of
// 1024 650 us, not held 643).
template <typename T, int KV, bool SELECT, bool ADD>
__global__ void __launch_bounds__(kVT, KV == 4 && sizeof(T) == 2 ? 3 : 1)
k_value_rows(const T* __restrict__ H, const T* __restrict__ w, float bias, int d, const int32_t* __restrict__ rowsel,
             int64_t n_sel, int n_rows, int n_clear, int clear_at, int64_t norm, int64_t rows_per_block, const float* __restrict__ value_old, const float* __restrict__ ret,
             const int32_t* __restrict__ tok_role, int n_roles, float clip_eps, float* __restrict__ value_new,
             T* __restrict__ dH, float* __restrict__ part_dw, double* __restrict__ blk_stats) {
  __shared__ double s_acc[(1 + UMAS_MAX_ROLES) * kVStat];
  __shared__ float s_g[kVWaves];
  extern __shared__ __attribute__((aligned(16))) char s_raw[];
  AccT<T>* const s_dw = reinterpret_cast<AccT<T>*>(s_raw);       // [d]
  constexpr int N = Vec<T>::N;
  const int nvec = d / N;
  const int nacc = (1 + n_roles) * kVStat;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  if constexpr (SELECT) {
    const int c = static_cast<int>(blockIdx.x) - clear_at;
    if (c >= 0 && c < n_clear) {
      __shared__ uint32_t s_map[kMapRows / 32];
      unselected_rows(c, n_clear, n_rows, rowsel, n_sel, s_map, ClearRows<T>{value_new, ADD ? nullptr : dH, nvec});
      return;
    }
  }
  const int blk = static_cast<int>(blockIdx.x) - (SELECT && clear_at == 0 ? n_clear : 0);
  const int64_t r_begin = static_cast<int64_t>(blk) * rows_per_block;
  const int64_t r_end = r_begin + rows_per_block < n_sel ? r_begin + rows_per_block : n_sel;
  for (int i = threadIdx.x; i < nacc; i += kVT) s_acc[i] = 0.0;
  __syncthreads();
  // w and the rows stay packed as loaded (16 bytes per vector) and are unpacked where they are used
  using A = AccT<T>;
  uint4 wp[KV];
  A acc[KV][N];
#pragma unroll
  for (int k = 0; k < KV; ++k) {
    const int cv = lane + k * kWave;
#pragma unroll
    for (int i = 0; i < N; ++i) acc[k][i] = 0;
    wp[k] = make_uint4(0u, 0u, 0u, 0u);
    if (cv < nvec) wp[k] = *reinterpret_cast<const uint4*>(w + cv * N);
  }
  float gsum = 0.f;
  const float inv_s = 1.f / static_cast<float>(norm);

  // The wavefront's rows, 64 at a time: a lane has what belongs to one of them besides H, its place, old value, return and role, so that in the
  // loop over them nothing is loaded but rows, the next one under way while this one is finished.  Every row is the same number of loads and
  // stores (columns past d and rows past the last are out of a buffer's range, which looks at the lane's offset only), and the waits are for the
  // row that is next, not for the stores of the last.  With the place and the role loaded row by row, each waited for together with everything
  // under way, values and update of 39 224 rows of 2048 108 us, now 97, 60 000 of 2560 247 and 184, 100 000 of 1088 186 and 157, 60 000 float32 rows of
  // 1024 159 and 146, 190 000 of 4032 1890 and 1892.
  const int row_bytes = nvec * 16;
  auto rsrc = [&](const void* base, int64_t row, bool there) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(static_cast<const T*>(base)) + row * d, 0, there ? row_bytes : 0, 0x00020000);
  };
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  constexpr int kPast = 2;                           // policy of a store past the caches
  // Statistics of the wavefront's rows of role `lane`, of those without a role in lane n_roles (if 64 roles leave a lane), as the rows are finished;
  // kept for 64 rows and added up across lanes behind them they took the registers that sixteen vectors spilled.
  double sum_l = 0.0, sum_v = 0.0;
  unsigned n_in = 0, n_clipped = 0;
  for (int64_t n0 = r_begin + __builtin_amdgcn_readfirstlane(wave); n0 < r_end; n0 += kVWaves * kWave) {
    const int64_t left = (r_end - n0 + kVWaves - 1) / kVWaves;
    const int cnt = left < kWave ? static_cast<int>(left) : kWave;
    int64_t my_row = 0;
    float my_vo = 0.f, my_ret = 0.f, my_v = 0.f;
    int my_role = -1;                                  // as it is: looked at here it would be waited for before the first row is asked for
    if (lane < cnt) {
      const int64_t n = n0 + lane * kVWaves;
      my_row = rowsel ? rowsel[n] : n;
      my_vo = value_old[my_row];
      my_ret = ret[my_row];
      if (tok_role && n_roles > 0) my_role = tok_role[my_row];
    }
    auto row_at = [&](int i) {
      return static_cast<int64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(my_row), i))) |
             static_cast<int64_t>(__builtin_amdgcn_readlane(static_cast<int>(my_row >> 32), i)) << 32;
    };
    auto float_at = [&](float v, int i) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), i)); };
    auto fetch = [&](int i, uint4 (&x)[KV]) {
      const __amdgpu_buffer_rsrc_t h = rsrc(H, i < cnt ? row_at(i) : 0, i < cnt);
#pragma unroll
      for (int k = 0; k < KV; ++k) x[k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(h, lane * 16 + k * kWave * 16, 0, 0));
      asm volatile("" : : : "memory");             // they go out here, not when they are wanted
    };
    uint4 even[KV], odd[KV];
    fetch(0, even);
    auto finish = [&](int i, const uint4 (&h)[KV]) {
      A dot = 0;
#pragma unroll
      for (int k = 0; k < KV; ++k) {
        float x[N], y[N];
        Vec<T>::unpack(h[k], x);
        Vec<T>::unpack(wp[k], y);
#pragma unroll
        for (int c = 0; c < N; ++c) dot = fma(static_cast<A>(x[c]), static_cast<A>(y[c]), dot);
      }
      dot = wave_sum(dot);
      // the value is a float32 result; loss and gradient are formed from that rounded value
      const float V = static_cast<float>(dot + static_cast<A>(bias)), vo = float_at(my_vo, i), R = float_at(my_ret, i);
      const float vc = fminf(fmaxf(V, vo - clip_eps), vo + clip_eps);   // V itself inside the range: an exact tie
      const float lu = (V - R) * (V - R), lc = (vc - R) * (vc - R);
      const bool unclipped = lu >= lc;
      const float g = unclipped ? (V - R) * inv_s : 0.f;
      gsum += g;
      my_v = lane == i ? V : my_v;
      const int role = __builtin_amdgcn_readlane(my_role, i), slot = role >= 0 && role < n_roles ? role : n_roles;
      const float loss = 0.5f * (unclipped ? lu : lc);
      if (slot == lane) {
        sum_l += static_cast<double>(loss);
        sum_v += static_cast<double>(V);
        ++n_in;
        n_clipped += unclipped ? 0u : 1u;
      }
      if (slot == kWave && lane == 0) add_stats(s_acc, static_cast<double>(loss), unclipped ? 0.0 : 1.0, static_cast<double>(V), 1.0);
      const __amdgpu_buffer_rsrc_t out = rsrc(dH, row_at(i), true);
#pragma unroll
      for (int k = 0; k < KV; ++k) {
        float x[N], y[N], o[N];
        Vec<T>::unpack(h[k], x);
        Vec<T>::unpack(wp[k], y);
        if constexpr (ADD) Vec<T>::unpack(__builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(out, lane * 16 + k * kWave * 16, 0, 0)), o);
#pragma unroll
        for (int c = 0; c < N; ++c) {
          acc[k][c] = fma(static_cast<A>(g), static_cast<A>(x[c]), acc[k][c]);
          o[c] = ADD ? o[c] + g * y[c] : g * y[c];
        }
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, Vec<T>::pack(o)), out, lane * 16 + k * kWave * 16, 0, kPast);
      }
    };
    if constexpr (KV > 8 && std::is_same<T, float>::value) {   // with float64 sums two turns of the loop in one spill (10 000 rows of 4096 129 us, like this 120)
#pragma unroll 1
      for (int i = 0; i < cnt; ++i) {
        fetch(i + 1, odd);
        finish(i, even);
#pragma unroll
        for (int k = 0; k < KV; ++k) even[k] = odd[k];
      }
    } else {
      if constexpr (!ADD) {                       // as many stores of nothing as a row has: the loop's first turn waits like the others
        const __amdgpu_buffer_rsrc_t none = rsrc(dH, 0, false);
#pragma unroll
        for (int k = 0; k < KV; ++k) __builtin_amdgcn_raw_buffer_store_b128(u32x4{0u, 0u, 0u, 0u}, none, lane * 16 + k * kWave * 16, 0, kPast);
      }
      for (int i = 0;; i += 2) {
        fetch(i + 1, odd);
        finish(i, even);
        if (i + 1 >= cnt) break;
        fetch(i + 2, even);
        finish(i + 1, odd);
        if (i + 2 >= cnt) break;
      }
    }
    if (lane < cnt && value_new) value_new[my_row] = my_v;
  }
  if (n_in) add_stats(s_acc + (lane < n_roles ? 1 + lane : 0) * kVStat, sum_l, static_cast<double>(n_clipped), sum_v, static_cast<double>(n_in));
  // the wavefronts' sums meet in LDS one after the other; the workgroup leaves one partial row: [blocks][part_pitch(d)].
  // (Four partial rows a workgroup, reduced in two launches, and the statistics of all roles in one workgroup took
  // 36 us after the rows; now 7.)
  for (int k = 0; k < kVWaves; ++k) {
    if (k == wave) {
#pragma unroll
      for (int q = 0; q < KV; ++q) {
        const int cv = lane + q * kWave;
        if (cv < nvec)
#pragma unroll
          for (int i = 0; i < N; ++i) s_dw[cv * N + i] = k == 0 ? acc[q][i] : s_dw[cv * N + i] + acc[q][i];
      }
      if (lane == 0) s_g[wave] = gsum;
    }
    __syncthreads();
  }
  float* pd = part_dw + static_cast<size_t>(blk) * part_pitch(d);
  for (int j = threadIdx.x; j < d; j += kVT) pd[j] = static_cast<float>(s_dw[j]);
  if (threadIdx.x == 0) pd[d] = (s_g[0] + s_g[1]) + (s_g[2] + s_g[3]);
  for (int i = threadIdx.x; i < nacc; i += kVT) {
    double x = s_acc[i];
    if (i < kVStat)                                  // all rows: those without a role and every role's
      for (int r = 1; r <= n_roles; ++r) x += s_acc[r * kVStat + i];
    blk_stats[static_cast<size_t>(blk) * nacc + i] = x;
  }
}

// What the workgroups of the row kernel left, added up in a fixed order.  The first col_blocks workgroups take 16 columns
// each (64-byte pieces of the partial rows; thread = 16 * group of rows + column) and add into or overwrite dw (columns
// < d) and db (column d); the others one statistics record each.
constexpr int kFinCols = 16, kFinT = 1024, kFinGroups = kFinT / kFinCols;
__global__ void __launch_bounds__(kFinT)
k_value_finish(const float* __restrict__ part, int nblk, int d, int col_blocks, int accumulate, float* __restrict__ dw,
               float* __restrict__ db, int n_roles, int64_t norm_rows, const double* __restrict__ blk_stats,
               umas_value_stats* __restrict__ stats) {
  const int tid = threadIdx.x;
  if (static_cast<int>(blockIdx.x) < col_blocks) {
    __shared__ float s_sum[kFinGroups][kFinCols + 1];
    const int col = tid & (kFinCols - 1), grp = tid / kFinCols, j = blockIdx.x * kFinCols + col;
    const size_t pitch = part_pitch(d);
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    if (j <= d)
      for (int b = grp; b < nblk; b += 4 * kFinGroups)
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (b + k * kFinGroups < nblk) s[k] += part[static_cast<size_t>(b + k * kFinGroups) * pitch + j];
    s_sum[grp][col] = (s[0] + s[1]) + (s[2] + s[3]);
    for (int o = kFinGroups / 2; o > 0; o >>= 1) {
      __syncthreads();
      if (grp < o) s_sum[grp][col] += s_sum[grp + o][col];
    }
    if (grp == 0 && j <= d) {
      float* dst = j < d ? dw + j : db;
      if (dst) *dst = accumulate ? *dst + s_sum[0][col] : s_sum[0][col];
    }
    return;
  }
  __shared__ double smem[32];
  const int nacc = (1 + n_roles) * kVStat, k = blockIdx.x - col_blocks;
  double sum[kVStat];
#pragma unroll
  for (int j = 0; j < kVStat; ++j) sum[j] = tid < nblk ? blk_stats[static_cast<size_t>(tid) * nacc + k * kVStat + j] : 0.0;   // nblk <= kMaxGrid
#pragma unroll
  for (int j = 0; j < kVStat; ++j) sum[j] = block_sum<double>(sum[j], smem);
  if (tid != 0) return;
  const double cnt = sum[3];
  umas_value_stats s;
  const double den = (k == 0 && norm_rows > 0) ? static_cast<double>(norm_rows) : cnt;   // the caller's normaliser
  s.loss = cnt > 0 ? static_cast<float>(sum[0] / den) : 0.f;
  s.clip_frac = cnt > 0 ? static_cast<float>(sum[1] / cnt) : 0.f;
  s.value_mean = cnt > 0 ? static_cast<float>(sum[2] / cnt) : 0.f;
  s.reserved = 0.f;
  s.n_scored = static_cast<int64_t>(cnt);
  stats[k] = s;
}
static_assert(kMaxGrid <= kFinT, "one thread per workgroup of the row kernel in the statistics");

unsigned value_grid(int64_t n_sel) {
  const int64_t b = (n_sel + kVWaves - 1) / kVWaves;
  return static_cast<unsigned>(b < 1 ? 1 : b > kMaxGrid ? kMaxGrid : b);
}
int max_d(umas_dtype dt) { return dt == UMAS_BF16 ? kWave * kMaxKV * 8 : kWave * kMaxKV * 4; }

// Workgroups of the row kernel that the device holds at once (the kernel's register use differs with KV): its grid is
// one resident round, so that no second, partly filled round follows.  Looked up once per instance.
template <typename T, int K, bool ADD>
unsigned resident_value_blocks() {
  static unsigned cached = 0;
  if (cached) return cached;
  int dev = 0, n_cu = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
    n_cu = 64;
  constexpr size_t kLds = static_cast<size_t>(K) * kWave * Vec<T>::N * sizeof(AccT<T>);   // the widest rows of the instance
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_value_rows<T, K, false, ADD>, kVT, kLds) != hipSuccess || per_cu < 1) per_cu = 1;
  cached = static_cast<unsigned>(per_cu) * static_cast<unsigned>(n_cu);
  return cached;
}

template <typename T, bool ADD>
unsigned resident_value_blocks_kv(int kv) {
  if (kv <= 1) return resident_value_blocks<T, 1, ADD>();
  if (kv <= 2) return resident_value_blocks<T, 2, ADD>();
  if (kv <= 4) return resident_value_blocks<T, 4, ADD>();
  if (kv <= 8) return resident_value_blocks<T, 8, ADD>();
  return resident_value_blocks<T, 16, ADD>();
}

template <typename T, bool ADD>
void launch_value_rows(int kv, unsigned grid, hipStream_t st, const void* H, const void* w, float bias, int d,
                       const int32_t* rowsel, int64_t n_sel, int64_t n_rows, unsigned n_clear, unsigned clear_at, int64_t norm, int64_t rpb, const float* value_old, const float* ret,
                       const int32_t* tok_role, int n_roles, float clip_eps, float* value_new, void* dH,
                       float* part_dw, double* blk_stats) {
#define UMAS_VALUE_CASE(K)                                                                                              \
  hipLaunchKernelGGL((n_clear ? k_value_rows<T, K, true, ADD> : k_value_rows<T, K, false, ADD>), dim3(n_clear + grid), dim3(kVT), d * sizeof(AccT<T>), st, static_cast<const T*>(H), static_cast<const T*>(w), \
                     bias, d, rowsel, n_sel, n_clear ? static_cast<int>(n_rows) : 0, static_cast<int>(n_clear), static_cast<int>(clear_at), norm, rpb, value_old, ret, tok_role, n_roles, clip_eps, value_new,         \
                     static_cast<T*>(dH), part_dw, blk_stats)
  if (kv <= 1) UMAS_VALUE_CASE(1);
  else if (kv <= 2) UMAS_VALUE_CASE(2);
  else if (kv <= 4) UMAS_VALUE_CASE(4);
  else if (kv <= 8) UMAS_VALUE_CASE(8);
  else UMAS_VALUE_CASE(16);
#undef UMAS_VALUE_CASE
}

hipError_t zero_words(void* p, int64_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_zero_u32, dim3(cdiv(n, 1024) < 8192 ? cdiv(n, 1024) : 8192), dim3(256), 0, st, static_cast<uint32_t*>(p), n);
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess && g_prof_on) prof_kernel("k_zero_u32", st);
  return e;
}

umas_status check_value_args(const void* H, const void* w, umas_dtype dt, int64_t n_rows, int d, const int32_t* rowsel,
                             int64_t n_sel) {
  UMAS_REQUIRE(dt == UMAS_F32 || dt == UMAS_BF16, UMAS_EDTYPE, "dtype=%d is neither F32 nor BF16", static_cast<int>(dt));
  UMAS_REQUIRE(n_rows >= 0 && n_sel >= 0 && n_sel <= n_rows, UMAS_EINVAL, "row counts must satisfy 0 <= n_sel <= n_rows");
  UMAS_REQUIRE(rowsel || n_sel == n_rows, UMAS_EINVAL, "rowsel is NULL but n_sel != n_rows");
  const int n = dt == UMAS_BF16 ? 8 : 4;
  UMAS_REQUIRE(d >= n && d % n == 0 && d <= max_d(dt), UMAS_ESHAPE, "d=%d must be a multiple of %d and at most %d", d, n, max_d(dt));
  UMAS_REQUIRE((H || n_rows == 0) && w, UMAS_EINVAL, "H and w must not be NULL");
  UMAS_REQUIRE(reinterpret_cast<uintptr_t>(H) % 16 == 0 && reinterpret_cast<uintptr_t>(w) % 16 == 0, UMAS_EINVAL,
               "H and w must be 16-byte aligned");
  return UMAS_OK;
}

}  // namespace
}  // namespace umas

using namespace umas;

extern "C" size_t umas_value_workspace_bytes(int64_t n_sel, int32_t d, umas_dtype dtype, int32_t n_roles) {
  if (n_sel < 0 || d < 1 || n_roles < 0) return 0;
  (void)dtype;
  const unsigned grid = value_grid(n_sel);
  Carver c(nullptr);
  c.take<float>(static_cast<size_t>(grid) * part_pitch(d));                                      // one partial row per workgroup
  c.take<double>(static_cast<size_t>(grid) * (1 + n_roles) * kVStat);
  return c.off;
}

extern "C" umas_status umas_values(const void* H, const void* w, float bias, umas_dtype dtype, int64_t n_rows, int32_t d,
                                   const int32_t* rowsel, int64_t n_sel, float* value, void* hip_stream) {
  umas_status s = check_value_args(H, w, dtype, n_rows, d, rowsel, n_sel);
  if (s != UMAS_OK) return s;
  UMAS_REQUIRE(value || n_rows == 0, UMAS_EINVAL, "value must not be NULL");
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  prof_mark(st);
  if (n_sel == 0) {
    if (n_rows > 0) UMAS_HIP(zero_words(value, n_rows, st));
    return UMAS_OK;
  }
  const unsigned n_clear = clear_grid(rowsel, n_rows, static_cast<int64_t>(d) * (dtype == UMAS_BF16 ? 2 : 4));
  if (rowsel && n_clear == 0) UMAS_HIP(zero_words(value, n_rows, st));
  auto fwd = [&](auto kernel, auto* h) {
    using T = std::remove_pointer_t<decltype(h)>;
    hipLaunchKernelGGL(kernel, dim3(n_clear + cdiv(n_sel, kVWaves)), dim3(kVT), 0, st, h, static_cast<T*>(w), bias, d, rowsel, n_sel,
                       n_clear ? static_cast<int>(n_rows) : 0, static_cast<int>(n_clear), value);
  };
  if (dtype == UMAS_BF16) fwd(n_clear ? k_value_fwd<uint16_t, true> : k_value_fwd<uint16_t, false>, static_cast<const uint16_t*>(H));
  else fwd(n_clear ? k_value_fwd<float, true> : k_value_fwd<float, false>, static_cast<const float*>(H));
  UMAS_LAUNCHED("k_value_fwd");
  return UMAS_OK;
}

extern "C" umas_status umas_value_loss_fwd_bwd(const void* H, const void* w, float bias, umas_dtype dtype, int64_t n_rows,
                                               int32_t d, const int32_t* rowsel, int64_t n_sel, const float* value_old,
                                               const float* ret, const int32_t* tok_role, int32_t n_roles,
                                               float clip_eps_v, int32_t accumulate_dH, int32_t accumulate_dw,
                                               int64_t norm_rows, umas_value_stats* stats, float* value_new, void* dH, float* dw, float* db,
                                               void* workspace, size_t workspace_bytes, void* hip_stream) {
  umas_status s = check_value_args(H, w, dtype, n_rows, d, rowsel, n_sel);
  if (s != UMAS_OK) return s;
  UMAS_REQUIRE(n_roles >= 0 && n_roles <= UMAS_MAX_ROLES, UMAS_ESHAPE, "n_roles=%d outside [0,%d]", n_roles, UMAS_MAX_ROLES);
  UMAS_REQUIRE(clip_eps_v > 0.f, UMAS_EINVAL, "clip_eps_v must be positive");
  UMAS_REQUIRE(stats && dw && (dH || n_rows == 0), UMAS_EINVAL, "stats, dw and dH must not be NULL");
  UMAS_REQUIRE((value_old && ret) || n_sel == 0, UMAS_EINVAL, "value_old and ret must not be NULL");
  UMAS_REQUIRE(reinterpret_cast<uintptr_t>(dH) % 16 == 0, UMAS_EINVAL, "dH must be 16-byte aligned");
  UMAS_REQUIRE(norm_rows == 0 || norm_rows >= n_sel, UMAS_EINVAL, "norm_rows=%lld must be 0 or at least n_sel=%lld",
               static_cast<long long>(norm_rows), static_cast<long long>(n_sel));
  const int64_t norm = norm_rows > 0 ? norm_rows : n_sel;   // rows the mean is taken over
  const size_t need = umas_value_workspace_bytes(n_sel, d, dtype, n_roles);
  UMAS_REQUIRE(workspace && reinterpret_cast<uintptr_t>(workspace) % kAlign == 0 && workspace_bytes >= need, UMAS_EWORKSPACE,
               "workspace must be 256-byte aligned and hold %zu bytes (got %zu)", need, workspace_bytes);
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  prof_mark(st);
  const size_t esz = dtype == UMAS_BF16 ? 2 : 4;
  const int nvec = d / (dtype == UMAS_BF16 ? 8 : 4);
  const int kv = (nvec + kWave - 1) / kWave;
  // at most value_grid(n_sel) workgroups (what the workspace is sized for), and no more than are resident at once
  const unsigned resident = dtype == UMAS_BF16 ? (accumulate_dH ? resident_value_blocks_kv<uint16_t, true>(kv) : resident_value_blocks_kv<uint16_t, false>(kv))
                                               : (accumulate_dH ? resident_value_blocks_kv<float, true>(kv) : resident_value_blocks_kv<float, false>(kv));
  // the workgroups that clear are part of that round and go first; behind a full round of rows where the instance holds so few at once
  // that giving them up costs more than a tail, those for rows of more than 4 KB (39 224 rows of 4096 233 us with them first, 204 behind;
  // values and update of 48 651 rows of 3008 246 and 222, of 268 000 float32 rows of 1728 1733 and 1455; the other way round shorter rows: 100 000 of 1088
  // 185.5 first, 195 behind)
  const size_t row_bytes = static_cast<size_t>(d) * esz;             // a multiple of 16
  const unsigned n_clear = n_sel > 0 ? clear_grid(rowsel, n_rows, row_bytes) : 0;
  const bool last = kv > 4;
  const unsigned grid = std::min({value_grid(n_sel), kv <= 2 && row_bytes >= 768 ? kShortRowsGrid - n_clear : kMaxGrid, last || resident <= n_clear ? resident : resident - n_clear});
  const unsigned clear_at = last ? grid : 0;
  const size_t part_bytes = static_cast<size_t>(grid) * part_pitch(d) * sizeof(float);
  Carver c(workspace);
  float* part_dw = c.take<float>(part_bytes / sizeof(float));
  double* blk_stats = c.take<double>(static_cast<size_t>(grid) * (1 + n_roles) * kVStat);

  if (rowsel && n_rows > 0 && n_clear == 0) {
    const bool mark = !accumulate_dH && n_sel * static_cast<int64_t>(row_bytes) >= kMarkBytes && align_up(n_rows, 16) <= part_bytes;
    const int64_t n16 = accumulate_dH ? 0 : static_cast<int64_t>(mark ? align_up(n_rows, 16) / 16 : n_rows * row_bytes / 16);
    uint8_t* map = reinterpret_cast<uint8_t*>(part_dw);
    hipLaunchKernelGGL(k_value_open, dim3(std::min(std::max(cdiv(n16, 1024), cdiv(n_rows, 1024)), 8192u)), dim3(256), 0, st,
                       reinterpret_cast<uint32_t*>(value_new), n_rows, static_cast<uint4*>(mark ? static_cast<void*>(map) : dH), n16);
    UMAS_LAUNCHED("k_value_open");
    if (mark) {
      hipLaunchKernelGGL(k_value_mark, dim3(cdiv(n_sel, 256)), dim3(256), 0, st, rowsel, n_sel, n_rows, map);
      UMAS_LAUNCHED("k_value_mark");
      hipLaunchKernelGGL(k_value_clear_rest, dim3(cdiv(n_rows, kClearRows)), dim3(256), 0, st, map, n_rows, static_cast<int>(row_bytes / 16),
                         static_cast<uint4*>(dH));
      UMAS_LAUNCHED("k_value_clear_rest");
    }
  }
  if (n_sel > 0) {
    const int64_t rpb = (n_sel + grid - 1) / grid;                 // rows per workgroup; every wavefront writes its partial row
    const auto launch = dtype == UMAS_BF16 ? (accumulate_dH ? launch_value_rows<uint16_t, true> : launch_value_rows<uint16_t, false>)
                                           : (accumulate_dH ? launch_value_rows<float, true> : launch_value_rows<float, false>);
    launch(kv, grid, st, H, w, bias, d, rowsel, n_sel, n_rows, n_clear, clear_at, norm, rpb, value_old, ret, tok_role, n_roles, clip_eps_v, value_new, dH,
           part_dw, blk_stats);
    UMAS_LAUNCHED("k_value_rows");
  } else {
    // an empty selection still defines the outputs: zero partials give zero statistics and gradients
    UMAS_HIP(zero_words(part_dw, static_cast<int64_t>(part_bytes / 4), st));
    UMAS_HIP(zero_words(blk_stats, static_cast<int64_t>(grid) * (1 + n_roles) * kVStat * 2, st));
  }
  const int col_blocks = static_cast<int>(cdiv(d + 1, kFinCols));
  hipLaunchKernelGGL(k_value_finish, dim3(col_blocks + 1 + n_roles), dim3(kFinT), 0, st, part_dw, static_cast<int>(grid), d, col_blocks,
                     accumulate_dw, dw, db, n_roles, norm_rows, blk_stats, stats);
  UMAS_LAUNCHED("k_value_finish");
  return UMAS_OK;
}
