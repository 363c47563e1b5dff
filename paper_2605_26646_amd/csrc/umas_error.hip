// Thread-local error message, the pinned staging ring for thin host arrays and the optional kernel timing aid of libumas.
#include <string.h>

#include <atomic>
#include <chrono>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "umas_common.h"

namespace umas {
namespace {
thread_local char g_msg[512] = "";

struct Interval {
  const char* name;
  hipEvent_t begin, end;
};
std::vector<Interval> g_intervals;
std::vector<hipEvent_t> g_events;
hipEvent_t g_last = nullptr;
constexpr size_t kMaxIntervals = 1 << 16;

hipEvent_t new_event(hipStream_t st) {
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  g_events.push_back(e);
  if (hipEventRecord(e, st) != hipSuccess) return nullptr;
  return e;
}
void reset() {
  for (hipEvent_t e : g_events) (void)hipEventDestroy(e);
  g_events.clear();
  g_intervals.clear();
  g_last = nullptr;
}
}  // namespace

bool g_prof_on = false;

// ------------------------------------------------------------------ pinned staging ring
namespace {
struct StageSlot {
  char* host = nullptr;
  char* dev = nullptr;           // the block's address on the device
  size_t cap = 0;
  int device = 0;                // where the kernel that reads the block was launched
  unsigned n_wg = 0;             // its workgroups: as many words at `words` say that it has read the block
  size_t words = 0;
  hipEvent_t read = nullptr;     // recorded behind a kernel launched under capture, in place of the words
  bool in_flight = false, by_event = false;
};
StageSlot g_slots[ThinStage::kSlots];
int g_next_slot = 0;
std::mutex g_stage_mutex;
constexpr unsigned kMaxReaders = 1u << 14;

// Waits until the kernel launched on the block has read it.  The words end the wait as soon as it has; should they not, the device is
// waited for after a minute, and what it says is the answer.
hipError_t wait_until_read(StageSlot& s) {
  if (s.by_event) return hipEventSynchronize(s.read);
  volatile uint32_t* const done = reinterpret_cast<uint32_t*>(s.host + s.words);
  using clock = std::chrono::steady_clock;
  clock::time_point start;
  unsigned seen = 0;
  for (unsigned spins = 0;; ++spins) {
    while (seen < s.n_wg && done[seen]) ++seen;
    if (seen == s.n_wg) break;
    if (spins < 4096) {
      __builtin_ia32_pause();
      continue;
    }
    if (spins == 4096) start = clock::now();
    if (clock::now() - start > std::chrono::seconds(60)) {
      int dev = 0;
      hipError_t e = hipGetDevice(&dev);
      if (e == hipSuccess && dev != s.device) e = hipSetDevice(s.device);
      if (e == hipSuccess) e = hipDeviceSynchronize();
      if (dev != s.device) (void)hipSetDevice(dev);
      return e;                  // the kernel has run, or never will
    }
    std::this_thread::sleep_for(std::chrono::microseconds(20));
  }
  std::atomic_thread_fence(std::memory_order_acquire);
  return hipSuccess;
}
}  // namespace

umas_status ThinStage::begin(size_t bytes) {
  g_stage_mutex.lock();
  slot_ = g_next_slot;
  g_next_slot = (g_next_slot + 1) % kSlots;
  StageSlot& s = g_slots[slot_];
  auto bail = [&](hipError_t e, const char* what) {
    slot_ = -1;
    cur_ = nullptr;
    g_stage_mutex.unlock();
    return fail(UMAS_EHIP, "%s failed: %s", what, hipGetErrorString(e));
  };
  if (s.in_flight) {             // the kernel launched on this block kSlots calls ago must have read it
    const hipError_t e = wait_until_read(s);
    if (e != hipSuccess) return bail(e, "waiting for a staging block");
    s.in_flight = false;
  }
  bytes_ = align_up(bytes);
  const size_t need = bytes_ + kMaxReaders * sizeof(uint32_t);
  if (s.cap < need) {
    if (s.host) (void)hipHostFree(s.host);
    s.host = nullptr;
    s.cap = 0;
    size_t cap = 1 << 17;
    while (cap < need) cap <<= 1;
    void* p = nullptr;
    // coherent: a kernel reads the block, at the same address again four calls later, and must not find old lines in a cache
    hipError_t e = hipHostMalloc(&p, cap, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent);
    if (e != hipSuccess) return bail(e, "hipHostMalloc");
    void* d = nullptr;
    e = hipHostGetDevicePointer(&d, p, 0);
    if (e != hipSuccess) {
      (void)hipHostFree(p);
      return bail(e, "hipHostGetDevicePointer");
    }
    s.host = static_cast<char*>(p);
    s.dev = static_cast<char*>(d);
    s.cap = cap;
  }
  cur_ = s.host;
  return UMAS_OK;
}

void ThinStage::put(size_t off, const void* src, size_t n) {
  if (src && n) memcpy(cur_ + off, src, n);
}

void ThinStage::zero(size_t off, size_t n) {
  if (n) memset(cur_ + off, 0, n);
}

// The block for a kernel of n_wg workgroups that is launched next on `st`.
umas_status ThinStage::lend(unsigned n_wg, hipStream_t st, Reader* r) {
  StageSlot& s = g_slots[slot_];
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  hipError_t e = hipStreamIsCapturing(st, &capture);
  if (e == hipSuccess) e = hipGetDevice(&s.device);
  s.by_event = capture != hipStreamCaptureStatusNone || n_wg > kMaxReaders;
  if (e == hipSuccess && s.by_event && !s.read) e = hipEventCreateWithFlags(&s.read, hipEventDisableTiming);
  if (e != hipSuccess) {
    abandon();
    return fail(UMAS_EHIP, "staging failed: %s", hipGetErrorString(e));
  }
  n_wg_ = n_wg;
  s.words = bytes_;
  if (!s.by_event) zero(bytes_, n_wg * sizeof(uint32_t));
  r->block = s.dev;
  r->done = s.by_event ? nullptr : reinterpret_cast<uint32_t*>(s.dev + bytes_);
  return UMAS_OK;
}

// Behind the launch: e is what it said.
umas_status ThinStage::launched(hipStream_t st, hipError_t e) {
  StageSlot& s = g_slots[slot_];
  if (e == hipSuccess && s.by_event) e = hipEventRecord(s.read, st);
  if (e == hipSuccess) {
    s.n_wg = n_wg_;
    s.in_flight = true;
  }
  slot_ = -1;
  cur_ = nullptr;
  g_stage_mutex.unlock();
  if (e != hipSuccess) return fail(UMAS_EHIP, "staging failed: %s", hipGetErrorString(e));
  return UMAS_OK;
}

namespace {
// The block is copied by a kernel that reads the pinned memory over the bus.  The runtime's own copy costs more at every size: below 16 KB it
// is a kernel too, but behind a hand-over on either side, above another engine's.  Neither is an event recorded behind it: that flushes the
// caches and holds the stream for 5 us; every workgroup says in a word of the pinned memory that it has read its share (the calls around
// a batch of 49 152 tokens, two blocks of 2.4 and 0.5 KB: 100.5 -> 90.6 us a pass; 25 million tokens, 1.9 and 0.3 MB: 587 -> 584).
constexpr int kStageWords = 4;                 // 16-byte words a thread has in flight
__global__ void __launch_bounds__(256)
k_stage_copy(ThinStage::Reader src, uint4* __restrict__ dst, int64_t n16) {
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * (256 * kStageWords) + threadIdx.x;
  const uint4* __restrict__ from = reinterpret_cast<const uint4*>(src.block);
  uint4 v[kStageWords];
#pragma unroll
  for (int k = 0; k < kStageWords; ++k)
    if (i0 + k * 256 < n16) v[k] = from[i0 + k * 256];
#pragma unroll
  for (int k = 0; k < kStageWords; ++k)
    if (i0 + k * 256 < n16) dst[i0 + k * 256] = v[k];
  stage_read_done(src);
}
}  // namespace

umas_status ThinStage::flush(void* dst, size_t bytes, hipStream_t st) {
  if (!bytes) {
    abandon();
    return UMAS_OK;
  }
  const int64_t n16 = static_cast<int64_t>(bytes / 16);                // whole arrays of the carver: a multiple of 256
  const unsigned n_wg = cdiv(static_cast<size_t>(n16), 256 * kStageWords);
  Reader r;
  const umas_status s = lend(n_wg, st, &r);
  if (s != UMAS_OK) return s;
  hipLaunchKernelGGL(k_stage_copy, dim3(n_wg), dim3(256), 0, st, r, static_cast<uint4*>(dst), n16);
  return launched(st, hipGetLastError());
}

void ThinStage::abandon() {
  if (slot_ < 0) return;
  slot_ = -1;
  cur_ = nullptr;
  g_stage_mutex.unlock();
}

umas_status fail(umas_status code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_msg, sizeof(g_msg), fmt, ap);
  va_end(ap);
  return code;
}

void prof_mark(hipStream_t st) {
  if (!g_prof_on) return;
  g_last = new_event(st);
}

void prof_kernel(const char* name, hipStream_t st) {
  if (!g_prof_on || g_intervals.size() >= kMaxIntervals) return;
  hipEvent_t e = new_event(st);
  if (g_last && e) g_intervals.push_back(Interval{name, g_last, e});
  g_last = e;
}
}  // namespace umas

extern "C" const char* umas_last_error(void) { return umas::g_msg; }

extern "C" umas_status umas_profile_enable(int32_t on) {
  umas::reset();
  umas::g_prof_on = on != 0;
  return UMAS_OK;
}

extern "C" int32_t umas_profile_read(char* names, float* total_ms, int32_t* launches, int32_t cap) {
  using namespace umas;
  std::map<std::string, std::pair<double, int>> agg;
  std::vector<std::string> order;
  for (const Interval& iv : g_intervals) {
    if (hipEventSynchronize(iv.end) != hipSuccess) return -1;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, iv.begin, iv.end) != hipSuccess) return -1;
    auto it = agg.find(iv.name);
    if (it == agg.end()) {
      order.push_back(iv.name);
      agg[iv.name] = {ms, 1};
    } else {
      it->second.first += ms;
      it->second.second += 1;
    }
  }
  int32_t n = 0;
  for (const std::string& k : order) {
    if (n >= cap) break;
    snprintf(names + 32 * n, 32, "%s", k.c_str());
    total_ms[n] = static_cast<float>(agg[k].first);
    launches[n] = agg[k].second;
    ++n;
  }
  return n;
}
