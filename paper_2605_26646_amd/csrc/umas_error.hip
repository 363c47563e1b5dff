// Thread-local error message, the pinned staging ring for thin host arrays and the optional kernel timing aid of libumas.
#include <string.h>

#include <map>
#include <mutex>
#include <string>
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
  hipEvent_t read = nullptr;     // recorded behind the last kernel launched on this block, ...
  int device = 0;                // ... an event of this device
  bool in_flight = false;
};
StageSlot g_slots[ThinStage::kSlots];
int g_next_slot = 0;
std::mutex g_stage_mutex;
}  // namespace

umas_status ThinStage::begin(size_t bytes, hipStream_t st) {
  // a graph would read the block again when later calls have overwritten it
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  UMAS_HIP(hipStreamIsCapturing(st, &capture));
  UMAS_REQUIRE(capture == hipStreamCaptureStatusNone, UMAS_EINVAL, "a call that takes host arrays cannot be recorded into a graph: hip_stream is being captured");
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
    const hipError_t e = hipEventSynchronize(s.read);
    if (e != hipSuccess) return bail(e, "hipEventSynchronize");
    s.in_flight = false;
  }
  int device = 0;
  hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return bail(e, "hipGetDevice");
  if (s.read && s.device != device) {
    (void)hipEventDestroy(s.read);
    s.read = nullptr;
  }
  if (!s.read) {
    e = hipEventCreateWithFlags(&s.read, hipEventDisableTiming | hipEventDisableSystemFence);
    if (e != hipSuccess) return bail(e, "hipEventCreateWithFlags");
    s.device = device;
  }
  if (s.cap < bytes) {
    if (s.host) (void)hipHostFree(s.host);
    s.host = nullptr;
    s.cap = 0;
    size_t cap = 1 << 16;
    while (cap < bytes) cap <<= 1;
    void* p = nullptr;
    // coherent: a kernel reads the block, at the same address again four calls later, and must not find old lines in a cache
    e = hipHostMalloc(&p, cap, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent);
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

const char* ThinStage::lend() const { return g_slots[slot_].dev; }

umas_status ThinStage::launched(hipStream_t st, hipError_t e) {
  StageSlot& s = g_slots[slot_];
  const hipError_t r = hipEventRecord(s.read, st);   // whatever e is: it may be an older error, and the kernel runs
  s.in_flight = r == hipSuccess;
  if (r != hipSuccess) (void)hipStreamSynchronize(st);
  slot_ = -1;
  cur_ = nullptr;
  g_stage_mutex.unlock();
  if (e == hipSuccess) e = r;
  if (e != hipSuccess) return fail(UMAS_EHIP, "staging failed: %s", hipGetErrorString(e));
  return UMAS_OK;
}

namespace {
// The block is copied by a kernel that reads the pinned memory over the bus.  The runtime's own copy costs more at every size: below 16 KB it
// is a kernel too, but behind a hand-over on either side, above another engine's.  The event behind it is one without the system-wide
// fence, which nobody needs for a kernel that has only read and which holds the stream for 5 us (the calls around a batch of 49 152 tokens, two
// blocks of 2.4 and 0.5 KB: 100.5 us a pass with it, without an event 90.6; two such events without it cost 0.9 us of the 52 that the calls
// around 46 000 tokens take, and 2.3 of 528 around 25 million).
constexpr int kStageWords = 4;                 // 16-byte words a thread has in flight
__global__ void __launch_bounds__(256)
k_stage_copy(const uint4* __restrict__ from, uint4* __restrict__ dst, int64_t n16) {
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * (256 * kStageWords) + threadIdx.x;
  uint4 v[kStageWords];
#pragma unroll
  for (int k = 0; k < kStageWords; ++k)
    if (i0 + k * 256 < n16) v[k] = from[i0 + k * 256];
#pragma unroll
  for (int k = 0; k < kStageWords; ++k)
    if (i0 + k * 256 < n16) dst[i0 + k * 256] = v[k];
}
}  // namespace

umas_status ThinStage::flush(void* dst, size_t bytes, hipStream_t st) {
  if (!bytes) {
    abandon();
    return UMAS_OK;
  }
  const int64_t n16 = static_cast<int64_t>(bytes / 16);                // whole arrays of the carver: a multiple of 256
  const unsigned n_wg = cdiv(static_cast<size_t>(n16), 256 * kStageWords);
  hipLaunchKernelGGL(k_stage_copy, dim3(n_wg), dim3(256), 0, st, reinterpret_cast<const uint4*>(lend()), static_cast<uint4*>(dst), n16);
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
