// The streams beside the caller's that weight gradients run on.
//
// HIP maps the streams of a process onto a few hardware queues (four by default), and two streams on one queue run one
// after the other.  A stream created per model therefore shares its queue with the caller's stream one time in four,
// and such a model loses all overlap (encoder of 32 x 128 tokens, everything but the embedding: 4.30 ms with the two
// streams on different queues, 5.80 ms on the same one).  The runtime does not say which queue a stream is on, so it is
// found out: per device there are four streams, and the first time a caller's stream is seen, one thread on it looks
// for flags that a kernel on each of the four sets.  A stream behind the same queue cannot set its flag before the
// looking ends (at the latest after 200 us, once per caller's stream and process).  Nothing waits on the host: the
// answer lands in pinned memory and is used from the first call that finds it there.
#include <mutex>
#include <vector>

#include "model.h"

namespace spb {
namespace {

constexpr int kSide = 4;           // streams per device: one more than can share the caller's queue
constexpr int kProbes = 64;        // caller's streams told apart per device; later ones take the streams in turn
constexpr int kMaxDevices = 64;
constexpr int kDone = 1 << 16;
constexpr long long kTick = 100;   // wall_clock64 ticks per microsecond (100 MHz)

__device__ unsigned g_flags[kProbes * kSide];   // each slot is used once, so they start at zero

__global__ void probe_set_kernel(int slot, int c) {
  if (c >= 0) __hip_atomic_store(&g_flags[slot * kSide + c], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Ends when all flags are up, 20 us after all but one are, or after 200 us; the iteration count bounds it without a clock.
__global__ void probe_look_kernel(int slot, int* result) {
  const long long start = wall_clock64();
  long long enough = 0;
  int seen = 0;
  for (int it = 0; it < 100000; ++it) {
    seen = 0;
    int n = 0;
    for (int c = 0; c < kSide; ++c)
      if (__hip_atomic_load(&g_flags[slot * kSide + c], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT)) { seen |= 1 << c; ++n; }
    const long long now = wall_clock64();
    if (n == kSide || now - start > 200 * kTick) break;
    if (n == kSide - 1) {
      if (enough == 0) enough = now;
      else if (now - enough > 20 * kTick) break;
    }
  }
  __hip_atomic_store(result, seen | kDone, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Both say what became of this launch: the thread's last error may be an earlier call's, and is then its caller's to read.
hipError_t set(int slot, int c, hipStream_t s) {
  void* args[] = {&slot, &c};
  return hipLaunchKernel(reinterpret_cast<const void*>(probe_set_kernel), dim3(1), dim3(1), args, 0, s);
}
hipError_t look(int slot, int* result, hipStream_t s) {
  void* args[] = {&slot, &result};
  return hipLaunchKernel(reinterpret_cast<const void*>(probe_look_kernel), dim3(1), dim3(1), args, 0, s);
}

struct DeviceStreams {
  bool ok = false;
  hipStream_t side[kSide] = {};
  int* result = nullptr;            // pinned, one word per probe
  std::vector<hipStream_t> seen;    // caller's streams, in slot order
};
std::mutex g_lock;
DeviceStreams g_devices[kMaxDevices];

void create(DeviceStreams& d) {
  // (an allocation would otherwise fail, and end the capture, while another thread captures a graph)
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  bool ok = hipHostMalloc(reinterpret_cast<void**>(&d.result), kProbes * sizeof(int), hipHostMallocDefault) == hipSuccess;
  for (int c = 0; ok && c < kSide; ++c) ok = hipStreamCreateWithFlags(&d.side[c], hipStreamNonBlocking) == hipSuccess;
  if (ok) {
    for (int i = 0; i < kProbes; ++i) d.result[i] = 0;
    for (int c = 0; ok && c < kSide; ++c) ok = set(0, -1, d.side[c]) == hipSuccess;   // a stream's first launch is slow
  }
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  d.ok = ok;
  if (ok) return;
  (void)hipGetLastError();
  for (auto& q : d.side) if (q) { (void)hipStreamDestroy(q); q = nullptr; }
  if (d.result) { (void)hipHostFree(d.result); d.result = nullptr; }
}

}  // namespace

hipStream_t side_stream_beside(hipStream_t s, unsigned turn) {
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices) { (void)hipGetLastError(); return nullptr; }
  std::lock_guard<std::mutex> guard(g_lock);
  DeviceStreams& d = g_devices[device];
  if (!d.ok) create(d);
  if (!d.ok) return nullptr;      // (the next forward pass tries again)
  size_t slot = 0;
  while (slot < d.seen.size() && d.seen[slot] != s) ++slot;
  if (slot == d.seen.size() && slot < (size_t)kProbes) {
    if (look((int)slot, d.result + slot, s) != hipSuccess) { (void)hipGetLastError(); return d.side[turn % kSide]; }
    d.seen.push_back(s);
    for (int c = 0; c < kSide; ++c)
      if (set((int)slot, c, d.side[c]) != hipSuccess) (void)hipGetLastError();
  }
  const int found = slot < (size_t)kProbes ? __atomic_load_n(d.result + slot, __ATOMIC_ACQUIRE) : 0;
  int good[kSide], n = 0;
  for (int c = 0; c < kSide; ++c) if (found & (1 << c)) good[n++] = c;
  return n > 0 ? d.side[good[turn % n]] : d.side[turn % kSide];
}

}  // namespace spb
