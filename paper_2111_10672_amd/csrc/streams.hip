// The streams beside the caller's that a model's weight gradients run on.
//
// HIP maps the streams of a process onto a few hardware queues (four by default), and two streams on one queue run one
// after the other.  A model with one stream of its own therefore shares its queue with the caller's stream one time in
// four, and loses all overlap (encoder of 32 x 128 tokens, everything but the embedding: 4.30 ms with the two streams on
// different queues, 5.80 ms on the same one).  The runtime does not say which queue a stream is on, so it is found out: a
// model has three streams (of two, made one after the other, both were seen on one queue), and asks for a caller's stream: a
// kernel there runs for 100 us, and an empty one goes to each of the three behind it.  One that ended well before the long
// kernel did runs beside it; behind the same queue it could not have.  Nothing waits on the host: the events' times are
// read by the first call that finds them there.  Where none was seen beside it (the other queues may have been busy with
// another model's work) the question is asked again, ever more rarely; and an answer holds for a number of calls only,
// because a handle says nothing about the stream behind it: one that was destroyed may come back on another queue.
#include "model.h"

namespace spb {
namespace {

constexpr float kBesideMs = 0.01f;   // ahead of the long kernel's end by this much: one queue's order never looks like it
// Questions come at least 1, 2, 4, ... and then this many calls after one another, however often s changes and whatever
// was seen; an answer holds for as many calls (100 us in 4096 steps of 1 ms are 0.002 %).
constexpr long kLongest = 4096;
constexpr long long kTick = 100;     // wall_clock64 ticks per microsecond (100 MHz)

// 100 us; the iteration count bounds it without a clock.
__global__ void spin_kernel() {
  const long long start = wall_clock64();
  for (int it = 0; it < 100000 && wall_clock64() - start < 100 * kTick; ++it) __builtin_amdgcn_s_sleep(1);
}
__global__ void empty_kernel() {}

// Says what became of this launch: the thread's last error may be an earlier call's, and is then its caller's to read.
bool launch(void (*kernel)(), hipStream_t s) {
  void* none[1] = {nullptr};
  return hipLaunchKernel(reinterpret_cast<const void*>(kernel), dim3(1), dim3(1), none, 0, s) == hipSuccess;
}

// While it lives, this thread's calls are not refused (nor end the capture) because another thread captures a graph.
struct Uncaptured {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  Uncaptured() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  ~Uncaptured() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

}  // namespace

SideStreams::~SideStreams() { release(); }

void SideStreams::release() {
  for (auto& q : side_) if (q) { (void)hipStreamDestroy(q); q = nullptr; }
  for (auto& e : ran_) if (e) { (void)hipEventDestroy(e); e = nullptr; }
  if (looked_) { (void)hipEventDestroy(looked_); looked_ = nullptr; }
}

bool SideStreams::create() {
  bool ok = hipEventCreate(&looked_) == hipSuccess;
  for (int c = 0; ok && c < kSide; ++c)
    ok = hipStreamCreateWithFlags(&side_[c], hipStreamNonBlocking) == hipSuccess && hipEventCreate(&ran_[c]) == hipSuccess &&
         launch(empty_kernel, side_[c]);     // a stream's first launch is slow
  if (ok) return true;
  (void)hipGetLastError();
  release();
  return false;
}

void SideStreams::ask(hipStream_t s) {
  bool ok = launch(spin_kernel, s) && hipEventRecord(looked_, s) == hipSuccess;
  for (int c = 0; ok && c < kSide; ++c) ok = launch(empty_kernel, side_[c]) && hipEventRecord(ran_[c], side_[c]) == hipSuccess;
  if (!ok) { (void)hipGetLastError(); return; }
  waiting_ = true;
  next_ = calls_ + wait_;
  if (wait_ < kLongest) wait_ *= 2;
}

void SideStreams::answer() {
  const hipError_t e = hipEventQuery(looked_);
  if (e != hipSuccess) (void)hipGetLastError();
  if (e == hipErrorNotReady) return;
  waiting_ = false;
  for (int i = 0; i < kSide && !known_; ++i) {
    const int c = (pick_ + i) % kSide;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, ran_[c], looked_) != hipSuccess) (void)hipGetLastError();   // still behind something: not known to run beside
    else if (ms > kBesideMs) { pick_ = c; known_ = true; until_ = calls_ + kLongest; }
  }
}

hipStream_t SideStreams::beside(hipStream_t s) {
  ++calls_;
  if (known_ && s == for_ && calls_ < until_) return side_[pick_];
  const Uncaptured guard;
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) { (void)hipGetLastError(); return side_[pick_]; }
  if (st != hipStreamCaptureStatusNone) return side_[pick_];
  if (hipPeekAtLastError() != hipSuccess) return side_[pick_];      // an earlier call's error: neither ours to clear nor to be taken for ours
  if (!side_[0] && !create()) return nullptr;                       // (the next forward pass tries again)
  if (known_ || s != for_) { for_ = s; known_ = waiting_ = false; }
  if (waiting_) answer();
  else if (calls_ >= next_) ask(s);
  return side_[pick_];
}

}  // namespace spb
