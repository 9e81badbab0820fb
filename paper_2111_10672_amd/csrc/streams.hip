// The streams beside the caller's that weight gradients run on.
//
// HIP maps the streams of a process onto a few hardware queues (four by default), and two streams on one queue run one
// after the other.  A stream made for the purpose therefore shares its queue with the caller's stream one time in four, and
// loses all overlap (encoder of 32 x 128 tokens, everything but the embedding: 4.30 ms with the two streams on different
// queues, 5.80 ms on the same one).  The runtime does not say which queue a stream is on, so it is found out: a side
// stream waits for the caller's and runs a kernel of 100 us, and the caller's runs an empty kernel that was enqueued behind
// that one.  If the empty one ended well before the long one did, the two run beside each other; on one queue it could not
// have.  Nothing waits on the host: the events' times are read by the first call that finds them there.  There is one side
// stream at first, and another (up to three) when none so far was seen beside the caller's: a stream takes 35 us to make
// and as long to destroy, and of two, made one after the other, both were seen on one queue.  Then the question is asked
// again, ever more rarely, since the caller's queue may only have been busy with other work.  An answer holds for a number
// of calls only, because a handle says nothing about the stream behind it: one that was destroyed may come back on another
// queue.
//
// Side streams belong to a caller's stream: the models that step on it run one after the other anyway, and going from one
// side stream to another on another queue costs up to 40 us a step (two encoders of 7 x 72 tokens in turn: 1.45 ms a step
// with their side streams on one queue, 1.49 ms on two).  Models on different callers' streams share none, so that neither
// waits for the other's work.  They are destroyed with the last model that holds on to them.
#include "model.h"

#include <algorithm>
#include <utility>

namespace spb {
namespace {

constexpr float kBesideMs = 0.01f;   // ended ahead of the long kernel by this much: one queue's order never looks like it
// Questions come at least 1, 2, 4, ... and then this many calls after one another, whatever was seen and whoever's streams
// these were before; an answer holds for as many calls (100 us in 4096 steps of 1 ms are 0.002 %).
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

// Side streams in use, by device and caller's stream.  (Never destroyed: models may outlive this file's statics.)
struct Registry {
  std::mutex lock;
  std::map<std::pair<int, hipStream_t>, std::weak_ptr<SideStreams>> of;
};
Registry& registry() { static Registry* r = new Registry; return *r; }

}  // namespace

SideStreams& CallersSides::of(hipStream_t s) {
  if (!uses_.empty() && uses_[0].caller == s) return *uses_[0].sides;
  for (size_t i = 1; i < uses_.size(); ++i)
    if (uses_[i].caller == s) { std::rotate(uses_.begin(), uses_.begin() + i, uses_.begin() + i + 1); return *uses_[0].sides; }
  Use u{s, 0, nullptr}, last{};
  if (hipGetDevice(&u.device) != hipSuccess) (void)hipGetLastError();
  if (uses_.size() == kKept) { last = std::move(uses_.back()); uses_.pop_back(); }
  Registry& r = registry();
  const std::lock_guard<std::mutex> hold(r.lock);
  for (auto it = r.of.begin(); it != r.of.end();) it = it->second.expired() ? r.of.erase(it) : std::next(it);
  // (one handle stands for as many streams as there are threads: not to be shared)
  const bool shared = s != hipStreamPerThread;
  const auto found = shared ? r.of.find({u.device, s}) : r.of.end();
  if (found != r.of.end()) u.sides = found->second.lock();
  if (!u.sides && last.sides && last.sides.use_count() == 1 && last.device == u.device) {   // no other model's: they move to s
    r.of.erase({last.device, last.caller});
    last.sides->forget();
    u.sides = std::move(last.sides);
  }
  if (!u.sides) u.sides = std::make_shared<SideStreams>();
  if (shared) r.of[{u.device, s}] = u.sides;
  uses_.insert(uses_.begin(), std::move(u));
  return *uses_[0].sides;
}

SideStreams::~SideStreams() {
  for (auto& x : side_) {
    if (x.stream) (void)hipStreamDestroy(x.stream);
    for (auto e : {x.asked, x.ran, x.passed}) if (e) (void)hipEventDestroy(e);
  }
}

// One more stream, if there may be and can be.
bool SideStreams::make() {
  if (made_ == kSide) return false;
  Side& x = side_[made_];
  if ((x.asked || hipEventCreateWithFlags(&x.asked, hipEventDisableTiming) == hipSuccess) && (x.ran || hipEventCreate(&x.ran) == hipSuccess) &&
      (x.passed || hipEventCreate(&x.passed) == hipSuccess) && hipStreamCreateWithFlags(&x.stream, hipStreamNonBlocking) == hipSuccess) {
    pick_ = made_++;
    return true;
  }
  (void)hipGetLastError();
  return false;
}

void SideStreams::ask(hipStream_t s) {
  next_ = calls_ + wait_;
  if (wait_ < kLongest) wait_ *= 2;
  waiting_ = true;
  for (int c = 0; c < made_ && waiting_; ++c) {       // one after the other: on s's queue one holds up s
    const Side& x = side_[c];
    waiting_ = hipEventRecord(x.asked, s) == hipSuccess && hipStreamWaitEvent(x.stream, x.asked, 0) == hipSuccess && launch(spin_kernel, x.stream) &&
               hipEventRecord(x.ran, x.stream) == hipSuccess && launch(empty_kernel, s) && hipEventRecord(x.passed, s) == hipSuccess;
  }
  if (!waiting_) (void)hipGetLastError();
}

void SideStreams::answer() {
  for (int i = 0; i < made_; ++i) {
    const int c = (pick_ + i) % made_;
    float ms = 0.f;
    const hipError_t e = hipEventElapsedTime(&ms, side_[c].passed, side_[c].ran);
    if (e != hipSuccess) (void)hipGetLastError();
    if (e == hipErrorNotReady) return;
    if (e == hipSuccess && ms > kBesideMs) { pick_ = c; known_ = true; until_ = calls_ + kLongest; return; }
  }
  waiting_ = false;
  (void)make();
}

hipStream_t SideStreams::beside(hipStream_t s) {
  const std::lock_guard<std::mutex> hold(lock_);
  ++calls_;
  if (known_ && calls_ < until_) return side_[pick_].stream;
  const Uncaptured guard;
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) { (void)hipGetLastError(); return side_[pick_].stream; }
  if (st != hipStreamCaptureStatusNone) return side_[pick_].stream;
  if (hipPeekAtLastError() != hipSuccess) return side_[pick_].stream;      // an earlier call's error: neither ours to clear nor to be taken for ours
  if (!made_ && !make()) return nullptr;                                   // (the next forward pass tries again)
  if (known_) known_ = waiting_ = false;
  if (waiting_) answer();
  if (!waiting_ && !known_ && calls_ >= next_) ask(s);
  return side_[pick_].stream;
}

void SideStreams::forget() {
  const std::lock_guard<std::mutex> hold(lock_);
  known_ = waiting_ = false;
}

}  // namespace spb
