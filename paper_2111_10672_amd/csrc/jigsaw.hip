// Iteration-level placement of training tasks (Sec. 3 of the paper, "Scheduling Algorithm") and its gang
// baseline.  Host code only; it lives in this library because its inputs are what the library measures (a step's
// time and workspace per depth) and its callers are the same.  The rules are stated with the declaration in
// spb.h; this file is one way to carry them out.  200 jobs on 45 devices, 47 k tasks: see Device and place_tasks.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <limits>
#include <set>
#include <tuple>
#include <utility>
#include <vector>

#include "model.h"

namespace spb {
namespace {

// A device's busy time as disjoint intervals in ascending order.  Tasks mostly start where another one ended; such
// neighbours are kept as one interval (`join`), so a lookup passes real gaps only (200 jobs on 45 devices: 430 intervals
// and 2.4 passed per lookup on average).  Joining changes no answer as long as t + d > t for every time t and
// duration d of the plan (the caller checks): no task then fits between an end and an equal start.
struct Device {
  std::vector<double> start, end;
  bool join;
  mutable size_t near = 0;          // where the last lookup ended; a job's chain asks for ascending times, so the next is close

  explicit Device(bool joins) : join(joins) {}

  // index of the first interval that ends after t: everything before it lies wholly before t
  size_t first_after(double t) const {
    const size_t n = end.size();
    size_t lo = std::min(near, n), hi = lo, step = 1;          // widened until end[lo - 1] <= t < end[hi]
    while (lo > 0 && end[lo - 1] > t) { hi = lo - 1; lo -= std::min(lo, step); step *= 2; }
    for (step = 1; hi < n && end[hi] <= t; step *= 2) { lo = hi + 1; hi = std::min(n, hi + step); }
    return near = std::upper_bound(end.begin() + lo, end.begin() + hi, t) - end.begin();
  }
  // earliest t >= ready with [t, t + d) free, or any time >= give_up once the answer is known to be no earlier than that
  double earliest(double ready, double d, double give_up = std::numeric_limits<double>::infinity()) const {
    double t = ready;
    for (size_t i = first_after(ready), n = end.size(); i < n && t < give_up; ++i) {
      if (end[i] <= t) continue;
      if (start[i] >= t + d) break;
      t = end[i];
    }
    return t;
  }
  bool free_at(double t, double d) const {
    const size_t i = first_after(t);
    return i == end.size() || start[i] >= t + d;
  }
  void take(double from, double to) {
    size_t i = std::lower_bound(start.begin(), start.end(), from) - start.begin();
    if (!join) {      // ascending by (start, end)
      while (i < start.size() && start[i] == from && end[i] < to) ++i;
      start.insert(start.begin() + i, from); end.insert(end.begin() + i, to);
      return;
    }
    const bool before = i > 0 && end[i - 1] == from, after = i < start.size() && start[i] == to;
    if (before && after) { end[i - 1] = end[i]; start.erase(start.begin() + i); end.erase(end.begin() + i); }
    else if (before) end[i - 1] = to;
    else if (after) start[i] = from;
    else { start.insert(start.begin() + i, from); end.insert(end.begin() + i, to); }
  }
};

// Whether t + d > t holds for every time and duration of a plan: no time exceeds the bound (everything one after the
// other, every task moved), and the shortest duration is at least one unit in the bound's last place.
bool may_join(const spb_sched_job* jobs, int n_jobs, double gamma) {
  double bound = 0.0, shortest = std::numeric_limits<double>::infinity();
  for (int j = 0; j < n_jobs; ++j) bound = std::max(bound, jobs[j].arrival);
  for (int j = 0; j < n_jobs; ++j) {
    double sum = 0.0;
    for (int w = 0; w < jobs[j].workers; ++w) {
      const double d = jobs[j].durations[w];
      sum += d + gamma * jobs[j].model_size;
      shortest = std::min(shortest, d);
    }
    bound += sum * jobs[j].iterations * jobs[j].workers;     // (a gang holds its devices for its slowest task)
  }
  bound *= 2.0;                                              // rounding of the sums
  return std::isfinite(bound) && bound + shortest / 2.0 > bound;
}

// The ready tasks in the order in which they are placed.  A task's weight belongs to its (job, worker), and a job has
// one iteration in the queue at a time, so the order is a fixed ranking of those pairs and the queue a set of ranks:
// one bit each, with one bit per 64 of them above.
struct ReadyQueue {
  std::vector<uint64_t> bits, words;
  explicit ReadyQueue(size_t n) : bits(n / 64 + 1), words(bits.size() / 64 + 1) {}
  void insert(size_t r) { bits[r / 64] |= 1ull << (r % 64); words[r / 4096] |= 1ull << (r / 64 % 64); }
  bool pop(size_t& r) {
    for (size_t a = 0; a < words.size(); ++a) {
      if (!words[a]) continue;
      const size_t b = a * 64 + __builtin_ctzll(words[a]);
      r = b * 64 + __builtin_ctzll(bits[b]);
      bits[b] &= bits[b] - 1;
      if (!bits[b]) words[a] &= words[a] - 1;
      return true;
    }
    return false;
  }
};

struct Progress {               // of one job's current iteration
  int iteration = 0;
  double release = 0.0;         // earliest start of its tasks
  int pending = 0;              // tasks not placed yet
  double latest_end = 0.0;
};

int validate(const spb_sched_job* jobs, int n_jobs, int n_machines, double gamma, double capacity, bool gang) {
  if (n_machines < 1 || !(gamma >= 0.0) || !(capacity >= 0.0)) { set_error("spb_schedule_tasks: n_machines %d, gamma %g, capacity %g", n_machines, gamma, capacity); return SPB_ERR_INVALID_ARG; }
  for (int j = 0; j < n_jobs; ++j) {
    const spb_sched_job& q = jobs[j];
    if (q.workers < 1 || !q.durations || !q.resources || q.iterations < 0 || !(q.arrival >= 0.0) || !(q.model_size >= 0.0)) {
      set_error("spb_schedule_tasks: job %d: workers %d, iterations %d, arrival %g, model size %g or a null array", j, q.workers, q.iterations, q.arrival, q.model_size);
      return SPB_ERR_INVALID_ARG;
    }
    for (int w = 0; w < q.workers; ++w)
      if (!(q.durations[w] > 0.0) || !std::isfinite(q.durations[w]) || !(q.resources[w] >= 0.0) || !(q.resources[w] <= capacity)) {
        set_error("spb_schedule_tasks: job %d worker %d: duration %g, resource %g (capacity %g)", j, w, q.durations[w], q.resources[w], capacity);
        return SPB_ERR_INVALID_ARG;
      }
    if (gang && q.workers > n_machines) { set_error("spb_schedule_tasks: job %d: a gang of %d workers on %d devices", j, q.workers, n_machines); return SPB_ERR_INVALID_ARG; }
  }
  return SPB_OK;
}

spb_sched_task* place_tasks(const spb_sched_job* jobs, int n_jobs, int n_machines, double gamma, spb_sched_task* out) {
  std::vector<Device> dev(n_machines, Device(may_join(jobs, n_jobs, gamma)));
  std::vector<Progress> prog(n_jobs);
  struct Slot { double key; int job, worker; };                // key: -resource * duration
  std::vector<Slot> order;
  std::vector<size_t> first(n_jobs);                           // of a job's workers in `rank` and `last`
  for (int j = 0; j < n_jobs; ++j) {
    first[j] = order.size();
    for (int w = 0; w < jobs[j].workers; ++w) order.push_back({-(jobs[j].resources[w] * jobs[j].durations[w]), j, w});
  }
  std::sort(order.begin(), order.end(), [](const Slot& a, const Slot& b) { return std::tie(a.key, a.job, a.worker) < std::tie(b.key, b.job, b.worker); });
  std::vector<size_t> rank(order.size());
  for (size_t r = 0; r < order.size(); ++r) rank[first[order[r].job] + order[r].worker] = r;
  std::vector<int> last(order.size(), -1);                     // device of each worker's previous iteration
  ReadyQueue ready(order.size());
  auto release_iteration = [&](int j, int i, double when) {
    prog[j].iteration = i; prog[j].release = when; prog[j].pending = jobs[j].workers; prog[j].latest_end = 0.0;
    for (int w = 0; w < jobs[j].workers; ++w) ready.insert(rank[first[j] + w]);
  };
  for (int j = 0; j < n_jobs; ++j) if (jobs[j].iterations > 0) release_iteration(j, 0, jobs[j].arrival);
  for (size_t r; ready.pop(r);) {
    const int j = order[r].job, w = order[r].worker;
    const spb_sched_job& q = jobs[j];
    const double d = q.durations[w];
    int& prev = last[first[j] + w];
    // Earlier start wins; at the same start the previous device, then the lower index.  So the previous device is asked
    // first; the others start no sooner than `moved_ready`, and one of them has to be strictly earlier than the best so far.
    // Without a previous device the first one always counts: an infinite or undefined time is earlier than nothing.
    const double release = prog[j].release, moved_ready = release + gamma * q.model_size;
    int best_m = prev;
    double best_start = prev >= 0 ? dev[prev].earliest(release, d) : std::numeric_limits<double>::infinity();
    for (int m = 0; m < n_machines && (best_m < 0 || best_start > moved_ready); ++m) {
      if (m == prev) continue;
      const double start = dev[m].earliest(moved_ready, d, best_start);
      if (start < best_start || best_m < 0) { best_m = m; best_start = start; }
    }
    spb_sched_task& t = *out++;
    t.job = j; t.iteration = prog[j].iteration; t.worker = w; t.machine = best_m; t.moved = (prev >= 0 && best_m != prev) ? 1 : 0;
    t.start = best_start; t.end = best_start + d; t.held_until = t.end;
    if (!std::isnan(t.start)) dev[best_m].take(t.start, t.end);   // (no time lies inside an interval that is not a number)
    prev = best_m;
    prog[j].latest_end = prog[j].pending == q.workers ? t.end : std::max(prog[j].latest_end, t.end);
    if (--prog[j].pending == 0 && prog[j].iteration + 1 < q.iterations) release_iteration(j, prog[j].iteration + 1, prog[j].latest_end);
  }
  return out;
}

spb_sched_task* place_gangs(const spb_sched_job* jobs, int n_jobs, int n_machines, double gamma, spb_sched_task* out) {
  std::vector<Device> dev(n_machines, Device(may_join(jobs, n_jobs, gamma)));
  std::vector<std::vector<int>> last(n_jobs);
  std::vector<double> weight(n_jobs), slowest(n_jobs);
  using Key = std::tuple<double, int, int>;                    // (-(sum of resources) * slowest duration, job, iteration)
  std::set<Key> ready;
  std::vector<double> release(n_jobs, 0.0);
  for (int j = 0; j < n_jobs; ++j) {
    const spb_sched_job& q = jobs[j];
    last[j].assign(q.workers, -1);
    double sum = 0.0, mx = 0.0;
    for (int w = 0; w < q.workers; ++w) { sum += q.resources[w]; mx = std::max(mx, q.durations[w]); }
    weight[j] = sum * mx; slowest[j] = mx;
    if (q.iterations > 0) { release[j] = q.arrival; ready.insert(Key(-weight[j], j, 0)); }
  }
  std::vector<double> gaps(n_machines);
  std::vector<int> assign, free_list;
  while (!ready.empty()) {
    const Key k = *ready.begin();
    ready.erase(ready.begin());
    const int j = std::get<1>(k), i = std::get<2>(k);
    const spb_sched_job& q = jobs[j];
    const double rel = release[j], hold = slowest[j];
    // (infinity times zero: nothing is known to be moved, and no start is too early for it)
    const double delay = gamma * q.model_size, moved_ready = std::isnan(delay) ? rel : rel + delay;
    // A gang starts at the earliest time at which all previous devices are free for `hold`, or - not before the model
    // can have moved - at which as many devices as it has workers are.  Both are found by jumps: from a time t, no start
    // lies before the latest (the workers-th) of the devices' own next gaps, and when that is t itself, it is the start.
    double t_found = moved_ready;
    for (;;) {
      for (int m = 0; m < n_machines; ++m) gaps[m] = dev[m].earliest(t_found, hold);
      std::nth_element(gaps.begin(), gaps.begin() + (q.workers - 1), gaps.end());
      if (gaps[q.workers - 1] <= t_found) break;
      t_found = gaps[q.workers - 1];
    }
    if (i > 0)
      for (double t = rel; t < t_found;) {
        double all = t;
        for (int m : last[j]) all = std::max(all, dev[m].earliest(t, hold, t_found));
        if (all == t) { t_found = t; break; }
        t = all;
      }
    free_list.clear();
    for (int m = 0; m < n_machines; ++m) if (dev[m].free_at(t_found, hold)) free_list.push_back(m);
    assign.assign(q.workers, -1);
    for (int w = 0; w < q.workers; ++w) {              // keep the previous device where it is free
      const int prev = i > 0 ? last[j][w] : -1;
      auto it = prev >= 0 ? std::find(free_list.begin(), free_list.end(), prev) : free_list.end();
      if (it != free_list.end()) { assign[w] = prev; free_list.erase(it); }
    }
    size_t next = 0;
    for (int w = 0; w < q.workers; ++w) {
      const int prev = i > 0 ? last[j][w] : -1;
      if (assign[w] < 0) assign[w] = free_list[next++];   // the others move
      spb_sched_task& t = *out++;
      t.job = j; t.iteration = i; t.worker = w; t.machine = assign[w]; t.moved = (i > 0 && assign[w] != prev) ? 1 : 0;
      t.start = t_found; t.end = t_found + q.durations[w]; t.held_until = t_found + hold;
      dev[assign[w]].take(t.start, t.held_until);
      last[j][w] = assign[w];
    }
    if (i + 1 < q.iterations) { release[j] = t_found + hold; ready.insert(Key(-weight[j], j, i + 1)); }
  }
  return out;
}

}  // namespace
}  // namespace spb

extern "C" int spb_schedule_tasks(const spb_sched_job* jobs, int32_t n_jobs, int32_t n_machines, double gamma, double capacity,
                                  int32_t gang, spb_sched_task* out, int64_t cap, int64_t* n_out, double* makespan) {
  using namespace spb;
  if (n_jobs < 0 || (n_jobs > 0 && !jobs) || !n_out || !makespan || cap < 0 || (cap > 0 && !out)) { set_error("spb_schedule_tasks: null argument or negative count"); return SPB_ERR_INVALID_ARG; }
  if (int rc = validate(jobs, n_jobs, n_machines, gamma, capacity, gang != 0)) return rc;
  int64_t total = 0;
  for (int j = 0; j < n_jobs; ++j) total += (int64_t)jobs[j].workers * jobs[j].iterations;
  *n_out = total;
  if (total > cap) { set_error("spb_schedule_tasks: %lld tasks, room for %lld", (long long)total, (long long)cap); return SPB_ERR_INVALID_ARG; }
  const spb_sched_task* end = gang ? place_gangs(jobs, n_jobs, n_machines, gamma, out) : place_tasks(jobs, n_jobs, n_machines, gamma, out);
  if (end - out != total) { set_error("spb_schedule_tasks: internal error, %lld of %lld tasks placed", (long long)(end - out), (long long)total); return SPB_ERR_STATE; }
  double latest = 0.0;
  for (const spb_sched_task* t = out; t != end; ++t) latest = std::max(latest, t->held_until);
  *makespan = latest;
  return SPB_OK;
}
