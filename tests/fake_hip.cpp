// A stand-in for the HIP runtime that libspb.so runs on in a process without a GPU: kernels do nothing, every call is
// written down, and streams lie on four queues that each run one thing at a time, in a time of its own.  Built and driven by
// test_host_streams.py.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Stream { int id, queue; bool capturing; };
struct Event { int id; bool recorded; double at; };
constexpr int kQueues = 4, kNotReady = 600;
Stream g_null{0, 0, false};
double g_clock[kQueues], g_now;                 // when each queue is free; the host's time
int g_streams, g_events, g_live_streams, g_live_events, g_next_queue, g_last_error;
bool g_refuse_launches;
std::string g_log;
std::map<const void*, std::string> g_names;
std::vector<std::string> g_symbols;

struct Config { uint64_t grid_xy; uint32_t grid_z; uint64_t block_xy; uint32_t block_z; size_t lds; void* stream; };
thread_local Config g_config;

Stream* of(void* s) { return s ? static_cast<Stream*>(s) : &g_null; }
double& free_at(void* s) { return g_clock[of(s)->queue]; }
int fail(int e) { return g_last_error = e; }
void note(const char* what, const std::string& arg, int id) { g_log += what; g_log += ' '; g_log += arg; g_log += ' ' + std::to_string(id) + '\n'; }
}  // namespace

extern "C" {
struct dim3_ { uint32_t x, y, z; };

void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { g_names[host] = name; }
int __hipPushCallConfiguration(dim3_ grid, dim3_ block, size_t lds, void* stream) {
  std::memcpy(&g_config.grid_xy, &grid.x, 8); g_config.grid_z = grid.z;
  std::memcpy(&g_config.block_xy, &block.x, 8); g_config.block_z = block.z;
  g_config.lds = lds; g_config.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_* grid, dim3_* block, size_t* lds, void** stream) {
  std::memcpy(&grid->x, &g_config.grid_xy, 8); grid->z = g_config.grid_z;
  std::memcpy(&block->x, &g_config.block_xy, 8); block->z = g_config.block_z;
  *lds = g_config.lds; *stream = g_config.stream;
  return 0;
}
int hipLaunchKernel(const void* fn, dim3_, dim3_, void**, size_t, void* stream) {
  const std::string& name = g_names[fn];
  if (g_refuse_launches) return fail(719);
  note("launch", name, of(stream)->id);
  double& t = free_at(stream);
  t = (t > g_now ? t : g_now) + (name.find("spin") != std::string::npos ? 0.1 : 0.001);
  return 0;
}
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetSymbolAddress(void** p, const void*) { static char room[256]; *p = room; return 0; }
const char* hipGetErrorString(int) { return "an error"; }
int hipGetLastError() { const int e = g_last_error; g_last_error = 0; return e; }
int hipPeekAtLastError() { return g_last_error; }
int hipHostMalloc(void** p, size_t n, unsigned) { note("call", "hipHostMalloc", 0); *p = std::calloc(1, n); return 0; }
int hipHostFree(void* p) { std::free(p); return 0; }
int hipThreadExchangeStreamCaptureMode(int*) { return 0; }

int hipStreamCreateWithFlags(void** s, unsigned) {
  auto* q = new Stream{++g_streams, g_next_queue, false};
  g_next_queue = (g_next_queue + 1) % kQueues;
  ++g_live_streams;
  note("call", "hipStreamCreateWithFlags", q->id);
  *s = q;
  return 0;
}
int hipStreamDestroy(void* s) { --g_live_streams; delete static_cast<Stream*>(s); return 0; }
int hipStreamIsCapturing(void* s, int* st) { note("call", "hipStreamIsCapturing", of(s)->id); *st = of(s)->capturing; return 0; }
int hipEventCreateWithFlags(void** e, unsigned) { *e = new Event{++g_events, false, 0.0}; ++g_live_events; note("call", "hipEventCreate", g_events); return 0; }
int hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void* e) { --g_live_events; delete static_cast<Event*>(e); return 0; }
int hipEventRecord(void* e, void* s) {
  auto* ev = static_cast<Event*>(e);
  ev->recorded = true; ev->at = free_at(s) > g_now ? free_at(s) : g_now;
  note("record", std::to_string(ev->id), of(s)->id);
  return 0;
}
int hipStreamWaitEvent(void* s, void* e, unsigned) {
  auto* ev = static_cast<Event*>(e);
  if (ev->recorded && ev->at > free_at(s)) free_at(s) = ev->at;
  note("wait", std::to_string(ev->id), of(s)->id);
  return 0;
}
int hipEventQuery(void* e) { return static_cast<Event*>(e)->at <= g_now ? 0 : fail(kNotReady); }
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) {
  auto *x = static_cast<Event*>(a), *y = static_cast<Event*>(b);
  if (!x->recorded || !y->recorded) return fail(400);
  if (x->at > g_now || y->at > g_now) return fail(kNotReady);
  *ms = static_cast<float>(y->at - x->at);
  return 0;
}

// ---- what a test may set and read ----
void* fake_stream(int queue) { g_next_queue = queue; void* s; hipStreamCreateWithFlags(&s, 1); g_next_queue = (queue + 1) % kQueues; return s; }
void fake_next_queue(int q) { g_next_queue = q; }
void fake_error(int e) { g_last_error = e; }
void fake_refuse_launches(int on) { g_refuse_launches = on; }
void fake_capture(void* s, int on) { of(s)->capturing = on; }
void fake_move(void* s, int queue) { of(s)->queue = queue; }
void fake_busy(int queue, double ms) { g_clock[queue] = (g_clock[queue] > g_now ? g_clock[queue] : g_now) + ms; }
void fake_wait() { for (double t : g_clock) if (t > g_now) g_now = t; }      // the host waits for the device
void fake_pass(double ms) { g_now += ms; }
int fake_queue(int stream_id, void** streams, int n) { for (int i = 0; i < n; ++i) if (of(streams[i])->id == stream_id) return of(streams[i])->queue; return -1; }
int fake_id(void* s) { return of(s)->id; }
int fake_live_streams() { return g_live_streams; }
int fake_live_events() { return g_live_events; }
const char* fake_log() { return g_log.c_str(); }
void fake_clear() { g_log.clear(); }
}
