// The HIP calls liblbm.so makes, answered on the host: "device" memory is host
// memory, copies are done, kernels are not run but written down.  Loaded before
// the library (launch_util.py), so that a test without a GPU sees which kernels
// the library would launch, in what order, on which tables, and what else it
// asks of the runtime.
//
// rec_log() holds one line per call:
//   launch <kernel's mangled name> <grid> <block> <stream> <a0> <a1> <a2>
//     (a0..a2: the first three arguments, for kernels of a batch, which all
//     take pointers there)
//   copy <destination> <source> <bytes> <stream>
//   capture, graph, host_malloc <bytes>, host_free
#include <chrono>
#include <condition_variable>
#include <cstdarg>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <utility>

namespace {
struct Dim3 {
  uint32_t x, y, z;
};
std::map<const void*, std::string> kernels;
std::string text, preferred;
bool refuse_host_memory, holding;
int waiting;
std::mutex text_lock;
std::condition_variable changed;
// time: a launch of a kernel whose name holds `preferred` takes 1 ms, others 1 s
double clock_ms = 0;
thread_local Dim3 call_grid, call_block;
thread_local size_t call_shared;
thread_local void* call_stream;
thread_local int last_error;

void note(const char* fmt, ...) {
  std::lock_guard<std::mutex> lock(text_lock);
  char line[1024];
  va_list a;
  va_start(a, fmt);
  std::vsnprintf(line, sizeof line, fmt, a);
  va_end(a);
  text += line;
}
}  // namespace

extern "C" {

const char* rec_log() { return text.c_str(); }
void rec_clear() { text.clear(); }
void rec_prefer(const char* name) { preferred = name; }
void rec_hold(int on) {
  std::lock_guard<std::mutex> lock(text_lock);
  holding = on != 0;
  changed.notify_all();
}
int rec_wait_for(int calls) {
  std::unique_lock<std::mutex> lock(text_lock);
  return changed.wait_for(lock, std::chrono::seconds(60),
                          [&] { return waiting >= calls; })
             ? 0
             : 1;
}
void rec_refuse_host_memory(int on) { refuse_host_memory = on != 0; }

void** __hipRegisterFatBinary(const void*) {
  static void* handle;
  return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name,
                           unsigned, void*, void*, void*, void*, int*) {
  kernels[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shared, void* stream) {
  call_grid = g;
  call_block = b;
  call_shared = shared;
  call_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* shared, void** stream) {
  *g = call_grid;
  *b = call_block;
  *shared = call_shared;
  *stream = call_stream;
  return 0;
}
int hipLaunchKernel(const void* host, Dim3 g, Dim3 b, void** args, size_t,
                    void* stream) {
  const std::string& name = kernels[host];
  void* a[3] = {};
  if (name.find("k_batch_tile") != name.npos ||
      name.find("k_adjoint") != name.npos || name.find("k_sweep") != name.npos ||
      name.find("k_loss") != name.npos || name.find("k_tile_sum") != name.npos)
    for (int i = 0; i < 3; ++i) std::memcpy(&a[i], args[i], sizeof a[i]);
  note("launch %s %u %u %p %p %p %p\n", name.c_str(), g.x, b.x, stream, a[0],
       a[1], a[2]);
  clock_ms += !preferred.empty() && name.find(preferred) != name.npos ? 1 : 1e3;
  return 0;
}

int hipMemcpyAsync(void* dst, const void* src, size_t bytes, int, void* stream) {
  note("copy %p %p %zu %p\n", dst, src, bytes, stream);
  std::memmove(dst, src, bytes);
  return 0;
}
int hipHostMalloc(void** p, size_t bytes, unsigned) {
  note("host_malloc %zu\n", bytes);
  if (refuse_host_memory) return last_error = 2;  // out of memory
  *p = std::calloc(1, bytes);
  return 0;
}
int hipHostFree(void* p) {
  note("host_free\n");
  std::free(p);
  return 0;
}

int hipEventCreate(void** e) { return *e = new double(0), 0; }
int hipEventCreateWithFlags(void** e, unsigned) { return hipEventCreate(e); }
int hipEventDestroy(void* e) { return delete static_cast<double*>(e), 0; }
int hipEventRecord(void* e, void*) {
  if (!e) return 400;
  *static_cast<double*>(e) = clock_ms;
  return 0;
}
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) {
  *ms = (float)(*static_cast<double*>(b) - *static_cast<double*>(a));
  return 0;
}

int hipStreamCreateWithFlags(void** s, unsigned) { return *s = new char(0), 0; }
int hipStreamDestroy(void* s) { return delete static_cast<char*>(s), 0; }
int hipStreamSynchronize(void*) {
  std::unique_lock<std::mutex> lock(text_lock);
  ++waiting;
  changed.notify_all();
  changed.wait(lock, [] { return !holding; });
  --waiting;
  return 0;
}
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamBeginCapture(void*, int) { return note("capture\n"), 0; }
int hipStreamEndCapture(void*, void** g) { return *g = new char(0), 0; }
int hipGraphInstantiate(void** e, void*, void**, char*, size_t) {
  return *e = new char(0), 0;
}
int hipGraphDestroy(void* g) { return delete static_cast<char*>(g), 0; }
int hipGraphExecDestroy(void* e) { return delete static_cast<char*>(e), 0; }
int hipGraphLaunch(void*, void*) { return note("graph\n"), 0; }

int hipGetLastError() { return std::exchange(last_error, 0); }
const char* hipGetErrorString(int) { return "error"; }
int hipGetDevice(int* d) { return *d = 0, 0; }
int hipGetDevicePropertiesR0600(void*, int) { return 999; }  // unknown
int hipGetSymbolAddress(void**, const void*) { return 999; }

}  // extern "C"
