// A HIP runtime that records instead of running, for tests of the library's host
// side on machines without a GPU. Loaded globally before liblbm.so, its
// definitions take the place of the runtime's: memory is host memory that no
// kernel ever writes, copies move nothing, and every kernel launch and copy is
// one line of a log that recorder_take returns.
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <thread>

namespace {

struct State {
  std::mutex m;
  std::string log;
  std::map<const void *, std::string> kernels;
  std::thread::id caller = std::this_thread::get_id();
};
State &state() {
  static State *s = new State;  // outlives the library's own static objects
  return *s;
}
std::atomic<int> capturing{0}, mallocs_left{-1}, async_left{-1}, launches_left{-1}, error{hipSuccess};
thread_local int news_left = -1;  // this thread's operator new: -1 never fails, else counts down
struct Config {
  dim3 grid, block;
  size_t shmem;
  hipStream_t stream;
};
thread_local Config pushed;
float last_ms = 1.0f;  // what events say about the last launch

void line(const char *fmt, const char *what, unsigned a, unsigned b, int c, hipStream_t s) {
  char buf[1024];
  State &st = state();
  const int left = news_left;
  news_left = -1;  // the log's own memory does not count
  std::lock_guard<std::mutex> lock(st.m);
  std::snprintf(buf, sizeof(buf), fmt, what, a, b, c, (unsigned long long)(uintptr_t)s,
                st.caller == std::this_thread::get_id() ? "caller" : "other");
  st.log += buf;
  news_left = left;
}

}  // namespace

void *operator new(size_t n) {
  if (news_left >= 0 && news_left-- == 0) throw std::bad_alloc();
  void *p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

extern "C" {

// ---- for the test
size_t recorder_take(char *out, size_t n) {  // the log so far, then empty
  State &st = state();
  std::lock_guard<std::mutex> lock(st.m);
  const size_t len = st.log.size();
  if (out && len < n) {
    std::memcpy(out, st.log.c_str(), len + 1);
    st.log.clear();
  }
  return len;
}
void recorder_capturing(int on) { capturing = on; }
void recorder_mallocs_left(int n) { mallocs_left = n; }  // hipMalloc calls that succeed, -1: all
void recorder_async_left(int n) { async_left = n; }  // hipMallocAsync calls that succeed, -1: all
void recorder_launches_left(int n) { launches_left = n; }  // kernel launches that succeed, -1: all
void recorder_news_left(int n) { news_left = n; }    // this thread's allocations that succeed

// ---- kernels
void **__hipRegisterFatBinary(const void *) {
  static void *h;
  return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *fn, char *, const char *name, unsigned, void *,
                           void *, void *, void *, int *) {
  state().kernels[fn] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t shmem, hipStream_t s) {
  pushed = Config{g, b, shmem, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shmem, hipStream_t *s) {
  *g = pushed.grid;
  *b = pushed.block;
  *shmem = pushed.shmem;
  *s = pushed.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 g, dim3 b, void **args, size_t, hipStream_t s) {
  if (launches_left >= 0 && launches_left-- == 0) {
    launches_left = 0;
    error = hipErrorLaunchFailure;
    return hipErrorLaunchFailure;
  }
  const std::string &name = state().kernels[fn];
  // strips of five and six steps are fastest in small workgroups, the others in large ones
  const bool more = name.find("ELi5EEE") != std::string::npos || name.find("ELi6EEE") != std::string::npos;
  last_ms = 1.0f + 0.001f * (more ? b.x : 512 - (b.x < 512 ? b.x : 512));
  // the tile kernel's third argument is its number of steps
  const int steps = name.find("11tile_kernel") != std::string::npos ? *(int *)args[2] : 0;
  line("launch %s %u %u %d %llx %s\n", name.c_str(), g.x, b.x, steps, s);
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int block, size_t) {
  *n = 512 / block > 0 ? 512 / block : 1;
  return hipSuccess;
}

// ---- memory
static hipError_t take_memory(void **p, size_t n) {
  *p = std::aligned_alloc(4096, (n + 4095) / 4096 * 4096);  // untouched pages cost nothing
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipMalloc(void **p, size_t n) {
  if (mallocs_left >= 0 && mallocs_left-- == 0) {
    mallocs_left = 0;
    return hipErrorOutOfMemory;
  }
  return take_memory(p, n);
}
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t) {
  if (async_left >= 0 && async_left-- == 0) {
    async_left = 0;
    return hipErrorOutOfMemory;
  }
  return take_memory(p, n);
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return take_memory(p, n); }
hipError_t hipFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipFreeAsync(void *p, hipStream_t) { return std::free(p), hipSuccess; }
hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *src, size_t, hipMemcpyKind kind, hipStream_t s) {
  char from[32];
  std::snprintf(from, sizeof(from), "%llx", (unsigned long long)(uintptr_t)src);
  line("copy %s %u %u %d %llx %s\n", from, 0, 0, (int)kind, s);
  return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) {
  return hipMemcpyAsync(d, s, n, k, nullptr);
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *) {
  std::memset(a, 0, sizeof(*a));
  a->type = hipMemoryTypeUnregistered;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) { return take_memory(p, 1 << 20); }

// ---- device, streams, events, graphs
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return (hipError_t)error.exchange(hipSuccess); }
const char *hipGetErrorString(hipError_t) { return "recorded"; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
  std::memset(p, 0, sizeof(*p));
  std::strcpy(p->gcnArchName, "gfx950");
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  *s = (hipStream_t)std::malloc(8);
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { return std::free(s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { return *g = (hipGraph_t)8, hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  return *e = (hipGraphExec_t)8, hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) {
  line("%s graph %u %u %d %llx %s\n", "launch", 0, 0, 0, s);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = (hipEvent_t)8, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = last_ms, hipSuccess; }

}  // extern "C"
