// lbm_readout.cpp -- large results to pageable host memory.
//
// A copy to pageable memory runs at the speed of one CPU thread, which also
// takes the page faults of a new destination: 537 MB take 31 ms into pages that
// are there, 52 ms into new 2 MiB pages and 127 ms into new 4 KiB pages, while the
// link moves them in 11. Here READ_THREADS threads each bring chunks into two
// pinned slots of their own and copy one out while the other fills: 14, 14 and
// 29 ms (2 threads 14, 25 and 72; 12 threads 14, 14 and 21; chunks of 4 MiB 12,
// 12 and 32 at twice the pinned memory).
//
// Taken from READ_MIN bytes on: below, what the slots cost the first read-out
// (4 ms) is more than the copy.
#include <algorithm>
#include <atomic>
#include <cstring>
#include <exception>
#include <thread>

#include "lbm_device.h"
#include "lbm_internal.h"

namespace lbm {

namespace {

constexpr int READ_THREADS = 6;
constexpr size_t READ_CHUNK = size_t(2) << 20;
constexpr size_t READ_MIN = size_t(64) << 20;

// true where the copy goes to memory that the runtime does not know (a program's
// own pages) on a stream that is not being captured
bool pageable(const void *dst, hipStream_t stream) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) {
    (void)hipGetLastError();
    return false;
  }
  hipPointerAttribute_t at;
  if (hipPointerGetAttributes(&at, dst) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  return at.type == hipMemoryTypeUnregistered;
}

bool prepare(ReadStage &s) {
  if (s.mem) return true;
  if (hipHostMalloc(&s.mem, READ_CHUNK * 2 * READ_THREADS, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    s.mem = nullptr;
    return false;
  }
  return true;
}

struct Job {
  const ReadPart *parts;
  size_t chunks;
  hipStream_t stream;
  int device;
  std::atomic<size_t> next{0};
  std::atomic<int> error{hipSuccess};
};

// the chunk's bytes: parts are cut into chunks one after another
size_t chunk_at(const Job &j, size_t c, char *&dst, const char *&src) {
  const ReadPart *p = j.parts;
  for (;; ++p) {
    const size_t n = (p->bytes + READ_CHUNK - 1) / READ_CHUNK;
    if (c < n) break;
    c -= n;
  }
  dst = (char *)p->dst + c * READ_CHUNK;
  src = (const char *)p->src + c * READ_CHUNK;
  return std::min(READ_CHUNK, p->bytes - c * READ_CHUNK);
}

// One thread's share: chunks from the common counter, in two slots in turn. Every
// copy that it has started has ended when it returns.
void share(Job &j, char *slots) {
  hipEvent_t ev[2] = {nullptr, nullptr};
  char *dst[2] = {nullptr, nullptr};
  size_t bytes[2] = {0, 0};
  hipError_t e = hipSetDevice(j.device);
  for (int k = 0; k < 2 && e == hipSuccess; ++k)
    e = hipEventCreateWithFlags(&ev[k], hipEventDisableTiming);
  for (int k = 0; e == hipSuccess; k ^= 1) {
    const size_t c = j.error.load(std::memory_order_relaxed) == hipSuccess
                         ? j.next.fetch_add(1, std::memory_order_relaxed)
                         : j.chunks;
    if (c < j.chunks) {
      const char *src;
      bytes[k] = chunk_at(j, c, dst[k], src);
      e = hipMemcpyAsync(slots + k * READ_CHUNK, src, bytes[k], hipMemcpyDeviceToHost, j.stream);
      if (e == hipSuccess) e = hipEventRecord(ev[k], j.stream);
    }
    const int o = k ^ 1;
    if (bytes[o] && e == hipSuccess) {
      e = hipEventSynchronize(ev[o]);
      if (e == hipSuccess) std::memcpy(dst[o], slots + o * READ_CHUNK, bytes[o]);
      bytes[o] = 0;
    }
    if (c >= j.chunks && !bytes[k]) break;
  }
  if (e != hipSuccess) {
    j.error.store(e, std::memory_order_relaxed);
    (void)hipGetLastError();
    (void)hipStreamSynchronize(j.stream);  // the slots are free again before they can be freed
  }
  for (int k = 0; k < 2; ++k)
    if (ev[k]) (void)hipEventDestroy(ev[k]);
}

}  // namespace

hipError_t read_out(ReadStage *stage, const ReadPart *parts, int nparts, hipStream_t stream) {
  size_t total = 0, chunks = 0;
  bool staged = stage != nullptr;
  for (int k = 0; k < nparts; ++k) {
    total += parts[k].bytes;
    chunks += (parts[k].bytes + READ_CHUNK - 1) / READ_CHUNK;
  }
  // hipStreamPerThread is another stream in each thread: the copies of the others
  // would not wait for what the caller's holds
  staged = staged && total >= READ_MIN && stream != hipStreamPerThread;
  for (int k = 0; k < nparts && staged; ++k) staged = pageable(parts[k].dst, stream);
  Job j;
  staged = staged && hipGetDevice(&j.device) == hipSuccess && prepare(*stage);
  if (!staged) {
    hipError_t e = hipSuccess;
    for (int k = 0; k < nparts && e == hipSuccess; ++k)
      e = hipMemcpyAsync(parts[k].dst, parts[k].src, parts[k].bytes, hipMemcpyDeviceToHost, stream);
    return e;
  }
  j.parts = parts;
  j.chunks = chunks;
  j.stream = stream;
  char *slots = (char *)stage->mem;
  std::thread workers[READ_THREADS];
  const int want = (int)std::min<size_t>(READ_THREADS, std::max(1u, std::thread::hardware_concurrency() / 2));
  int n = 1;
  try {  // with fewer threads (none left, or no memory for one) the others take more chunks
    for (; n < want; ++n)
      workers[n] = std::thread([&j, slots, n] { share(j, slots + 2 * n * READ_CHUNK); });
  } catch (const std::exception &) {
  }
  share(j, slots);
  for (int t = 1; t < READ_THREADS; ++t)
    if (workers[t].joinable()) workers[t].join();
  return (hipError_t)j.error.load();
}

void read_stage_free(ReadStage &s) {
  if (s.mem) (void)hipHostFree(s.mem);
  s.mem = nullptr;
}

}  // namespace lbm
