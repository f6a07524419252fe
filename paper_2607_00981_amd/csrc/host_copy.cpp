// Device-to-host copies of whole tensors into ordinary (pageable) host memory.
//
// A plain hipMemcpy into pageable memory runs at about 8 GB/s here when the
// destination is freshly allocated (the runtime moves 1 MB at a time through
// one buffer and one thread, and every page of the destination is touched for
// the first time on that thread), against 57 GB/s into pinned memory.  The
// staged copy keeps the link busy: a few threads each own two pinned buffers,
// let the copy engine fill one while they move the other to its place, and
// take the next chunk from a shared counter.  Fresh destination, on MI355X,
// plain -> staged: 3 MB 0.71 -> 0.46 ms, 8 MB 0.80 -> 0.61 ms, 32 MB 3.16 ->
// 1.16 ms, 93 MB 9.4 -> 2.6 ms, 1 GB 101 -> 26 ms (41 GB/s; the first touch of
// the destination's pages is what is left).
//
// The pinned buffers belong to one pool per process of at most kSlots x
// kSlotBytes, shared by every context (threads that copy at the same time
// divide the buffers between them; one that gets none takes the plain copy),
// given back when the last object that may copy is destroyed.  Pinning them takes
// about as long as they save on 16 MB (1 ms: a first copy of 2 MB took 0.98 ms in
// place of 0.12), so they are allocated once that much has been copied.
#include "internal.h"

#include <algorithm>
#include <atomic>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

namespace cct {
namespace {

constexpr size_t kSlotBytes = (size_t)2 << 20;
constexpr int kSlots = 16;    // two for each of eight threads
constexpr int kWorkers = 8;
// Below this the runtime's own copy is as fast as starting the threads.
constexpr size_t kMinBytes = (size_t)2 << 20;
// Bytes copied, this copy's among them, from which the buffers are worth pinning.
constexpr size_t kWorthPinning = (size_t)16 << 20;

struct Pool {
  std::mutex mu;
  int users = 0;
  char* base = nullptr;   // kSlots x kSlotBytes of pinned memory
  bool failed = false;    // pinned memory was refused: plain copies until the pool is empty again
  size_t plain = 0;       // bytes copied without it
  bool busy[kSlots] = {};
};
Pool& pool() {
  static Pool* p = new Pool();  // never destroyed: objects may outlive static destructors
  return *p;
}

// Up to `want` pairs of buffers (two adjacent slots each) for a copy of `bytes`.
int take_pairs(int want, size_t bytes, char* out[kWorkers]) {
  Pool& p = pool();
  std::lock_guard<std::mutex> g(p.mu);
  if (!p.base) p.plain += bytes;
  if (!p.base && !p.failed && p.plain >= kWorthPinning) {
    void* b = nullptr;
    if (hipHostMalloc(&b, kSlots * kSlotBytes, hipHostMallocPortable) == hipSuccess) {
      p.base = (char*)b;
    } else {
      (void)hipGetLastError();
      p.failed = true;
    }
  }
  if (!p.base) return 0;
  int n = 0;
  for (int i = 0; i + 1 < kSlots && n < want; i += 2)
    if (!p.busy[i]) {
      p.busy[i] = true;
      out[n++] = p.base + (size_t)i * kSlotBytes;
    }
  return n;
}
void give_pairs(int n, char* const pairs[kWorkers]) {
  Pool& p = pool();
  std::lock_guard<std::mutex> g(p.mu);
  for (int k = 0; k < n; ++k) p.busy[(size_t)(pairs[k] - p.base) / kSlotBytes] = false;
}

struct Job {
  char* dst;
  const char* src;
  size_t bytes, chunk;
  long long nchunk;
  int dev;
  hipStream_t s;
  std::atomic<long long> next{0};
  std::atomic<int> err{0};
};

void worker(Job& j, char* pair) {
  hipError_t e = hipSetDevice(j.dev);
  hipEvent_t ev[2] = {nullptr, nullptr};
  for (int k = 0; k < 2 && e == hipSuccess; ++k) e = hipEventCreateWithFlags(&ev[k], hipEventDisableTiming);
  long long at[2] = {-1, -1};  // the chunk in flight into each buffer
  auto start = [&](int k) {
    at[k] = -1;
    if (j.err.load() != 0) return;
    const long long c = j.next.fetch_add(1);
    if (c >= j.nchunk) return;
    const size_t off = (size_t)c * j.chunk, len = std::min(j.chunk, j.bytes - off);
    e = hipMemcpyAsync(pair + (size_t)k * kSlotBytes, j.src + off, len, hipMemcpyDeviceToHost, j.s);
    if (e == hipSuccess) e = hipEventRecord(ev[k], j.s);
    if (e == hipSuccess) at[k] = c;
  };
  if (e == hipSuccess) start(0);
  if (e == hipSuccess) start(1);
  for (int k = 0; e == hipSuccess && at[k] >= 0; k ^= 1) {
    e = hipEventSynchronize(ev[k]);
    if (e != hipSuccess) break;
    const size_t off = (size_t)at[k] * j.chunk, len = std::min(j.chunk, j.bytes - off);
    std::memcpy(j.dst + off, pair + (size_t)k * kSlotBytes, len);
    start(k);
  }
  if (e != hipSuccess) {
    int none = 0;
    j.err.compare_exchange_strong(none, (int)e);
    (void)hipStreamSynchronize(j.s);  // no copy may be in flight into a buffer that goes back to the pool
  }
  for (hipEvent_t x : ev)
    if (x) (void)hipEventDestroy(x);
}

// Whether dst is ordinary host memory (pinned, managed or device memory takes
// the runtime's own copy, which is direct there).
bool pageable(const void* dst) {
  hipPointerAttribute_t a{};
  if (hipPointerGetAttributes(&a, dst) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  return a.type == hipMemoryTypeUnregistered;
}

}  // namespace

StageUser::StageUser() {
  Pool& p = pool();
  std::lock_guard<std::mutex> g(p.mu);
  ++p.users;
}
StageUser::~StageUser() {
  Pool& p = pool();
  std::lock_guard<std::mutex> g(p.mu);
  if (--p.users > 0) return;
  if (p.base) (void)hipHostFree(p.base);
  p.base = nullptr;
  p.failed = false;
  p.plain = 0;
}

hipError_t copy_to_host(void* dst, const void* src, size_t bytes, int dev, hipStream_t s) {
  if (bytes >= kMinBytes && pageable(dst)) {
    const int want = (int)std::min<size_t>(kWorkers, bytes >> 20);
    char* pairs[kWorkers];
    const int n = take_pairs(want, bytes, pairs);
    if (n > 0) {
      Job j;
      j.dst = (char*)dst;
      j.src = (const char*)src;
      j.bytes = bytes;
      // at least two chunks per thread, in whole 64 KB pieces
      const size_t even = (bytes / (2 * (size_t)n) + 65535) / 65536 * 65536;
      j.chunk = std::min(kSlotBytes, even);
      j.nchunk = (long long)((bytes + j.chunk - 1) / j.chunk);
      j.dev = dev;
      j.s = s;
      std::thread th[kWorkers];
      int started = 1;
      try {
        for (; started < n; ++started) th[started] = std::thread(worker, std::ref(j), pairs[started]);
      } catch (...) {
        // fewer threads than wanted: the ones that run take all chunks
      }
      int cur = 0;
      const bool have_cur = hipGetDevice(&cur) == hipSuccess;
      worker(j, pairs[0]);
      if (have_cur) (void)hipSetDevice(cur);
      for (int k = 1; k < started; ++k) th[k].join();
      give_pairs(n, pairs);
      return (hipError_t)j.err.load();
    }
  }
  const hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, s);
  return e != hipSuccess ? e : hipStreamSynchronize(s);
}

}  // namespace cct
