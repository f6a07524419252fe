// Device memory of the library's objects, and the block that cct_energy_q keeps
// from one call to the next.
//
// One block per GPU whatever the number of contexts: a call takes it whole and
// gives it back when its stream has drained, so that calls of other contexts,
// streams and threads find it idle or do without.  It goes with the context that
// used it last, and before that to any allocation of the library that is refused.
#include <cstdint>
#include <mutex>

#include "internal.h"

namespace cct {
namespace {

struct Kept {
  void* p = nullptr;
  size_t bytes = 0;
  const void* user = nullptr;
  bool busy = false;
};
constexpr int kMaxDevices = 64;
struct Blocks {
  std::mutex mu;
  Kept dev[kMaxDevices];
};
Blocks& blocks() {
  static Blocks* b = new Blocks();  // never destroyed: objects may outlive static destructors
  return *b;
}

bool drop(Kept& k) {  // with the lock held
  if (!k.p || k.busy) return false;
  (void)hipFree(k.p);
  k = Kept{};
  return true;
}

// The idle block of the current device given back; false if there was none.
bool release_idle() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
  Blocks& b = blocks();
  std::lock_guard<std::mutex> g(b.mu);
  return drop(b.dev[dev]);
}

}  // namespace

void* device_alloc(size_t bytes, cct_alloc_fn alloc, cct_free_fn free_fn, void* user, const char** why) {
  const char* msg = "";
  auto attempt = [&]() -> void* {
    void* p = nullptr;
    if (alloc) {
      p = alloc(bytes, user);
      msg = "caller allocator: NULL";
      if ((uintptr_t)p & 255) {
        free_fn(p, user);
        p = nullptr;
        msg = "caller allocator: pointer not 256-byte aligned";
      }
    } else if (hipMalloc(&p, bytes) != hipSuccess) {
      p = nullptr;
      msg = "hipMalloc failed";
    }
    // the refusal is answered by a smaller request or by an error code; left
    // pending, the check after the next launch would report it
    if (!p) (void)hipGetLastError();
    return p;
  };
  void* p = attempt();
  if (!p && release_idle()) p = attempt();
  if (!p && why) *why = msg;
  return p;
}

hipError_t device_mem_info(size_t* free_b, size_t* total_b) {
  const hipError_t e = hipMemGetInfo(free_b, total_b);
  int dev = 0;
  if (e != hipSuccess || hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return e;
  Blocks& b = blocks();
  std::lock_guard<std::mutex> g(b.mu);
  if (!b.dev[dev].busy) *free_b += b.dev[dev].bytes;
  return e;
}

hipError_t kept_take(int dev, const void* user, size_t bytes, void** p, size_t* got) {
  if (dev < 0 || dev >= kMaxDevices) return hipErrorNotReady;
  Blocks& b = blocks();
  std::lock_guard<std::mutex> g(b.mu);
  Kept& k = b.dev[dev];
  if (k.busy) return hipErrorNotReady;
  if (k.bytes < bytes) {
    drop(k);
    if (hipMalloc(&k.p, bytes) != hipSuccess) {
      (void)hipGetLastError();
      k.p = nullptr;
      return hipErrorOutOfMemory;
    }
    k.bytes = bytes;
  }
  k.busy = true;
  k.user = user;
  *p = k.p;
  *got = k.bytes;
  return hipSuccess;
}

void kept_give(int dev) {
  Blocks& b = blocks();
  std::lock_guard<std::mutex> g(b.mu);
  b.dev[dev].busy = false;
}

void kept_drop(const void* user) {
  Blocks& b = blocks();
  std::lock_guard<std::mutex> g(b.mu);
  for (Kept& k : b.dev)
    if (k.user == user) drop(k);
}

}  // namespace cct
