// Device memory of the library's objects.
#include <cstdint>

#include "internal.h"

namespace cct {

void* device_alloc(size_t bytes, cct_alloc_fn alloc, cct_free_fn free_fn, void* user, const char** why) {
  void* p = nullptr;
  const char* msg = "hipMalloc failed";
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
  }
  if (!p) {
    // the refusal is answered by a smaller request or by an error code; left
    // pending, the check after the next launch would report it
    (void)hipGetLastError();
    if (why) *why = msg;
  }
  return p;
}

}  // namespace cct
