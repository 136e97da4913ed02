// Driver of table creation without host memory: the nth allocation of the
// calling thread inside ct_create_table throws std::bad_alloc, for every n.
// Linked against the built library (its allocations come here); needs no
// device: creation gets as far as its first device call.  Prints "alloc
// driver: ok" when every call returned CT_E_NOMEM, or the device's error once
// no allocation was left to fail.  Test infrastructure only.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <new>

#include "ct.h"

static thread_local int g_left = 0;  // allocations still to go; 0: none fails

void* operator new(std::size_t n) {
  if (g_left > 0 && --g_left == 0) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void* operator new(std::size_t n, const std::nothrow_t&) noexcept {
  if (g_left > 0 && --g_left == 0) return nullptr;
  return std::malloc(n ? n : 1);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

int main() {
  int count = 0;
  (void)hipGetDeviceCount(&count);  // the runtime's own first allocations
  int32_t lo[3] = {0, 0, 0}, ds[3] = {70, 3, 200}, tup[9] = {0, 1, 2, 69, 2, 199, 5, 0, 9};
  int bad = 0, nomem = 0;
  for (int32_t kind : {CT_KIND_POSITIVE, CT_KIND_NEGATIVE})
    for (int n = 1;; ++n) {
      ct_table* t = (ct_table*)1;
      g_left = n;
      const int st = ct_create_table(tup, 3, 3, lo, ds, nullptr, nullptr, kind, &t);
      const bool fired = g_left == 0;
      g_left = 0;
      if (t || (fired ? st != CT_E_NOMEM && st != CT_E_DEVICE : st != CT_E_DEVICE)) {
        std::printf("kind %d, allocation %d: status %d\n", kind, n, st);
        bad = 1;
      }
      nomem += st == CT_E_NOMEM;
      if (!fired || n > 1000) break;
    }
  if (!bad && nomem >= 6) std::printf("alloc driver: ok\n");
  return bad;
}
