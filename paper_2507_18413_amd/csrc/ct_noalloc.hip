// ct_noalloc.hip -- device scratch of ct_propagate_batch_noalloc (include/ct.h).
//
// The batch entry point keeps its error word, the job descriptors and the
// schedules' scratch in memory it allocates per stream.  Its no-allocation variant takes them from one static device
// array instead: every GPU the library runs on holds its own copy until the
// process ends, and every no-allocation call on that GPU shares it.  Host
// code never passes the array's name to a kernel or a copy (on the host the
// name is a stand-in, not a device address): it asks the runtime for the
// current device's address of the array once per device and uses that.
#include <hip/hip_runtime.h>

#include <mutex>

#include "ct_device.h"

namespace ctk {

constexpr size_t NA_SCRATCH_BYTES = (size_t)16 << 20;

// [0, 256): the error word (the fourth); then the staging copy (2 MiB: the
// staged schedule's item counts and the descriptors); then the search-node or
// the staged schedule's scratch (the rest)
static __device__ __align__(256) char scratch[NA_SCRATCH_BYTES];

namespace {

constexpr int NA_MAX_DEVICES = 64;
std::mutex g_mu;
char* g_ptr[NA_MAX_DEVICES];

}  // namespace

// The current device's address of the scratch array and its size; the
// address is looked up on a device's first use and kept.
hipError_t noalloc_scratch(char** ptr, size_t* bytes) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= NA_MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_mu);
  if (!g_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_ptr[dev] = (char*)p;
  }
  *ptr = g_ptr[dev];
  *bytes = NA_SCRATCH_BYTES;
  return hipSuccess;
}

}  // namespace ctk
