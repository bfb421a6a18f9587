// Device scratch of the allocation-free decode step (spec_step_noalloc): a
// file-scope device array of 69 MiB that every GPU the library
// runs on holds until the process ends.  In host code the array's name is
// only a stand-in; its device address on the current GPU is looked up once
// per device with hipGetSymbolAddress and cached, and only that address is
// ever handed to kernels.
#include <mutex>

#include "internal.h"

namespace spec {

static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes + kStaticScratchRoom];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices];  // device address of `scratch` per device, once looked up
}  // namespace

hipError_t static_scratch(void** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));  // with `dev` current
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

}  // namespace spec
