// The limit of a kernel's dynamic LDS, which has to be raised above 64 KB.  It belongs to the kernel on one device.
#pragma once
#include <hip/hip_runtime_api.h>

namespace mg {

// done: the devices on which the kernel's limit has been raised, a bit each, kept beside the launch (calls enqueue one at a
// time).  Devices beyond the bits are asked every time.
inline hipError_t raise_lds_limit(const void* kern, int bytes, unsigned long& done) {
  int dev = 0;
  const hipError_t d = hipGetDevice(&dev);
  if (d != hipSuccess) return d;
  const unsigned long bit = dev < 64 ? 1ul << dev : 0ul;
  if (done & bit) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done |= bit;
  return e;
}

}  // namespace mg
