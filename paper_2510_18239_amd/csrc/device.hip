// Properties of the current device that the launchers size their grids by.
#include "common.hpp"

namespace lime {

int compute_units() {
  static const int n = [] {
    int dev = 0, cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cu <= 0)
      cu = 256;
    return cu;
  }();
  return n;
}

hipError_t allow_lds(PerDevice& granted, const void* kernel, int bytes) {
  int device = -1;
  if (hipError_t e = hipGetDevice(&device); e != hipSuccess) return e;
  return granted.ensure(device, [&] { return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); });
}

}  // namespace lime
