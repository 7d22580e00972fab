// Host-side helpers shared by the entry points.
#pragma once
#include <hip/hip_runtime.h>
#include "../../include/fog.h"

// Maps the runtime's sticky launch error (if any) to a status code.
static inline fog_status fog_launch_status() { return hipGetLastError() == hipSuccess ? FOG_OK : FOG_ERR_HIP; }

// Number of compute units of the current device (256 where there is none), queried once per process.
static inline int fog_compute_units() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cus = n;
  }
  return cus;
}
