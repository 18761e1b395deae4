// Device memory that may not be there.
#pragma once

#include <hip/hip_runtime.h>

namespace dlx {

// hipMalloc; where it fails, *out is null and no error is left behind: the runtime keeps the last one, also through
// calls that succeed, and the check after the next launch would report it as that launch's.
inline bool device_alloc(void** out, size_t bytes) {
  if (hipMalloc(out, bytes) == hipSuccess) return true;
  *out = nullptr;
  (void)hipGetLastError();
  return false;
}

}  // namespace dlx
