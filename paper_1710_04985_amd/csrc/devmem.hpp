// Device memory of the library.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>

namespace sptrsv {

// Allocates `bytes` (at least one) on the current device; contents undefined.
// Large blocks come from a store of freed ones where one fits.  A failure is
// the returned status alone: it is not left behind as the thread's last error.
hipError_t dev_alloc(void** p, int64_t bytes);

// Returns memory of dev_alloc once the device that holds it is idle (as
// hipFree waits).  Large blocks go to the store.  Safe from any thread.
void dev_free(void* p);

// Gives back all that the store keeps.  Safe from any thread.
void dev_release();

}  // namespace sptrsv
