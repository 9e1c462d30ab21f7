// Device memory of the library's handles and setup scratch (memory.hip).
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstddef>

namespace fvpcg {

// Device memory, kept for reuse when freed.
hipError_t pool_alloc(void** out, size_t bytes);
void pool_free(void* p);

}  // namespace fvpcg
