// Device memory of the library's handles and setup scratch (memory.hip).
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstddef>

namespace fvpcg {

// Device memory, kept for reuse when freed.  Neither throws: frees run in
// destructors, and on the way out of a C entry point.
hipError_t pool_alloc(void** out, size_t bytes) noexcept;
void pool_free(void* p) noexcept;

}  // namespace fvpcg
