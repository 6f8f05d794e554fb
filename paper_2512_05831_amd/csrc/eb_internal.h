// Shared by the library's sources; not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

namespace eb_detail {

// Record a printf-style message as the calling thread's last error
// (eb_last_error) and return code.  The message goes into a fixed
// thread-local buffer (truncated if longer): no allocation, no exception.
int fail(int code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));

// The calling thread's last message ("" if none).
const char *last_error();

// What an entry point returns when something below it threw (its own paths
// allocate nothing, so only a runtime library could): EB_ERR_NOMEM.
int unexpected_exception(const char *who);

// A wave-uniform load through the scalar cache, of memory that the kernel does
// not write.
template <typename T>
__device__ __forceinline__ T scalar_load(const T *p)
{
    return *(const __attribute__((address_space(4))) T *)(uint64_t)p;
}

} // namespace eb_detail
