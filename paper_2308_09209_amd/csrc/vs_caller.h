// vs_caller.h -- callers' buffers that a runtime copy takes anywhere and a kernel
// only on its own device.
#pragma once
#include <cstddef>
#include <cstdint>

#include <hip/hip_runtime.h>

namespace vs {

// p .. p + bytes lies in one allocation of the current device's memory: kernels may
// address it.  Buffers on another device (no peer access is asked for), in host memory
// or past their allocation's end are left to hipMemcpyAsync, which copies or refuses
// them.  Two look-ups in the runtime's table, no device work, allowed under capture.
inline bool kernel_reaches(const void* p, size_t bytes)
{
    int dev = 0;
    hipPointerAttribute_t a;
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    const bool ok = p && hipGetDevice(&dev) == hipSuccess && hipPointerGetAttributes(&a, p) == hipSuccess &&
                    a.type == hipMemoryTypeDevice && a.device == dev &&
                    hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)p) == hipSuccess &&
                    (uintptr_t)p - (uintptr_t)base <= size && bytes <= size - ((uintptr_t)p - (uintptr_t)base);
    if (!ok) (void)hipGetLastError();   // an unknown pointer is no error of the call's
    return ok;
}

}  // namespace vs
