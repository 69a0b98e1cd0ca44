// Whether kernels of a device may address an array where it lies.
#include <hip/hip_runtime.h>

#include "runtime_internal.hpp"

namespace msdd_rt {

bool device_holds(int device, const void *p, size_t bytes)
{
    hipPointerAttribute_t a{};
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipPointerGetAttributes(&a, p) == hipSuccess && a.type == hipMemoryTypeDevice && a.device == device &&
        hipMemGetAddressRange(&base, &size, const_cast<void *>(p)) == hipSuccess) {
        const size_t at = (size_t)(static_cast<const char *>(p) - static_cast<const char *>(base));
        return at <= size && bytes <= size - at;
    }
    (void)hipGetLastError();   // the failed query is no error of the next launch
    return false;
}

}  // namespace msdd_rt
