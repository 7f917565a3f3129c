// What the HIP runtime knows about memory that a caller hands over.
#include "lora_internal.h"

namespace lora {

bool allocation_holds(const void *p, size_t bytes)
{
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)p) != hipSuccess) {
        (void)hipGetLastError();  // memory that HIP does not know: not an error of the caller's
        return false;
    }
    const uintptr_t first = (uintptr_t)p, from = (uintptr_t)base;
    return first >= from && first - from <= size && bytes <= size - (first - from);
}

bool pinned_holds(const void *host, size_t bytes)
{
    hipPointerAttribute_t at;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || hipPointerGetAttributes(&at, host) != hipSuccess) {
        (void)hipGetLastError();  // as above
        return false;
    }
    // pinned for this device (another's pinned memory need not be mapped here), at the same address
    return at.type == hipMemoryTypeHost && at.devicePointer == host && at.device == dev && allocation_holds(host, bytes);
}

}  // namespace lora
