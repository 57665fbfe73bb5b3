// The fixed device array that stands in for the caller's workspace in
// ppr_matrix_noalloc.  It is alone in this file: a file's device code is a module
// of its own, which the runtime loads on a GPU with the first use there, so that
// only programs that make the call hold the array.
#include <mutex>

#include "internal.hpp"

namespace pprviz {

static __device__ __align__(256) unsigned char scratch[kScratchBytes + kScratchExtraBytes];
constexpr int kMaxDevices = 64;

// Host code never passes the array's name to a kernel: this resolves it once per
// device, with that device current, and keeps the device address.
ppr_status scratch_address(hipStream_t s, void** out) {
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    int dev = 0;
    if (s != nullptr) {
        hipDevice_t d = 0;
        PPRVIZ_HIP_TRY(hipStreamGetDevice(s, &d));
        dev = (int)d;
    } else {
        PPRVIZ_HIP_TRY(hipGetDevice(&dev));
    }
    if (dev < 0 || dev >= kMaxDevices) return PPR_EUNSUPPORTED;
    std::lock_guard<std::mutex> lock(mu);
    if (addr[dev] == nullptr) {
        int cur = 0;
        PPRVIZ_HIP_TRY(hipGetDevice(&cur));
        if (cur != dev) PPRVIZ_HIP_TRY(hipSetDevice(dev));
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != dev) PPRVIZ_HIP_TRY(hipSetDevice(cur));
        if (e != hipSuccess || p == nullptr) return PPR_EHIP;
        addr[dev] = p;
    }
    *out = addr[dev];
    return PPR_OK;
}

}  // namespace pprviz
