// What the launchers share.
#pragma once

#include <hip/hip_ext.h>

#include <atomic>

#include "d2ft_common.h"

namespace d2ft {

// How many workgroups of a kernel the current device holds at once, and that the kernel may use its dynamic LDS there: both belong
// to a device's copy of the kernel, so they are settled on its first launch on that device.  One static object per kernel;
// several threads may call it together (they would ask for the same twice).
class KernelLimits {
public:
    hipError_t get(const void* kern, int threads, size_t lds, int* workgroups) {
        int dev = 0, cus = 0, per_cu = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < kDevices && (*workgroups = known_[dev].load()) > 0) return hipSuccess;
        if ((e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) != hipSuccess) return e;
        if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
        if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, threads, lds)) != hipSuccess) return e;
        *workgroups = cus * (per_cu < 1 ? 1 : per_cu);
        if (dev < kDevices) known_[dev].store(*workgroups);
        return hipSuccess;
    }

private:
    static constexpr int kDevices = 32;   // beyond: asked for every time
    std::atomic<int> known_[kDevices] = {};
};

// a multiple of the eight XCDs, so that ids with the same value mod 8 stay on one of them
inline int in_eights(int workgroups) { return workgroups < 8 ? 8 : workgroups / 8 * 8; }

// A launch that an event waits for (launch_signal_next) carries the event as its own completion signal.
template <typename Kernel, typename... Args>
hipError_t launch_signalling(Kernel kern, dim3 grid, dim3 block, size_t lds, hipStream_t s, const Args&... args) {
    if (hipEvent_t ev = launch_signal_take()) hipExtLaunchKernelGGL(kern, grid, block, lds, s, nullptr, ev, 0, args...);
    else hipLaunchKernelGGL(kern, grid, block, lds, s, args...);
    return hipGetLastError();
}

inline bool mult8(long v) { return (v & 7) == 0; }
inline bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace d2ft
