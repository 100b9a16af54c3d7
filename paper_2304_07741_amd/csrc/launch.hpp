// Kernel launch wrapper.  Normally a plain launch; while a timed call is running (see
// canvas_dag_set_timing) the launch carries a start and a stop event, so that the elapsed time between
// the two is the kernel's own execution time on the device.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <atomic>
#include <cstdint>

namespace canvas {

// More than 64 KB of dynamic LDS must be asked for, once per kernel and device.  `asked`: the kernel's own, a bit per device (beyond the 64th: asked for
// with every launch).  A refusal is the error that the caller finds behind its launches (hipGetLastError), and the next launch asks again.
inline void allow_lds(std::atomic<uint64_t>& asked, const void* kernel, int bytes) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return;
    const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
    if (asked.load(std::memory_order_relaxed) & bit) return;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) == hipSuccess) asked.fetch_or(bit, std::memory_order_relaxed);
}

struct TimingEvents {
    hipEvent_t start = nullptr, stop = nullptr;
};
extern thread_local TimingEvents g_timing;

}  // namespace canvas

#define CANVAS_LAUNCH(kernel, grid, block, shmem, stream, ...)                                                       \
    do {                                                                                                             \
        if (::canvas::g_timing.start)                                                                                \
            hipExtLaunchKernelGGL(kernel, grid, block, shmem, stream, ::canvas::g_timing.start, ::canvas::g_timing.stop, 0, \
                                  __VA_ARGS__);                                                                      \
        else                                                                                                         \
            hipLaunchKernelGGL(kernel, grid, block, shmem, stream, __VA_ARGS__);                                     \
    } while (0)
