// fgh_dispatch.hpp -- launch of a pass kernel with dynamic LDS and, while a pass is being timed, the
// profiler's events attached to the dispatch itself.
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <atomic>
#include <mutex>

#include "fgh_launch.hpp"

namespace fgh {

// Allow dynamic LDS above 64 KB for a kernel (gfx950 has 160 KB per compute unit).
inline hipError_t allow_lds(const void* fn, size_t bytes)
{
    if (bytes <= 65536) return hipSuccess;
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}
// The attribute of each kernel only ever rises, so that no attribute call is made while a stream
// is being captured into a graph once the largest size has been seen.  Raising is serialised per
// kernel: the recorded size is stored only after the call has succeeded and only while holding the
// kernel's lock, so concurrent launches from several threads (server workers, plan-time tuning)
// can neither lower the attribute nor record a size the attribute does not allow.
#define LAUNCH_LDS_T(KERNEL, GRID, THREADS, LDS, STREAM, ...)                                   \
    do {                                                                                        \
        static std::atomic<size_t> lds_set_{65536};                                            \
        static std::mutex lds_mu_;                                                              \
        if ((LDS) > lds_set_.load(std::memory_order_acquire)) {                                 \
            std::lock_guard<std::mutex> lds_lk_(lds_mu_);                                       \
            if ((LDS) > lds_set_.load(std::memory_order_relaxed)) {                             \
                hipError_t e_ = allow_lds(reinterpret_cast<const void*>(&KERNEL), (LDS));       \
                if (e_ != hipSuccess) return e_;                                                \
                lds_set_.store((LDS), std::memory_order_release);                               \
            }                                                                                   \
        }                                                                                       \
        if (g_pass_events.start) {                                                              \
            const PassEvents pe_ = g_pass_events;                                               \
            g_pass_events = PassEvents{};                                                       \
            hipExtLaunchKernelGGL(KERNEL, GRID, dim3(THREADS), (LDS), (STREAM), pe_.start, pe_.stop, 0, \
                                  __VA_ARGS__);                                                 \
        } else {                                                                                \
            hipLaunchKernelGGL(KERNEL, GRID, dim3(THREADS), (LDS), (STREAM), __VA_ARGS__);      \
        }                                                                                       \
    } while (0)
#define LAUNCH_LDS(KERNEL, GRID, LDS, STREAM, ...) \
    LAUNCH_LDS_T(KERNEL, GRID, kThreads, LDS, STREAM, __VA_ARGS__)

}  // namespace fgh
