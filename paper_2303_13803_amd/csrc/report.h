// How a kernel tells the host something (see mf_report): words stored straight into pinned memory that the host
// watches, a number last.
#pragma once
#include "internal.h"

namespace {

// The constant clock all of the device's dies share, in ticks of 1 / mf_ctx::clock_khz ms.
__device__ __forceinline__ unsigned long long device_time() { return wall_clock64(); }

// The first thread of a launch notes when it began.  times: null where nobody wants to know.
__device__ __forceinline__ void note_time(unsigned long long *times, int stage)
{
    if (times && (blockIdx.x | blockIdx.y | blockIdx.z | threadIdx.x) == 0u) times[stage] = device_time();
}

// Called by all lanes of one wavefront, which is all of the launch.
__device__ __forceinline__ void tell(const void *from, void *to, int words, int lane)
{
    for (int t = lane; t < words; t += 64) __hip_atomic_store((unsigned *)to + t, ((const unsigned *)from)[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void tell_number(unsigned *told, unsigned number, int lane)
{
    __threadfence_system();                             // what this wavefront has stored is there before the number is
    if (lane == 0) __hip_atomic_store(told, number, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace
