// A barrier over the grid of a launch whose workgroups are all resident, and what the kernels that use it have in common.
#pragma once
#include "common.hpp"

namespace sun {

constexpr int kCounters = 16;       // arrivals are spread over this many counters, 128 bytes apart
constexpr uint32_t kSpinLimit = 1u << 22;  // polls (about a microsecond each) before a workgroup stops waiting

// The kernel's arguments, read again where they are used: all of them kept in registers across the phases do not fit.
template <class T>
__device__ __forceinline__ const T& kernel_args() {
    auto p = (const __attribute__((address_space(4))) T*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const T*)p;
}

// The lane, read again where it is used: what can be computed from it would otherwise be computed once in front of the layers
// and carried through them in registers that the phases need.
__device__ __forceinline__ int lane_here() {
    int l = threadIdx.x & 63;
    asm volatile("" : "+v"(l));
    return l;
}

__device__ __forceinline__ void grid_arrive(uint32_t* counters) {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // what this wave has stored is in memory
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_fetch_add(counters + (blockIdx.x % kCounters) * 32, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Wave 0 polls until every workgroup has arrived `times` times.  The wait ends by itself: the grid is resident, and past
// kSpinLimit (a device in trouble) the workgroup goes on, marks the step and waits no more.  fresh: what this compute unit's caches
// hold of other workgroups' data is dropped as well.
__device__ __forceinline__ void grid_wait(uint32_t* counters, uint32_t times, int* dead, bool fresh = false) {
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0) {
        const uint32_t lane = lane_here();
        const uint32_t want = lane < kCounters ? times * ((gridDim.x + kCounters - 1 - lane) / kCounters) : 0u;
        uint32_t* mine = counters + min(lane, (uint32_t)kCounters - 1) * 32;
#pragma unroll 1
        for (uint32_t n = 0; !*(volatile int*)dead; ++n) {
            if (__all(ld_agent(mine) >= want)) break;
            if (n == kSpinLimit) {
                if (lane == 0) *dead = 1;
                break;
            }
        }
        if (fresh) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    asm volatile("" ::: "memory");
    __syncthreads();
    asm volatile("" ::: "memory");
}

}  // namespace sun
