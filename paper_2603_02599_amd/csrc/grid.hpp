// A barrier over the grid of a launch whose workgroups are all resident, and what the kernels that use it have in common.
#pragma once
#include "common.hpp"

namespace sun {

// Arrivals are spread over this many counters, 128 bytes apart: what arrives on one counter is added up one after the other, and wave 0
// looks at all of them with one load, so a counter per lane is the most.  8 layers of the 8B shape with 4 / 8 / 16 / 32 / 64 counters, us:
// one request 961 / 928 / 908 / 889 / 884, five with 4-bit weights 762 / 716 / 686 / 668 / 663, sixteen 1261 / 1218 / 1180 / 1169 / 1163.
// A flag per workgroup, stored without an add and looked at four a lane (64 lines as here, or 16): 902 and 964, 680 and 730, 1179 and
// 1219.  A pause of 64 cycles between two looks: no difference.
constexpr int kCounters = 64;
static_assert(kCounters <= 64, "wave 0 polls one counter a lane");
constexpr uint32_t kSpinLimit = 1u << 25;  // polls (about a microsecond each) before a workgroup stops waiting

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

// A word of LDS that another wave has written, behind a barrier.  (Read as volatile it becomes a flat load and a wait for every load in
// flight.)
__device__ __forceinline__ int lds_word(const int* p) {
    return __hip_atomic_load((const __attribute__((address_space(3))) int*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// A workgroup that has given up a wait (given_up, LDS) arrives nowhere any more.
__device__ __forceinline__ void grid_arrive(uint32_t* counters, const int* given_up) {
    const int gone = lds_word(given_up);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // what this wave has stored is in memory
    __syncthreads();
    if (threadIdx.x == 0 && !gone)
        __hip_atomic_fetch_add(counters + (blockIdx.x % kCounters) * 32, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Wave 0 polls until every workgroup has arrived `times` times.  After `polls` polls in vain (something else holds a compute unit for that
// long) it gives up: *given_up, and *lost, where the others see it while they wait.  The workgroup arrives nowhere from then on, so
// nobody passes a wait that is not complete, whatever others make of complete data is right, and every wait ends.  The workgroup itself
// may go on to where it would store what others could take for a result, and looks at *given_up there, beside other loads from
// LDS (looked at behind every wait: 5 to 10 us a step of 8 layers).  fresh: what this compute unit's caches
// hold of other workgroups' data is dropped as well.
__device__ __forceinline__ void grid_wait(uint32_t* counters, uint32_t* lost, uint32_t times, uint32_t polls, int* given_up, bool fresh = false) {
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0) {
        const uint32_t lane = lane_here();
        const uint32_t want = lane < kCounters ? times * ((gridDim.x + kCounters - 1 - lane) / kCounters) : 0u;
        const uint32_t* mine = counters + min(lane, (uint32_t)kCounters - 1) * 32;
        bool all = false;
#pragma unroll 1
        for (uint32_t n = 1; n <= polls; ++n) {
            all = __all(ld_agent(mine) >= want);
            if (all || (n % 64 == 0 && ld_agent(lost))) break;
        }
        if (!all && lane == 0) {
            st_agent(lost, 1u);
            *given_up = 1;
        }
        if (fresh) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    asm volatile("" ::: "memory");
    __syncthreads();
    asm volatile("" ::: "memory");
}

}  // namespace sun
