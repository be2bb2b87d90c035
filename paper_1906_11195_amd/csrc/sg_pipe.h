// What the SK sweep pipelines (sg_sk.hip, sg_skg.hip) share: LDS accesses between
// roles of a workgroup, and waits that end.
#pragma once
#include "sg_internal.h"

#define SG_L __attribute__((address_space(3)))

namespace sg {

constexpr int kSpinLimit = 1 << 22; // bounded waits: a stuck pipeline aborts

// LDS accesses of a pipeline.  The LDS executes one wavefront's operations in
// order, so data written before a flag is there once the flag is seen, and data
// read after a flag is no older than it: the accesses only have to stay in program
// order, which volatile accesses do, with no wait between them.
template <class T>
__device__ __forceinline__ T lds_get(uint32_t off)
{
    return *(const volatile SG_L T*)(size_t)off;
}
template <class T>
__device__ __forceinline__ void lds_put(uint32_t off, T v)
{
    *(volatile SG_L T*)(size_t)off = v;
}

// One poll of a wait that has not been met yet: true when the wait must end
// without its condition (abort raised, or this wait was the one that ran out
// of polls: after kSpinLimit polls the pipeline is declared stuck, the abort
// flag, the word after `sync`, releases every other wait and is reported at the end
// of the kernel: a global atomic here would count as a memory operation that may be
// in flight after every wait, and make each wait for streamed words a wait for all).
__device__ __forceinline__ bool wait_giveup(uint32_t sync, int& spins)
{
    if (__builtin_amdgcn_readfirstlane(lds_get<int32_t>(sync + 4))) return true;
    if (++spins > kSpinLimit) {
        lds_put<int32_t>(sync + 4, 1);
        return true;
    }
    return false;
}

}  // namespace sg
