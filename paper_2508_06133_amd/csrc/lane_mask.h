// Stores of some of a wavefront's lanes without a branch.
//
// A branch that depends on the lane, anywhere inside a loop, makes the compiler carry the exits of the loops around it as
// flags in scalar registers, which are set and tested at every turn (half of the scalar instructions of the kernels that
// are one wavefront's chain of small steps).  With the lanes masked in place every branch of such a loop is the same for all of them,
// and the compiler (told to leave such branches alone, see SOURCE_FLAGS in build.py) emits them as written.
//
// `mask` has a bit per lane; lanes outside it store nothing, whatever their address.  LDS instructions of a wavefront are served in
// order, so the compiler's own reads before and after need no wait for these stores.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

// The LDS address of p (what a ds instruction takes).
__device__ __forceinline__ unsigned lds_at(const void *p)
{
    return (unsigned)(size_t)(const __attribute__((address_space(3))) void *)p;
}

// (the same in all lanes, and in scalar registers whether the compiler knows that or not)
__device__ __forceinline__ unsigned long long scalar_mask(unsigned long long mask)
{
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)mask);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(mask >> 32));
    return ((unsigned long long)hi << 32) | lo;
}

#define KVS_MASKED_DS(NAME, TYPE, INSTRUCTION)                                          \
    __device__ __forceinline__ void NAME(unsigned long long mask, const void *p, TYPE v) \
    {                                                                                   \
        unsigned long long all;                                                         \
        asm volatile("s_and_saveexec_b64 %[all], %[mask]\n" INSTRUCTION " %[p], %[v]\n" \
                     "s_mov_b64 exec, %[all]\n"                                         \
                     : [all] "=&s"(all)                                                 \
                     : [mask] "s"(scalar_mask(mask)), [p] "v"(lds_at(p)), [v] "v"(v)                 \
                     : "memory", "scc");                                                \
    }
KVS_MASKED_DS(put_b32, unsigned, "ds_write_b32")
KVS_MASKED_DS(put_b64, unsigned long long, "ds_write_b64")
KVS_MASKED_DS(or_b32, unsigned, "ds_or_b32")
#undef KVS_MASKED_DS

__device__ __forceinline__ void put_global(unsigned long long mask, int32_t *p, int v)
{
    unsigned long long all;
    asm volatile("s_and_saveexec_b64 %[all], %[mask]\n"
                 "global_store_dword %[p], %[v], off\n"
                 "s_mov_b64 exec, %[all]\n"
                 : [all] "=&s"(all)
                 : [mask] "s"(scalar_mask(mask)), [p] "v"(p), [v] "v"(v)
                 : "memory", "scc");
}

}  // namespace
