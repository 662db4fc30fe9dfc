// Device helpers shared by the timeline kernels: wavefront reductions and the mapping from a
// position of a candidate order to a request id.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/kvsched.h"
#include "kvsched_internal.h"

namespace {

constexpr int WAVE = 64;

template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xf, 0xf, false);
}

// Maximum over the 64 lanes; all lanes must be active.  Four DPP steps leave every lane of a
// 16-lane row with the row's maximum (quad swaps, then mirror within 8 and within 16); the
// four row results are combined on the scalar unit.
__device__ __forceinline__ int wave_max_i32(int v)
{
    v = max(v, dpp_mov<0xB1>(v));   // quad_perm [1,0,3,2]
    v = max(v, dpp_mov<0x4E>(v));   // quad_perm [2,3,0,1]
    v = max(v, dpp_mov<0x141>(v));  // row_half_mirror
    v = max(v, dpp_mov<0x140>(v));  // row_mirror
    const int a = __builtin_amdgcn_readlane(v, 0);
    const int b = __builtin_amdgcn_readlane(v, 16);
    const int c = __builtin_amdgcn_readlane(v, 32);
    const int d = __builtin_amdgcn_readlane(v, 48);
    return max(max(a, b), max(c, d));
}

// Device-scope atomics and stores issued so far have been performed.  They go through to where every compute unit
// sees them, so this is all that has to separate them from the atomic that announces them; a device-scope fence would
// write the whole L2 back as well (5 us behind a kernel that has just stored a few megabytes).
__device__ __forceinline__ void device_writes_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Results for the host, by one lane: stores that go through to its memory by themselves, so that nothing but their arrival separates
// them from the number that announces them.  (A system-scope release writes the L2 back:
// one order of 61 requests without a bound on the decodes 10.3 us a call, 9.6 so.)
__device__ __forceinline__ void to_host(int32_t *host, int value)
{
    __hip_atomic_store(host, value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// ... the longest decode, whether the decode lengths are few and the number in one store, behind which nothing waits
__device__ __forceinline__ void longest_to_host(int32_t *host, int longest, int seq, bool few = false)
{
    static_assert(KVS_H_OMAX == 0 && KVS_H_SEQ == 1, "one word of 64 bits");
    __hip_atomic_store((unsigned long long *)host, (unsigned long long)(unsigned)seq << 32 | (few ? 1u << 31 : 0u) | (unsigned)longest,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// What a length scan leaves behind, by one lane of a launch that has had none ahead of it (SimParams::scan_here).
template <class Params>
__device__ __forceinline__ void report_lengths(const Params &p, int longest, int flags)
{
    p.d_words[2 * KVS_W_STATUS_TURN + 1 - p.status_word] = 0;  // (the other one)
    p.d_words[KVS_W_STATUS_AT] = p.status_word;
    if (flags) atomicOr(&p.d_words[p.status_word], flags);
    p.d_words[KVS_W_OMAX] = longest;
    p.d_words[KVS_W_MINPOS] = 0x7fffffff;
    p.d_words[KVS_W_MAXPOS] = -1;
    if (p.host) longest_to_host(p.host, longest, p.seq);
}

// Are there at most KVS_FEW_LENGTHS different ones among the lanes' decode lengths?
__device__ __forceinline__ bool few_lengths(int o)
{
    unsigned long long others = ~0ull;
    for (int k = 0; k < KVS_FEW_LENGTHS && others != 0; ++k)
        others &= ~__builtin_amdgcn_ballot_w64(o == __builtin_amdgcn_readlane(o, __builtin_ctzll(others)));
    return others == 0;
}

// The request whose decode length is a lane's part of that sample.
__device__ __forceinline__ int sampled(int lane, int n) { return (int)(((long long)lane * n) >> 6); }

// (only what the host did not know: the end of a launch waits for the store, half a microsecond)
template <class Params>
__device__ __forceinline__ void report_few(const Params &p, bool few)
{
    if (few != (p.few_known != 0)) to_host(p.few_out, few ? 1 : 0);
}

// The flags that one request's lengths give (bound: the caller's on the decode lengths, or 0).
__device__ __forceinline__ int length_flags(int s, int o, int M, int bound)
{
    return (s < 1 || o < 1 || (long long)s + (long long)o > (long long)M ? KVSCHED_DEV_BAD_LENGTH : 0) |
           (bound > 0 && o > bound ? KVSCHED_DEV_O_MAX : 0);
}

// Position k of candidate order -> request id.
template <bool MOVES>
struct OrderReader {
    const int32_t *row;  // explicit row, or the base order
    int mt, mi, mj;      // the move (MOVES only)

    __device__ __forceinline__ int at(int k) const
    {
        if (!MOVES) return row[k];
        int pos = k;
        if (mt == KVSCHED_MOVE_SWAP) {
            pos = (k == mi) ? mj : ((k == mj) ? mi : k);
        } else if (mi < mj) {  // entry i moves back to j; (i, j] shift forward by one
            if (k >= mi && k <= mj) pos = (k == mj) ? mi : k + 1;
        } else {  // entry i moves up to j; [j, i) shift back by one
            if (k >= mj && k <= mi) pos = (k == mj) ? mi : k - 1;
        }
        return row[pos];
    }
};

}  // namespace
