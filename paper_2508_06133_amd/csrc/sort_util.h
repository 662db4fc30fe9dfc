// Sorting and scanning building blocks of the Phase 1 kernels: wave-level scans by DPP lane moves and a
// workgroup-wide bitonic sort of 64-bit keys held in registers.
#pragma once

#include "kvsched_internal.h"

namespace {

typedef unsigned long long u64;

template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned dpp_or_zero(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}

// Inclusive sum over the lanes up to this one (all 64 lanes active).
__device__ __forceinline__ unsigned wave_scan_u32(unsigned v)
{
    v += dpp_or_zero<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8: sums inside the rows of 16
    v += dpp_or_zero<0x112, 0xf>(v);
    v += dpp_or_zero<0x114, 0xf>(v);
    v += dpp_or_zero<0x118, 0xf>(v);
    v += dpp_or_zero<0x142, 0xa>(v);  // row_bcast 15 into rows 1, 3; row_bcast 31 into rows 2, 3
    v += dpp_or_zero<0x143, 0xc>(v);
    return v;
}

template <int CTRL, int ROWS>
__device__ __forceinline__ u64 dpp_or_zero64(u64 v)
{
    return (u64)dpp_or_zero<CTRL, ROWS>((unsigned)v) | ((u64)dpp_or_zero<CTRL, ROWS>((unsigned)(v >> 32)) << 32);
}

__device__ __forceinline__ u64 wave_scan_u64(u64 v)
{
    v += dpp_or_zero64<0x111, 0xf>(v);
    v += dpp_or_zero64<0x112, 0xf>(v);
    v += dpp_or_zero64<0x114, 0xf>(v);
    v += dpp_or_zero64<0x118, 0xf>(v);
    v += dpp_or_zero64<0x142, 0xa>(v);
    v += dpp_or_zero64<0x143, 0xc>(v);
    return v;
}

__device__ __forceinline__ u64 lane_value_u64(u64 v, int lane)
{
    return (u64)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, lane) |
           ((u64)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), lane) << 32);
}

// Least value over the 64 lanes, in every lane (all lanes active).
__device__ __forceinline__ unsigned wave_min_u32(unsigned v)
{
    v = min(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xf, 0xf, false));   // lanes 1 apart
    v = min(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xf, 0xf, false));   // 2 apart
    v = min(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xf, 0xf, false));  // mirror in halves of a row
    v = min(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xf, 0xf, false));  // mirror in rows
    const unsigned a = (unsigned)__builtin_amdgcn_readlane((int)v, 0), b = (unsigned)__builtin_amdgcn_readlane((int)v, 16);
    const unsigned c = (unsigned)__builtin_amdgcn_readlane((int)v, 32), d = (unsigned)__builtin_amdgcn_readlane((int)v, 48);
    return min(min(a, b), min(c, d));
}

// The value of the lane whose number differs in bit X (X = 1, 2, 4, ..., 32).
template <int X>
__device__ __forceinline__ unsigned lane_xor(unsigned v)
{
    if constexpr (X == 1) return (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xf, 0xf, false);
    else if constexpr (X == 2) return (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xf, 0xf, false);
    else if constexpr (X == 8) return (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x128, 0xf, 0xf, false);  // rotate a row by 8
    else if constexpr (X == 4 || X == 16) return (unsigned)__builtin_amdgcn_ds_swizzle((int)v, (X << 10) | 0x1f);
    else return (unsigned)__shfl_xor((int)v, X);
}

template <int X>
__device__ __forceinline__ u64 lane_xor64(u64 v)
{
    return (u64)lane_xor<X>((unsigned)v) | ((u64)lane_xor<X>((unsigned)(v >> 32)) << 32);
}

// Steps of the bitonic network over N = TPB * E keys: element i = 64 E wave + 64 e + lane is kept in k[e]
// of its thread.  Partners a stride apart: in the same wavefront by lane moves, in the same thread, or (the
// larger strides) through LDS; two buffers alternate so that one barrier serves an exchange.
__device__ __forceinline__ u64 keep_one(u64 mine, u64 other, bool least) { return (other < mine) == least ? other : mine; }

// Strides below 64 (only those below `size`).
template <int E, int STRIDE>
__device__ __forceinline__ void bitonic_lanes(u64 (&k)[E], int i0, int size)
{
    if (STRIDE < size) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = i0 + 64 * e;
            k[e] = keep_one(k[e], lane_xor64<STRIDE>(k[e]), ((i & size) == 0) == ((i & STRIDE) == 0));
        }
    }
    if constexpr (STRIDE > 1) bitonic_lanes<E, STRIDE / 2>(k, i0, size);
}

// Strides 64 STEP inside a thread.
template <int E, int STEP>
__device__ __forceinline__ void bitonic_thread(u64 (&k)[E], int i0, int size)
{
    if constexpr (STEP >= 1) {
        if (64 * STEP < size) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if ((e & STEP) == 0) {
                    const bool asc = ((i0 + 64 * e) & size) == 0;
                    const u64 x = k[e], y = k[e | STEP];
                    const bool sw = (x > y) == asc;
                    k[e] = sw ? y : x;
                    k[e | STEP] = sw ? x : y;
                }
            }
        }
        bitonic_thread<E, STEP / 2>(k, i0, size);
    }
}

// Ascending sort of TPB * E keys.  lds: 2 TPB E keys; the caller separates its own use of it by barriers.  From 1024 threads on the
// stages are a loop over one piece of code of some 1.5 KB: unrolled, a sort of 2048 keys is 11 KB of instructions that run once and
// have to be fetched (Sorted-F order of 2000 requests 53 -> 47 us).  Few keys are quicker unrolled (61 requests 6.0 us, 6.9 as a loop).
template <int TPB, int E>
__device__ __forceinline__ void block_sort(u64 (&k)[E], u64 *lds)
{
    constexpr int N = TPB * E;
    const int i0 = 64 * E * (threadIdx.x >> 6) + (threadIdx.x & 63);
    u64 *b = lds, *other = lds + N;
    constexpr int kStages = TPB < 1024 ? 16 : 1;  // (to unroll)
#pragma unroll kStages
    for (int size = 2; size <= N; size <<= 1) {
        if constexpr (TPB > 64) {
#pragma unroll kStages
            for (int stride = size >> 1; stride >= 64 * E; stride >>= 1) {
#pragma unroll
                for (int e = 0; e < E; ++e) b[i0 + 64 * e] = k[e];
                __syncthreads();
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int i = i0 + 64 * e;
                    k[e] = keep_one(k[e], b[i ^ stride], ((i & size) == 0) == ((i & stride) == 0));
                }
                u64 *const t = b;
                b = other;
                other = t;
            }
        }
        bitonic_thread<E, E / 2>(k, i0, size);
        bitonic_lanes<E, 32>(k, i0, size);
    }
}

}  // namespace
