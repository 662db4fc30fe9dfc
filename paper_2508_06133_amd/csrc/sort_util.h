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
// have to be fetched (two such sorts 53 -> 47 us).  Few keys are quicker unrolled (61 requests 6.0 us, 6.9 as a loop).
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

// The same network for 32-bit keys of one wavefront, element i = 64 e + lane in k[e]: three instructions an exchange (least,
// greatest, choice by a mask that is a constant), partners 16 and 32 lanes apart by swaps of rows.
template <int STRIDE>
__device__ __forceinline__ unsigned exchanged(unsigned v, u64 least_in)
{
    unsigned a = v, b;
    if constexpr (STRIDE == 16) {
        const auto x = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        a = x[0], b = x[1];
    } else if constexpr (STRIDE == 32) {
        const auto x = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        a = x[0], b = x[1];
    } else if constexpr (STRIDE == 4) {  // mirrored in eights, then in fours
        b = (unsigned)__builtin_amdgcn_update_dpp(0, __builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true), 0x1B, 0xf, 0xf, true);
    } else {
        b = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, STRIDE == 1 ? 0xB1 : STRIDE == 2 ? 0x4E : 0x128, 0xf, 0xf, true);
    }
    unsigned r;
    asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(r) : "v"(max(a, b)), "v"(min(a, b)), "s"(least_in));
    return r;
}

// Lanes that keep the lesser of two elements STRIDE apart in the stage of `size`, row e.
__device__ constexpr u64 least_lanes(int size, int stride, int e)
{
    u64 m = 0;
    for (int lane = 0; lane < 64; ++lane)
        if ((((64 * e + lane) & size) == 0) == ((lane & stride) == 0)) m |= 1ull << lane;
    return m;
}

template <int E, int SIZE, int STRIDE>
__device__ __forceinline__ void wave_sort_stage(unsigned (&k)[4])
{
    if constexpr (STRIDE >= 64) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if ((e & (STRIDE / 64)) == 0) {
                const unsigned lo = min(k[e], k[e + STRIDE / 64]), hi = max(k[e], k[e + STRIDE / 64]);
                const bool asc = ((64 * e) & SIZE) == 0;
                k[e] = asc ? lo : hi;
                k[e + STRIDE / 64] = asc ? hi : lo;
            }
        }
    } else {
        constexpr u64 even = least_lanes(SIZE, STRIDE, 0), odd = least_lanes(SIZE, STRIDE, 1), two = least_lanes(SIZE, STRIDE, 2),
                      three = least_lanes(SIZE, STRIDE, 3);
#pragma unroll
        for (int e = 0; e < E; ++e) k[e] = exchanged<STRIDE>(k[e], e == 0 ? even : e == 1 ? odd : e == 2 ? two : three);
    }
    if constexpr (STRIDE > 1) wave_sort_stage<E, SIZE, STRIDE / 2>(k);
    else if constexpr (SIZE < 64 * E) wave_sort_stage<E, SIZE * 2, SIZE>(k);
}

// Ascending sort of the first 64 E of 256 keys of a wavefront (those behind stay).
template <int E>
__device__ __forceinline__ void wave_sort(unsigned (&k)[4]) { wave_sort_stage<E, 2, 1>(k); }

__device__ __forceinline__ u64 wave_min_u64(u64 v)
{
    v = min(v, lane_xor64<1>(v));
    v = min(v, lane_xor64<2>(v));
    v = min(v, (u64)(unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)v, (int)(unsigned)v, 0x141, 0xf, 0xf, false) |
                   ((u64)(unsigned)__builtin_amdgcn_update_dpp((int)(v >> 32), (int)(v >> 32), 0x141, 0xf, 0xf, false) << 32));
    v = min(v, lane_xor64<8>(v));
    return min(min(lane_value_u64(v, 0), lane_value_u64(v, 16)), min(lane_value_u64(v, 32), lane_value_u64(v, 48)));
}

}  // namespace
