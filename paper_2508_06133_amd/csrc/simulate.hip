// Timeline kernels: Phase 2 of Algorithm 1 ("Scheduling Execution") for many candidate
// orders at once, one 64-lane wavefront per candidate, plus the small kernels around it
// (length scan, order / move validation, argmin over candidates).
//
// Per-timeline state is the future-memory profile P(tau) = memory held at round tau by the
// requests admitted so far (the quantity M(X, t*) of Section 4), kept for the next H rounds
// in a ring of H int32 slots in LDS (H = power of two >= the longest decode length).
//
// Because admission is strictly in order and stops at the first request that does not fit
// (Algorithm 1's `break`), the start round of the k-th request of an order is the smallest
// t >= (start of the (k-1)-th) at which it fits beside everything admitted before it.  For a
// request (s, o), round tau rules out exactly the starts t with tau - o <= t <= tau - 1 and
// t < P(tau) + s + tau - M (Eq. 1 rearranged), so the search scans the window (t, t + o],
// moves t to the largest bound any scanned round imposes, and only has to look at the
// rounds that entered the window since.  Each round is therefore inspected once per request
// (o + waited rounds), then the admitted request's own ramp s+1..s+o is added to the ring.
#include "kvsched_internal.h"
#include "device_util.h"
#include "sort_util.h"

#include <limits.h>

namespace {

template <int H, int WPB, bool MOVES>
__global__ __launch_bounds__(WAVE *WPB) void timeline_kernel(SimParams p)
{
    __shared__ int ring_all[H * WPB];
    const int lane = threadIdx.x & (WAVE - 1);
    const int cand = __builtin_amdgcn_readfirstlane(blockIdx.x * WPB + (threadIdx.x >> 6));
    if (cand >= p.C) return;
    int *ring = ring_all + (threadIdx.x >> 6) * H;
    for (int i = lane; i < H; i += WAVE) ring[i] = 0;

    const int n = p.n;
    const int M = p.M;
    OrderReader<MOVES> rd;
    if (MOVES) {
        rd.row = p.src.base;
        rd.mt = KVSCHED_MOVE_SWAP;
        rd.mi = rd.mj = 0;
        if (cand < p.C - 1) {  // the last timeline is the base order itself
            rd.mt = p.src.moves[3 * (size_t)cand];
            rd.mi = min(max(p.src.moves[3 * (size_t)cand + 1], 0), n - 1);
            rd.mj = min(max(p.src.moves[3 * (size_t)cand + 2], 0), n - 1);
        }
    } else {
        rd.row = p.src.orders + (size_t)cand * (size_t)n;
        rd.mt = rd.mi = rd.mj = 0;
    }
    int32_t *crow = p.completion_out ? p.completion_out + (size_t)cand * (size_t)n : nullptr;

    long long tel = 0;
    int t = 0;  // start round of the previous request in the order
    __builtin_amdgcn_wave_barrier();

    for (int k0 = 0; k0 < n; k0 += WAVE) {
        // 64 positions of the order at a time: ids read coalesced, lengths gathered
        const int k = k0 + lane;
        int r = 0, sv = 1, ov = 1;
        if (k < n) {
            r = min(max(rd.at(k), 0), n - 1);
            sv = p.s[r];
            ov = p.o[r];
        }
        const bool bad = (sv < 1) | (ov < 1) | (ov > p.o_bound) | ((long long)sv + (long long)ov > (long long)M);
        if (__builtin_amdgcn_ballot_w64(bad) != 0) {  // cannot be scheduled: report, do not loop forever
            if (lane == 0) p.tel_out[cand] = -1;
            return;
        }
        const int cnt = min(WAVE, n - k0);
        int cv = 0;  // completion round of position k0 + lane
        for (int j = 0; j < cnt; ++j) {
            const int sj = __builtin_amdgcn_readlane(sv, j);
            const int oj = __builtin_amdgcn_readlane(ov, j);
            const int bias = sj - M;
            int lo = t + 1;
            for (;;) {
                const int hi = t + oj;
                int acc = INT_MIN;
                for (int tau0 = lo; tau0 <= hi; tau0 += WAVE) {
                    const int tau = tau0 + lane;
                    if (tau <= hi) {
                        const int need = ring[tau & (H - 1)] + bias + tau;  // least start round tau allows
                        acc = max(acc, min(tau, need));                      // tau constrains only t < tau
                    }
                }
                const int tn = wave_max_i32(acc);
                if (tn <= t) break;
                // rounds (t, tn] are behind every later start: their slots become rounds + H
                for (int tau0 = t + 1; tau0 <= tn; tau0 += WAVE) {
                    const int tau = tau0 + lane;
                    if (tau <= tn) ring[tau & (H - 1)] = 0;
                }
                __builtin_amdgcn_wave_barrier();
                lo = hi + 1;
                t = tn;
            }
            // admitted at round t: holds sj + a tokens at round t + a
            for (int tau0 = t + 1; tau0 <= t + oj; tau0 += WAVE) {
                const int tau = tau0 + lane;
                if (tau <= t + oj) ring[tau & (H - 1)] += sj + (tau - t);
            }
            __builtin_amdgcn_wave_barrier();
            const int c = t + oj;
            tel += c;
            cv = (lane == j) ? c : cv;
        }
        if (crow && k < n) crow[p.completion_by_position ? k : r] = cv;
    }
    if (lane == 0) p.tel_out[cand] = tel;
}

// Largest decode length and well-formedness of (s, o), and the lowest and highest position that any of K moves
// touches (malformed ones are clamped by the timeline kernel: they leave no shared prefix); resets the status word.
// Bound by latency: one workgroup up to 4096 lengths and moves, then one per 4096 (at most 64; 100000 lengths: 41 us
// by one workgroup, 5 us so), the last to finish writes the results.  A caller that waits for them (host, in pinned
// memory) finds them there: the wait is one store across the bus instead of a copy and a stream synchronisation.
constexpr int kScanFew = 1 << 30;  // among the flags (no status bit): the decode lengths are few
__global__ __launch_bounds__(1024) void scan_lengths_kernel(const int32_t *s, const int32_t *o, int32_t n, int32_t M,
                                                            int32_t o_bound, const int32_t *moves, int32_t K,
                                                            int32_t *words, int32_t *host, int32_t seq, int32_t *few_out)
{
    __shared__ int sh_max[16], sh_flag[16], sh_min[16], sh_top[16];
    const int first = blockIdx.x * 1024 + threadIdx.x, stride = gridDim.x * 1024;
    int mx = 0, flag = 0, lowest = INT_MAX, top = -1;
    for (int i = first; i < n; i += stride) {
        const int sv = s[i], ov = o[i];
        mx = max(mx, ov);
        if (sv < 1 || ov < 1 || (long long)sv + (long long)ov > (long long)M) flag |= KVSCHED_DEV_BAD_LENGTH;
        if (o_bound > 0 && ov > o_bound) flag |= KVSCHED_DEV_O_MAX;
    }
    for (int m = first; m < K; m += stride) {
        const int ty = moves[3 * (size_t)m], i = moves[3 * (size_t)m + 1], j = moves[3 * (size_t)m + 2];
        const bool ok = (ty == KVSCHED_MOVE_SWAP || ty == KVSCHED_MOVE_INSERT) && i >= 0 && j >= 0 && i < n && j < n;
        if (!ok) lowest = 0;
        else if (i != j) lowest = min(lowest, min(i, j));
        top = max(top, min(max(max(i, j), 0), n - 1));  // (as the timeline kernel clamps)
    }
    bool few = false;
    if (few_out && first < WAVE) {
        few = few_lengths(o[sampled(first, n)]);
        if (first == 0) to_host(few_out, few ? 1 : 0);
    }
    mx = wave_max_i32(mx);
    flag = wave_max_i32(flag & 1) | wave_max_i32(flag & KVSCHED_DEV_O_MAX) | (few ? kScanFew : 0);
    lowest = ~wave_max_i32(~lowest);
    top = wave_max_i32(top);
    if ((threadIdx.x & 63) == 0) {
        sh_max[threadIdx.x >> 6] = mx;
        sh_flag[threadIdx.x >> 6] = flag;
        sh_min[threadIdx.x >> 6] = lowest;
        sh_top[threadIdx.x >> 6] = top;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < 16; ++w) {
        mx = max(mx, sh_max[w]);
        flag |= sh_flag[w];
        lowest = min(lowest, sh_min[w]);
        top = max(top, sh_top[w]);
    }
    if (gridDim.x > 1) {
        atomicMax(&words[KVS_W_SCAN_OMAX], mx);
        atomicOr(&words[KVS_W_SCAN_FLAGS], flag);
        atomicMin(&words[KVS_W_SCAN_MINPOS], lowest);
        atomicMax(&words[KVS_W_SCAN_MAXPOS], top);
        device_writes_done();
        if (atomicAdd(&words[KVS_W_SCAN_DONE], 1) != (int)gridDim.x - 1) return;
        mx = atomicExch(&words[KVS_W_SCAN_OMAX], 0);
        flag = atomicExch(&words[KVS_W_SCAN_FLAGS], 0);
        lowest = atomicExch(&words[KVS_W_SCAN_MINPOS], INT_MAX);
        top = atomicExch(&words[KVS_W_SCAN_MAXPOS], -1);
        atomicExch(&words[KVS_W_SCAN_DONE], 0);
    }
    words[KVS_W_STATUS] = flag & ~kScanFew;
    words[KVS_W_STATUS_AT] = KVS_W_STATUS;
    words[KVS_W_OMAX] = mx;
    words[KVS_W_MINPOS] = lowest;
    words[KVS_W_MAXPOS] = top;
    words[KVS_W_ESTMAX] = 0;
    if (host) {
        if (moves) {
            to_host(&host[KVS_H_MINPOS], lowest);
            to_host(&host[KVS_H_MAXPOS], top);
            device_writes_done();
        }
        longest_to_host(host, mx, seq, (flag & kScanFew) != 0);
    }
}

// One wavefront per row: is it a permutation of 0..n-1?  Bitmap of n bits per wave in LDS.
template <int WPB>
__global__ __launch_bounds__(WAVE *WPB) void check_orders_kernel(const int32_t *orders, int32_t C, int32_t n,
                                                                 int64_t *tel_out, int32_t *words, int32_t o_limit, const int32_t *todo)
{
    extern __shared__ unsigned int bitmap_all[];
    const int o_max = words[KVS_W_OMAX];
    const int lane = threadIdx.x & (WAVE - 1);
    const int cand = blockIdx.x * WPB + (threadIdx.x >> 6);
    if (cand >= C || (todo && todo[cand] == 0)) return;
    const int nw = (n + 31) >> 5;
    unsigned int *bm = bitmap_all + (size_t)(threadIdx.x >> 6) * nw;
    for (int i = lane; i < nw; i += WAVE) bm[i] = 0;
    __builtin_amdgcn_wave_barrier();
    const int32_t *row = orders + (size_t)cand * (size_t)n;
    bool bad = false;
    for (int k = lane; k < n; k += WAVE) {
        const int r = row[k];
        if (r < 0 || r >= n) {
            bad = true;
        } else {
            const unsigned int bit = 1u << (r & 31);
            if (atomicOr(&bm[r >> 5], bit) & bit) bad = true;
        }
    }
    if (__builtin_amdgcn_ballot_w64(bad) != 0 && lane == 0 && o_max <= o_limit) {  // (else the rows have not been placed)
        tel_out[cand] = -1;
        atomicOr(&words[KVS_W_STATUS], KVSCHED_DEV_BAD_ORDER);
    }
}

// The same for long rows: a workgroup per row (a single wavefront would walk a row of 100000 entries in 1563
// dependent turns), of 1024 threads up to 512 rows, which then run at a time, and of 256 beyond, of which a compute unit takes eight.
// n entries in range set n bits exactly if none is there twice, so nothing is read back before the end, and eight
// reads of a thread are in flight.  1025 rows of 100000: 184 us by 1024 threads a row, which take three turns, 139 so; one of 10000 4.7.
template <int TPB>
__global__ __launch_bounds__(TPB) void check_orders_wide_kernel(const int32_t *orders, int32_t C, int32_t n,
                                                                int64_t *tel_out, int32_t *words, int32_t o_limit, const int32_t *todo)
{
    extern __shared__ unsigned int bitmap_all[];
    constexpr int E = 8;
    if (todo && todo[blockIdx.x] == 0) return;
    const int o_max = words[KVS_W_OMAX];
    const int cand = blockIdx.x;
    const int nw = (n + 31) >> 5;
    for (int i = threadIdx.x; i < nw; i += TPB) bitmap_all[i] = 0;
    __syncthreads();
    const int32_t *row = orders + (size_t)cand * (size_t)n;
    int bad = 0;
    for (int k = threadIdx.x; k < n; k += TPB * E) {
        int r[E];
#pragma unroll
        for (int e = 0; e < E; ++e) r[e] = row[min(k + TPB * e, n - 1)];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (k + TPB * e >= n) continue;
            if ((unsigned)r[e] >= (unsigned)n) bad = 1;
            else atomicOr(&bitmap_all[r[e] >> 5], 1u << (r[e] & 31));
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nw; i += TPB)
        if (bitmap_all[i] != (32 * i + 32 <= n ? ~0u : (1u << (n & 31)) - 1u)) bad = 1;
    if (__syncthreads_or(bad) && threadIdx.x == 0 && o_max <= o_limit) {  // (else the rows have not been placed)
        tel_out[cand] = -1;
        atomicOr(&words[KVS_W_STATUS], KVSCHED_DEV_BAD_ORDER);
    }
}

// Index of the least non-negative tel[0..K), lowest index among equals.  (Least latency, then lowest index) is a total order: any
// reduction tree gives the same winner.  One workgroup up to 4096 entries, then one per 2048 (at most
// KVS_ARGMIN_GROUPS), the last to finish reduces the others' winners: 40321 entries 16 us by one, 4 us so.
// Bound by latency: the lanes' least latency first and then the lowest index among its holders, by moves within the vector unit, and
// the last workgroup's 64 partial winners by one wavefront (pairs exchanged through LDS, and a second round over a workgroup: 40321 entries
// 5.9 us a call, 4.2 now, 8191 5.5 and 3.9, 4096 4.4 and 3.9).
// MOVES: the end of a local-search step in the same pass (see kvs_launch_neighbor_finish).
template <bool MOVES>
__global__ __launch_bounds__(1024) void argmin_kernel(const int64_t *tel, int32_t K, int64_t *result_out,
                                                      const int32_t *rejoin, const int32_t *moves, int32_t n,
                                                      int64_t *tel_out, int32_t *words)
{
    __shared__ u64 sh_tel[16];
    __shared__ unsigned sh_idx[16];
    __shared__ int sh_last;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    u64 bt = ~0ull;     // as numbers without a sign none, -1, is the largest
    unsigned bi = ~0u;
    auto among_lanes = [&]() {  // into all lanes of a wavefront: the least latency, and of those with it the lowest index
        const u64 least = wave_min_u64(bt);
        bi = wave_min_u32(bt == least ? bi : ~0u);
        bt = least;
    };
    auto reduce = [&]() {  // over the workgroup, into the first wavefront
        among_lanes();
        if (lane == 0) {
            sh_tel[wave] = bt;
            sh_idx[wave] = bi;
        }
        __syncthreads();
        if (wave == 0) {
            bt = lane < 16 ? sh_tel[lane] : ~0ull;
            bi = lane < 16 ? sh_idx[lane] : ~0u;
            among_lanes();
        }
    };
    for (int m = blockIdx.x * 1024 + threadIdx.x; m < K; m += gridDim.x * 1024) {
        long long v = tel[m];
        if constexpr (MOVES) {
            if (rejoin && rejoin[m] != INT_MAX) {  // its sum of completion rounds is relative to the base order's
                const long long t0 = tel[K];
                v = t0 < 0 ? -1 : v + t0;
            }
            const int ty = moves[3 * (size_t)m], i = moves[3 * (size_t)m + 1], j = moves[3 * (size_t)m + 2];
            if ((ty != KVSCHED_MOVE_SWAP && ty != KVSCHED_MOVE_INSERT) || i < 0 || j < 0 || i >= n || j >= n) {
                v = -1;
                atomicOr(&words[KVS_W_STATUS], KVSCHED_DEV_BAD_MOVE);
            }
            if (tel_out) tel_out[m] = v;
        }
        if (v >= 0 && (u64)v < bt) {  // (indices ascend)
            bt = (u64)v;
            bi = (unsigned)m;
        }
    }
    reduce();
    if (gridDim.x > 1) {
        long long *part = (long long *)(words + KVS_W_ARGMIN_PART);
        if (threadIdx.x == 0) {
            __hip_atomic_store(&part[2 * blockIdx.x], (long long)bt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&part[2 * blockIdx.x + 1], (long long)bi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            device_writes_done();
            sh_last = atomicAdd(&words[KVS_W_ARGMIN_DONE], 1) == (int)gridDim.x - 1;
        }
        __syncthreads();
        if (!sh_last) return;
        static_assert(KVS_ARGMIN_GROUPS <= 64, "a lane each");
        if (wave == 0) {
            bt = ~0ull;
            bi = ~0u;
            if (lane < (int)gridDim.x) {
                bt = (u64)__hip_atomic_load(&part[2 * lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                bi = (unsigned)__hip_atomic_load(&part[2 * lane + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            among_lanes();
        }
        if (threadIdx.x == 0) words[KVS_W_ARGMIN_DONE] = 0;
    }
    if (threadIdx.x == 0) {
        const bool base_ok = !MOVES || tel[K] >= 0;  // a faulty base order makes every neighbour faulty
        result_out[0] = base_ok ? (int)bi : -1;
        result_out[1] = base_ok ? (int64_t)bt : -1;
        if (MOVES) result_out[2] = tel[K];
    }
}

template <int H, int WPB>
int launch_timeline(const SimParams &p, hipStream_t st)
{
    const unsigned blocks = (unsigned)((p.C + WPB - 1) / WPB);
    if (p.src.orders)
        hipLaunchKernelGGL((timeline_kernel<H, WPB, false>), dim3(blocks), dim3(WAVE * WPB), 0, st, p);
    else
        hipLaunchKernelGGL((timeline_kernel<H, WPB, true>), dim3(blocks), dim3(WAVE * WPB), 0, st, p);
    return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}

}  // namespace

int kvs_launch_scan_lengths(const int32_t *s, const int32_t *o, int32_t n, int32_t M, int32_t o_bound,
                            int32_t *d_words, hipStream_t st, const int32_t *moves, int32_t K, int32_t *host,
                            int32_t seq, int32_t *few_out)
{
    const int32_t most = moves && K > n ? K : n;
    const unsigned blocks = most <= 4096 ? 1u : most < 64 * 4096 ? (unsigned)((most + 4095) / 4096) : 64u;
    hipLaunchKernelGGL(scan_lengths_kernel, dim3(blocks), dim3(1024), 0, st, s, o, n, M, o_bound, moves, moves ? K : 0,
                       d_words, host, seq, few_out);
    return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}

int kvs_launch_simulate(const SimParams &p, int32_t ring_slots, hipStream_t st)
{
    switch (ring_slots) {
        case 64: return launch_timeline<64, 4>(p, st);
        case 128: return launch_timeline<128, 4>(p, st);
        case 256: return launch_timeline<256, 4>(p, st);
        case 512: return launch_timeline<512, 4>(p, st);
        case 1024: return launch_timeline<1024, 4>(p, st);
        case 2048: return launch_timeline<2048, 4>(p, st);
        case 4096: return launch_timeline<4096, 4>(p, st);
        case 8192: return launch_timeline<8192, 2>(p, st);
        case 16384: return launch_timeline<16384, 1>(p, st);
        default: return KVSCHED_ERANGE;
    }
}

int kvs_launch_check_orders(const int32_t *orders, int32_t C, int32_t n, int64_t *tel_out, int32_t *d_words,
                            hipStream_t st, int32_t o_limit, const int32_t *todo)
{
    const size_t per_wave = (size_t)((n + 31) >> 5) * sizeof(unsigned int);
    if (per_wave > 65536) return KVSCHED_ERANGE;
    // long rows, not enough of them to fill the chip with a wavefront each (one row of 10000: 31 us by a wavefront)
    if ((n >= 16384 && C <= 8192) || (n >= 1024 && C <= 512)) {
        if (C <= 512)
            hipLaunchKernelGGL(check_orders_wide_kernel<1024>, dim3((unsigned)C), dim3(1024), per_wave, st, orders, C, n,
                               tel_out, d_words, o_limit, todo);
        else
            hipLaunchKernelGGL(check_orders_wide_kernel<256>, dim3((unsigned)C), dim3(256), per_wave, st, orders, C, n,
                               tel_out, d_words, o_limit, todo);
    } else if (per_wave * 4 <= 65536) {
        hipLaunchKernelGGL((check_orders_kernel<4>), dim3((unsigned)((C + 3) / 4)), dim3(256), per_wave * 4, st,
                           orders, C, n, tel_out, d_words, o_limit, todo);
    } else {
        hipLaunchKernelGGL((check_orders_kernel<1>), dim3((unsigned)C), dim3(64), per_wave, st, orders, C, n,
                           tel_out, d_words, o_limit, todo);
    }
    return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}

static unsigned argmin_groups(int32_t K)
{
    return K <= 4096 ? 1u : K < KVS_ARGMIN_GROUPS * 2048 ? (unsigned)((K + 2047) / 2048) : (unsigned)KVS_ARGMIN_GROUPS;
}

int kvs_launch_argmin(const int64_t *tel, int32_t K, int64_t *result_out, int32_t *d_words, hipStream_t st)
{
    hipLaunchKernelGGL((argmin_kernel<false>), dim3(argmin_groups(K)), dim3(1024), 0, st, tel, K, result_out,
                       (const int32_t *)nullptr, (const int32_t *)nullptr, 0, (int64_t *)nullptr, d_words);
    return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}

int kvs_launch_neighbor_finish(const int64_t *tel, const int32_t *rejoin, const int32_t *moves, int32_t K, int32_t n,
                               int64_t *tel_out, int64_t *result_out, int32_t *d_words, hipStream_t st)
{
    hipLaunchKernelGGL((argmin_kernel<true>), dim3(argmin_groups(K)), dim3(1024), 0, st, tel, K, result_out, rejoin, moves,
                       n, tel_out, d_words);
    return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}
