// Kernels of the receding-horizon step (an offline adaptation of the paper's Sorted-F-Online,
// Section 6 "Heuristics under Online Arrival": plan on a look-ahead window of the pending
// order, commit what the timeline admits, plan again).  All requests are present at round 0;
// the committed part of the order is the prefix of positions already admitted.
#include "kvsched_internal.h"
#include "device_util.h"
#include "sort_util.h"

#include <limits.h>

namespace {

// position k of the order with move (ty, i, j) applied = position moved_from(...) of the order before
__device__ __forceinline__ int moved_from(int k, int ty, int i, int j)
{
    if (ty == KVSCHED_MOVE_SWAP) return k == i ? j : (k == j ? i : k);
    if (i < j) {
        if (k >= i && k <= j) return k == j ? i : k + 1;
    } else {
        if (k >= j && k <= i) return k == j ? i : k - 1;
    }
    return k;
}

// order_out = order with move moves[result[0]] applied (result[0] < 0: unchanged).
__global__ __launch_bounds__(256) void apply_best_move_kernel(const int32_t *order, int32_t n, const int32_t *moves,
                                                              const int64_t *result, int32_t *order_out)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const long long best = result[0];
    int pos = k;
    if (best >= 0)
        pos = moved_from(k, moves[3 * best], min(max(moves[3 * best + 1], 0), n - 1), min(max(moves[3 * best + 2], 0), n - 1));
    order_out[k] = order[pos];
}

// The values of a workgroup of 1024 that order statistics are taken of: HELD of them per thread stay in registers
// (16384 in all), any beyond are fetched again at every turn.  A turn counts the values in 1024 parts of the range that is left, in LDS,
// and takes the part that holds the one looked for: two turns up to 2^20.  (By halving the range, some fifteen turns of comparisons, a sum over the
// lanes, a word of LDS and a barrier: horizon_choose_kernel and horizon_advance_kernel 9.2 and 11.5 us at 10000 requests, 8.4 and 9.9 now.)
constexpr int HELD = 16, PARTS = 1024;
struct StatLds {
    int part[PARTS], wave[16], most, chosen, before, upto;
};
template <class F>
struct Values {
    F at;
    int count;
    int held[HELD];
    StatLds &L;

    __device__ __forceinline__ Values(F f, int n, StatLds &lds) : at(f), count(n), L(lds)
    {
#pragma unroll
        for (int e = 0; e < HELD; ++e) {
            const int k = threadIdx.x + 1024 * e;
            held[e] = k < count ? at(k) : INT_MAX;
        }
    }

    // the k-th smallest, 1 <= k <= count, and how many are no larger; values lie in [0, 2^30) (of others fewer than k may be counted: then
    // the answer is of no use, but the same in every call)
    __device__ __forceinline__ int kth(int k, int &upto)
    {
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
        int mx = 0;
#pragma unroll
        for (int e = 0; e < HELD; ++e)
            if (held[e] != INT_MAX) mx = max(mx, held[e]);
        for (int q = tid + 1024 * HELD; q < count; q += 1024) mx = max(mx, at(q));
        mx = wave_max_i32(mx);
        if (tid == 0) L.most = L.chosen = L.before = L.upto = 0;
        L.part[tid] = 0;
        __syncthreads();
        if (lane == 0) atomicMax(&L.most, mx);
        __syncthreads();
        int base = 0, before = 0;  // the values below base
        for (int shift = max(22 - __builtin_clz(L.most | 1), 0);; shift = max(shift - 10, 0)) {
            auto enter = [&](int v) {
                const unsigned part = (unsigned)(v - base) >> shift;
                if (part < PARTS) atomicAdd(&L.part[part], 1);
            };
#pragma unroll
            for (int g = 0; g < HELD; g += 4) {
                if (1024 * g >= count) continue;  // (uniform)
#pragma unroll
                for (int e = g; e < g + 4; ++e) enter(held[e]);
            }
            for (int q = tid + 1024 * HELD; q < count; q += 1024) enter(at(q));
            __syncthreads();
            const int mine = L.part[tid];
            int incl = (int)wave_scan_u32((unsigned)mine);
            if (lane == 63) L.wave[wave] = incl;
            L.part[tid] = 0;
            __syncthreads();
            incl += before;
            for (int w = 0; w < 15; ++w) incl += w < wave ? L.wave[w] : 0;
            if (incl >= k && incl - mine < k) {
                L.chosen = tid;
                L.before = incl - mine;
                L.upto = incl;
            }
            __syncthreads();
            base += L.chosen << shift;
            before = L.before;
            if (shift == 0) break;
        }
        upto = L.upto;
        return base;
    }
};

// Is what the context keeps still true?  Several workgroups, the last to finish draws the conclusion.
__global__ __launch_bounds__(256) void horizon_begin_kernel(HorizonKept h, int32_t kept, const int32_t *order,
                                                            const int32_t *s, const int32_t *o, int32_t n,
                                                            const int32_t *moves, int32_t K, int32_t *blocks)
{
    const int first = blockIdx.x * 256 + threadIdx.x, stride = gridDim.x * 256;
    const int avail = kept ? h.ctrl[KVS_HZ_AVAIL] : 0;
    int bad = !kept;
    for (int i = first; i < n; i += stride) {
        const int sv = s[i], ov = o[i], id = order[i];
        if (kept) bad |= (sv != h.s[i]) | (ov != h.o[i]) | (i < 64 * avail && id != h.order[i]);
        h.s[i] = sv;
        h.o[i] = ov;
        h.order[i] = id;
    }
    const int cap = (n - 1) >> 6;
    for (int m = first; m <= K; m += stride) {  // (as move_blocks_kernel)
        int nb = 0;
        if (m < K) {
            const int ty = moves[3 * (size_t)m], i = moves[3 * (size_t)m + 1], j = moves[3 * (size_t)m + 2];
            const bool ok = (ty == KVSCHED_MOVE_SWAP || ty == KVSCHED_MOVE_INSERT) && i >= 0 && j >= 0 && i < n && j < n;
            if (ok) nb = i == j ? cap : min(min(i, j) >> 6, cap);
        }
        blocks[m] = nb;
    }
    const bool any = __syncthreads_or(bad) != 0;
    __shared__ int last;
    if (threadIdx.x == 0) {
        if (any) atomicOr(&h.ctrl[KVS_HZ_BAD], 1);
        device_writes_done();
        last = atomicAdd(&h.ctrl[KVS_HZ_DONE], 1) == (int)gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    __shared__ int valid;
    if (threadIdx.x == 0) {
        valid = atomicExch(&h.ctrl[KVS_HZ_BAD], 0) ? 0 : avail;
        atomicExch(&h.ctrl[KVS_HZ_DONE], 0);
        h.ctrl[KVS_HZ_AVAIL] = valid;
        h.ctrl[KVS_HZ_ZERO] = 0;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < KVS_PROGRESS_COPIES; i += 256) h.progress[KVS_PROGRESS_STRIDE_WORDS * i] = valid;
}

// One workgroup.  The move is applied to the order (and its copy).  The new order's timeline is wanted up to the round
// by which k = completed_in + complete_every requests have completed.  The positions before the block of the first
// one any move touches are placed already: the k-th smallest completion among them bounds that round from above, and every position behind starts no
// earlier than the ones before it; so the timeline may stop once its round has passed that bound.
__global__ __launch_bounds__(1024) void horizon_choose_kernel(HorizonKept h, int32_t *order, int32_t n, const int32_t *moves,
                                                              const int64_t *result, const int32_t *words, int32_t stride,
                                                              long long completed_in, int32_t complete_every, int32_t full)
{
    __shared__ StatLds lds;
    const int first_block = min(max(words[KVS_W_MINPOS], 0) >> 6, (n - 1) >> 6);  // no move touches what lies before
    const long long best = result[0];
    if (best >= 0) {
        const int ty = moves[3 * best];
        const int i = min(max(moves[3 * best + 1], 0), n - 1), j = min(max(moves[3 * best + 2], 0), n - 1);
        const int lo = min(i, j), hi = max(i, j);
        for (int k = lo + threadIdx.x; k <= hi; k += 1024) order[k] = h.order[moved_from(k, ty, i, j)];
        __syncthreads();
        for (int k = lo + threadIdx.x; k <= hi; k += 1024) h.order[k] = order[k];
    }
    __syncthreads();
    const int placed = 64 * first_block;
    const long long k = min(completed_in + complete_every, (long long)n);
    int limit = INT_MAX;
    if (!full && k <= placed && best >= 0) {  // (uniform)
        auto completion = [&](int p) { return h.start[p] + h.o[min(max(h.order[p], 0), n - 1)]; };
        Values<decltype(completion)> c(completion, placed, lds);
        int upto;
        limit = c.kth((int)max(k, 1ll), upto);
    }
    if (threadIdx.x == 0) {
        h.ctrl[KVS_HZ_FIRST] = first_block;
        h.ctrl[KVS_HZ_LIMIT] = limit;
        h.ctrl[KVS_HZ_PLACED] = 0;
        // no valid candidate: the states may be missing; the timeline then ends where it would start
        if (best < 0 && first_block > 0) h.snapshots[(size_t)(first_block - 1) * (size_t)stride + 1] = -1;
    }
}

// One workgroup.  T = round by which min(n, completed_in + complete_every) requests have completed (the k-th smallest
// completion round); result = {positions admitted by T (they form a prefix of the order, start rounds being
// nondecreasing along it), requests completed by T, T}.
template <class START, class COMPLETION>
__device__ __forceinline__ void commit_point(int n, int placed, START start, COMPLETION completion, long long completed_in,
                                             int complete_every, int64_t *result_out, StatLds &lds, int *sum)
{
    const int k = (int)max(min(min(completed_in + complete_every, (long long)n), (long long)placed), 1ll);
    int T = 0, done = 0;
    if (placed > 0) {
        Values<COMPLETION> c(completion, placed, lds);
        T = c.kth(k, done);
    }
    int admitted = 0;
    for (int q = threadIdx.x; q < placed; q += 1024) admitted += start(q) <= T;
    admitted = (int)wave_scan_u32((unsigned)admitted);
    if ((threadIdx.x & 63) == 63) atomicAdd(sum, admitted);
    __syncthreads();
    if (threadIdx.x == 0) {
        result_out[0] = *sum;
        result_out[1] = done;
        result_out[2] = T;
    }
}

__global__ __launch_bounds__(1024) void horizon_advance_kernel(HorizonKept h, const int32_t *order, int32_t n, int32_t blocks,
                                                              long long completed_in, int32_t complete_every,
                                                              int32_t *completion_out, int64_t *result_out)
{
    __shared__ StatLds lds;
    __shared__ int sum;
    if (threadIdx.x == 0) sum = 0;
    __syncthreads();
    const int placed = min(h.ctrl[KVS_HZ_PLACED], n);
    auto start = [&](int p) { return h.start[p]; };
    auto completion = [&](int p) { return h.start[p] + h.o[min(max(order[p], 0), n - 1)]; };
    if (completion_out)
        for (int p = threadIdx.x; p < placed; p += 1024) completion_out[min(max(order[p], 0), n - 1)] = completion(p);
    commit_point(n, placed, start, completion, completed_in, complete_every, result_out, lds, &sum);
    if (threadIdx.x == 0) h.ctrl[KVS_HZ_AVAIL] = min(placed >> 6, blocks);
}

// result: all six of the step's numbers, of which the last three are written here.  An order or lengths that are faulty (result[2] < 0, the
// latency of the order before the move) have no timeline: the ids may be none, completion rounds may be missing, and nothing is committed.
__global__ __launch_bounds__(1024) void horizon_advance_by_id_kernel(const int32_t *order, const int32_t *by_id,
                                                                    const int32_t *o, int32_t n, long long completed_in,
                                                                    int32_t complete_every, int64_t *result)
{
    __shared__ StatLds lds;
    __shared__ int sum;
    if (result[2] < 0) {  // (uniform)
        if (threadIdx.x < 3) result[3 + threadIdx.x] = 0;
        return;
    }
    if (threadIdx.x == 0) sum = 0;
    __syncthreads();
    auto start = [&](int p) { return by_id[order[p]] - o[order[p]]; };
    auto completion = [&](int i) { return by_id[i]; };
    commit_point(n, n, start, completion, completed_in, complete_every, result + 3, lds, &sum);
}

__global__ __launch_bounds__(256) void horizon_completion_kernel(HorizonKept h, const int32_t *order, const int32_t *o,
                                                                 int32_t n, int32_t *completion_out)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= n || p >= h.ctrl[KVS_HZ_PLACED]) return;
    const int id = min(max(order[p], 0), n - 1);
    completion_out[id] = h.start[p] + o[id];
}

int ok() { return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP; }

}  // namespace

int kvs_launch_apply_best_move(const int32_t *order, int32_t n, const int32_t *moves, const int64_t *result,
                               int32_t *order_out, hipStream_t st)
{
    hipLaunchKernelGGL(apply_best_move_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, order, n, moves,
                       result, order_out);
    return ok();
}

int kvs_launch_horizon_begin(const HorizonKept &h, int32_t kept, const int32_t *order, const int32_t *s, const int32_t *o,
                             int32_t n, const int32_t *moves, int32_t K, int32_t *blocks, hipStream_t st)
{
    const int most = n > K + 1 ? n : K + 1;
    const unsigned groups = most >= 64 * 1024 ? 64u : (unsigned)((most + 1023) / 1024);
    hipLaunchKernelGGL(horizon_begin_kernel, dim3(groups), dim3(256), 0, st, h, kept, order, s, o, n, moves, K, blocks);
    return ok();
}

int kvs_launch_horizon_choose(const HorizonKept &h, int32_t *order, int32_t n, const int32_t *moves, const int64_t *result,
                              const int32_t *d_words, int32_t stride, int64_t completed_in, int32_t complete_every,
                              int32_t full, hipStream_t st)
{
    hipLaunchKernelGGL(horizon_choose_kernel, dim3(1), dim3(1024), 0, st, h, order, n, moves, result, d_words, stride,
                       (long long)completed_in, complete_every, full);
    return ok();
}

int kvs_launch_horizon_advance(const HorizonKept &h, const int32_t *order, int32_t n, int32_t blocks, int64_t completed_in,
                               int32_t complete_every, int32_t *completion_out, int64_t *result_out, hipStream_t st)
{
    hipLaunchKernelGGL(horizon_advance_kernel, dim3(1), dim3(1024), 0, st, h, order, n, blocks, (long long)completed_in,
                       complete_every, completion_out, result_out);
    return ok();
}

int kvs_launch_horizon_advance_by_id(const int32_t *order, const int32_t *completion, const int32_t *o, int32_t n,
                                     int64_t completed_in, int32_t complete_every, int64_t *result, hipStream_t st)
{
    hipLaunchKernelGGL(horizon_advance_by_id_kernel, dim3(1), dim3(1024), 0, st, order, completion, o, n,
                       (long long)completed_in, complete_every, result);
    return ok();
}

int kvs_launch_horizon_completion(const HorizonKept &h, const int32_t *order, const int32_t *o, int32_t n,
                                  int32_t *completion_out, hipStream_t st)
{
    hipLaunchKernelGGL(horizon_completion_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, h, order, o, n,
                       completion_out);
    return ok();
}
