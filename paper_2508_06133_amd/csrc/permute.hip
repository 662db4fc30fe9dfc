// Completion rounds from position order to request-id order.
//
// The timeline kernels produce the completion round of every position of a candidate order;
// callers want it per request id (c_i of Section 2, "Objective").  Storing by id from the
// timeline kernel means 4-byte stores scattered over an 8 KB row while thousands of rows are
// in flight: measured HBM write traffic was 9x the payload.  Instead the timeline kernel stores
// by position (256 contiguous bytes per 64 positions) and this kernel permutes each row in
// place: one workgroup per row, the row staged in LDS, read and written coalesced.  The same pass
// over the order row checks that it is a permutation of 0..n-1 (a bitmap of n bits beside the row).
// A row that was resumed from row 0's timeline after 64 b positions did not place those itself: their
// completion rounds are row 0's, taken from a copy of row 0's row in position order.  Likewise a row
// that stopped at position 64 b' because its timeline had become row 0's again: from there on every
// request completes when it does in row 0 (the positions are then those of row 0's order: behind the
// last difference the two orders are the same, and a row that placed nothing holds the same requests
// as row 0 wherever they differ).
#include "kvsched_internal.h"

#include <limits.h>

namespace {

__global__ __launch_bounds__(256) void permute_rows_kernel(const int32_t *orders, int32_t n, int32_t *completion,
                                                           int64_t *tel_out, int32_t *words,
                                                           const int32_t *resume_block, const int32_t *row0,
                                                           const int32_t *rejoin_block, int32_t o_limit, const int32_t *todo)
{
    if (todo && todo[blockIdx.x] == 0) return;
    const int o_max = words[KVS_W_OMAX];
    extern __shared__ int row_by_id[];
    unsigned int *seen = (unsigned int *)(row_by_id + n);  // one bit per request id
    const int32_t *order = orders + (size_t)blockIdx.x * (size_t)n;
    int32_t *comp = completion + (size_t)blockIdx.x * (size_t)n;
    for (int i = threadIdx.x; i < ((n + 31) >> 5); i += blockDim.x) seen[i] = 0;
    const int shared = resume_block ? min(64 * resume_block[blockIdx.x], n) : 0;  // positions placed by row 0 only
    int tail = n;  // ... and from here on
    if (rejoin_block && rejoin_block[blockIdx.x] != INT_MAX) tail = min(64 * rejoin_block[blockIdx.x], n);
    __syncthreads();
    int bad = 0;
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        const int raw = order[k];
        const int r = min(max(raw, 0), n - 1);
        const unsigned int bit = 1u << (r & 31);
        if (raw != r || (atomicOr(&seen[r >> 5], bit) & bit)) bad = 1;  // out of range, or met before
        if (k < tail) row_by_id[r] = k < shared ? row0[k] : comp[k];
    }
    for (int k = tail + threadIdx.x; k < n; k += blockDim.x) row_by_id[min(max(orders[k], 0), n - 1)] = row0[k];
    bad = __syncthreads_or(bad);
    if (o_max > o_limit) return;  // the rows have not been placed (looked at this late: the other reads hide it)
    if (bad && threadIdx.x == 0) {  // the row is no permutation: its results are void
        tel_out[blockIdx.x] = -1;
        atomicOr(&words[KVS_W_STATUS], KVSCHED_DEV_BAD_ORDER);
    }
    if (bad)  // (-1 for requests that do not occur)
        for (int i = threadIdx.x; i < n; i += blockDim.x)
            if (((seen[i >> 5] >> (i & 31)) & 1u) == 0) row_by_id[i] = -1;
    for (int i = threadIdx.x; i < n; i += blockDim.x) comp[i] = row_by_id[i];
}

// The same for short rows placed in full: a workgroup takes as many whole rows as make some 1024 entries and runs
// over them as one contiguous stretch.  (A workgroup per row of 8 entries leaves 248 threads idle and costs its
// launch: 40321 such rows 31.5 us, so 4.2.)
constexpr int kShortRow = 256, kShortEntries = 1024;
__global__ __launch_bounds__(256) void permute_short_rows_kernel(const int32_t *orders, int32_t C, int32_t n, int32_t rows,
                                                                 int32_t *completion, int64_t *tel_out, int32_t *words,
                                                                 int32_t o_limit)
{
    const int o_max = words[KVS_W_OMAX];
    __shared__ int by_id[kShortEntries];
    __shared__ unsigned int seen[kShortEntries + kShortEntries / 32];
    __shared__ int bad[kShortEntries];
    const int row0 = blockIdx.x * rows;
    const int mine = min(rows, C - row0), entries = mine * n, nw = (n + 31) >> 5;
    const int32_t *order = orders + (size_t)row0 * (size_t)n;
    int32_t *comp = completion + (size_t)row0 * (size_t)n;
    for (int i = threadIdx.x; i < mine * nw; i += 256) seen[i] = 0;
    for (int i = threadIdx.x; i < mine; i += 256) bad[i] = 0;
    for (int e = threadIdx.x; e < entries; e += 256) by_id[e] = -1;  // (what requests that do not occur are left with)
    __syncthreads();
    for (int e = threadIdx.x; e < entries; e += 256) {
        const int row = e / n;
        const int raw = order[e];
        const int r = min(max(raw, 0), n - 1);
        const unsigned int bit = 1u << (r & 31);
        if (raw != r || (atomicOr(&seen[row * nw + (r >> 5)], bit) & bit)) bad[row] = 1;
        by_id[row * n + r] = comp[e];
    }
    __syncthreads();
    if (o_max > o_limit) return;  // the rows have not been placed (looked at this late: the other reads hide it)
    for (int i = threadIdx.x; i < mine; i += 256) {
        if (bad[i]) {
            tel_out[row0 + i] = -1;
            atomicOr(&words[KVS_W_STATUS], KVSCHED_DEV_BAD_ORDER);
        }
    }
    for (int e = threadIdx.x; e < entries; e += 256) comp[e] = by_id[e];
}

}  // namespace

int kvs_launch_permute_rows(const int32_t *orders, int32_t C, int32_t n, int32_t *completion, int64_t *tel_out,
                            int32_t *d_words, const int32_t *resume_block, const int32_t *row0,
                            const int32_t *rejoin_block, hipStream_t st, int32_t o_limit, const int32_t *todo)
{
    if (n > KVS_PERMUTE_MAX_N) return KVSCHED_ERANGE;
    if (n <= kShortRow && !resume_block && !todo) {
        const int rows = kShortEntries / n;
        hipLaunchKernelGGL(permute_short_rows_kernel, dim3((unsigned)((C + rows - 1) / rows)), dim3(256), 0, st, orders, C, n,
                           rows, completion, tel_out, d_words, o_limit);
        return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
    }
    const size_t lds = sizeof(int32_t) * ((size_t)n + (((size_t)n + 31) >> 5));
    hipLaunchKernelGGL(permute_rows_kernel, dim3((unsigned)C), dim3(256), lds, st, orders, n, completion, tel_out,
                       d_words, resume_block, row0, rejoin_block, o_limit, todo);
    return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}
