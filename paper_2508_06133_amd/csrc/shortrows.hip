// Phase 2 of Algorithm 1 for many orders of a few requests: ONE LANE PER ORDER.
//
// A wavefront per order (timeline_reg.hip) is made for profiles of many rounds; an order of eight requests costs it
// its start, two dependent rounds of loads and a turn for each request, all of which 64 lanes share here.  A lane keeps
// the requests it has placed as pairs (completion round c_i, s_i - start) in registers, latest completion first.  The memory
// reserved for round c_i is then the sum of the first i + 1 second parts plus (i + 1) c_i, a running sum with
// factors known at compile time.  Memory rises from one completion to the next, so a request (s, o) may start in round t
// iff the completion rounds among t + 1 .. t + o, and round t + o, have room for it.  Round tau rules out every start
// before min(tau, memory(tau) + s + tau - M): the start moves to the largest of these until none is behind it.  If round t + o
// has no room, no start has whose last round comes before the next completion or with it, as memory only rises until then.
// (Without that a request of one round, which looks at the round ahead only, went through every round it waited: 8192 orders
// of 16 requests of 1 or 4096 tokens and rounds, M = 8192, 17 ms instead of 25 us.)  Every turn that moves the
// start settles a completion round for good, so there is at most one more turn than there are completions.
//
// The ids are read as whole rows and the completion rounds written by request id through LDS; that an order is a
// permutation comes out on the way.  So there is no second pass over the rows.
//
// Bound by the chain of its vector instructions, ten for each place of the arrays in each look at a start round: a call of
// 65536 orders of 4 or 8 chat requests takes 11 us where the timeline kernel takes 36 and 44, of 16 requests 20 (55), of 24 40 (79),
// of 32 58 (103).  The chain grows with the square of the requests and does not shrink with the orders, so longer orders
// need more of them: 8192 orders of 9 requests 12.1 us (12.4), of 12 14.6 (12.4), of 16 17.8 (13.0), 16384 of 16 18.1 (18.5), of
// 24 37 (26), 32768 of 17 / 24 / 32 27 / 39 / 55 (36 / 44 / 57).  Where many short requests wait for long ones the timeline kernel
// looks at many more rounds: 16 requests of 1 or 4096 tokens and rounds, 8192 orders at M = 8192 25 us (4400), 16384 at M = 16384
// 24 (73).  So orders of 9 to 16 requests take this way from 8192 on, where the chat ones alone would have it at 16384.
#include "kvsched_internal.h"
#include "device_util.h"

namespace {

template <int N>
__global__ __launch_bounds__(64) void short_rows_kernel(SimParams p, int32_t o_limit)
{
    constexpr int PITCH = N + 1;  // (odd: the lanes' entries lie in different banks)
    __shared__ int row[64 * PITCH], done[64 * PITCH], len_s[N], len_o[N];
    const int lane = threadIdx.x, n = p.n, M = p.M;
    const int first = (int)blockIdx.x * 64, mine = min(64, p.C - first);
    const int32_t *orders = p.src.orders + (size_t)first * (size_t)n;
    const int entries = mine * n;
    int o_max = p.scan_here ? 0 : p.d_words[KVS_W_OMAX];
    for (int e = lane; e < entries; e += 64) row[(e / n) * PITCH + e % n] = orders[e];
    const int s_mine = lane < n ? p.s[lane] : 1, o_mine = lane < n ? p.o[lane] : 1;
    if (lane < N) {
        len_s[lane] = s_mine;
        len_o[lane] = o_mine;
    }
    if (p.scan_here) {
        o_max = wave_max_i32(lane < n ? o_mine : 0);
        o_limit = p.scan_limit;
        if (blockIdx.x == 0) {
            const int flags = lane < n ? length_flags(s_mine, o_mine, M, p.scan_bound) : 0;
            const int all = wave_max_i32(flags & KVSCHED_DEV_BAD_LENGTH) | wave_max_i32(flags & KVSCHED_DEV_O_MAX);
            if (lane == 0) report_lengths(p, o_max, all);
        }
    }
    __syncthreads();
    if (o_max > o_limit) return;  // (the rows are placed by a later launch)

    int c[N], a[N];
#pragma unroll
    for (int i = 0; i < N; ++i) c[i] = -1, a[i] = 0;  // none placed
    int t = 0, tel = 0, met = 0;
    bool permutation = true, valid = true;
    const int *ids = row + lane * PITCH;  // (lanes without an order place what is there, of no account)
    for (int k = 0; k < n; ++k) {
        const int raw = lane < mine ? ids[k] : 0;
        const int id = min(max(raw, 0), n - 1);
        permutation &= raw == id && ((met >> id) & 1) == 0;
        met |= 1 << id;
        int s = len_s[id], o = len_o[id];
        if (s < 1 || o < 1 || o > p.o_bound || (long long)s + o > (long long)M) {  // cannot be scheduled
            valid = false;
            s = o = 0;  // ends where it starts and holds nothing: the look below moves no start for it
        }
        for (;;) {
            const int end = t + o;
            int start = t, sum = s - M, at_end = sum, behind = 1;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                sum += a[i];
                const bool holds = c[i] >= end;
                at_end = holds ? sum : at_end;
                behind = holds ? i + 2 : behind;
                const int bound = min(c[i], sum + (int)__umul24((unsigned)c[i], i + 2));
                start = (unsigned)(c[i] - t - 1) < (unsigned)o ? max(start, bound) : start;
            }
            const int free_end = at_end + (int)__umul24((unsigned)end, (unsigned)behind);
            if (__builtin_amdgcn_ballot_w64(free_end > t && o > 0) != 0) {
                int next = 0;  // the first completion round at or behind `end` (there is one)
#pragma unroll
                for (int i = 0; i < N; ++i) next = c[i] >= end ? c[i] : next;
                if (free_end > t && o > 0) start = max(start, max(min(end, free_end), next - o + 1));
            }
            const bool moved = start > t;
            t = start;
            if (__builtin_amdgcn_ballot_w64(moved) == 0) break;
        }
        const int c_new = t + o, a_new = s - t;
        tel += c_new;
        done[lane * PITCH + id] = c_new;
#pragma unroll
        for (int i = N - 1; i >= 0; --i) {  // to its place among the completions
            const bool keep = c[i] >= c_new, here = i == 0 || c[i > 0 ? i - 1 : 0] >= c_new;
            const int from_c = here ? c_new : c[i > 0 ? i - 1 : 0], from_a = here ? a_new : a[i > 0 ? i - 1 : 0];
            c[i] = keep ? c[i] : from_c;
            a[i] = keep ? a[i] : from_a;
        }
    }
    if (lane < mine) {
        if (!permutation) atomicOr(&p.d_words[p.status_word], KVSCHED_DEV_BAD_ORDER);
        p.tel_out[first + lane] = permutation && valid ? (int64_t)tel : -1;
    }
    if (!p.completion_out) return;
    if (!permutation)  // requests that do not occur
        for (int i = 0; i < n; ++i)
            if (((met >> i) & 1) == 0) done[lane * PITCH + i] = -1;
    __syncthreads();
    int32_t *out = p.completion_out + (size_t)first * (size_t)n;
    for (int e = lane; e < entries; e += 64) out[e] = done[(e / n) * PITCH + e % n];
}

}  // namespace

// Are `rows` orders of n requests placed a lane each?  (The lines are measured at the top of the file.)
bool kvs_short_rows(int32_t rows, int32_t n)
{
    return n <= 8 ? rows >= KVS_SHORT_ROWS_8 : n <= 16 ? rows >= KVS_SHORT_ROWS_16 : n <= 32 && rows >= KVS_SHORT_ROWS_32;
}

// p.tel_out and p.completion_out (by request id) of every row, checked; nothing is written if words[KVS_W_OMAX] > o_limit.
int kvs_launch_short_rows(const SimParams &p, int32_t o_limit, hipStream_t st)
{
    const dim3 blocks((unsigned)((p.C + 63) / 64));
    if (p.n <= 8) hipLaunchKernelGGL(short_rows_kernel<8>, blocks, dim3(64), 0, st, p, o_limit);
    else if (p.n <= 16) hipLaunchKernelGGL(short_rows_kernel<16>, blocks, dim3(64), 0, st, p, o_limit);
    else if (p.n <= 32) hipLaunchKernelGGL(short_rows_kernel<32>, blocks, dim3(64), 0, st, p, o_limit);
    else return KVSCHED_ERANGE;
    return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}
