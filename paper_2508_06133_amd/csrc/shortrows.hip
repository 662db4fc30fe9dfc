// Phase 2 of Algorithm 1 for many orders of a few requests: ONE LANE PER ORDER.
//
// A wavefront per order (timeline_reg.hip) is made for profiles of many rounds; an order of eight requests costs it
// its start, two dependent rounds of loads and a turn for each request, all of which 64 lanes share here.  A lane keeps
// the completion rounds c_i of the requests it has placed in registers, latest first, and with each the memory reserved for that
// round and the round once more, b_i: as request k holds s_k - start_k + tau in round tau, b_i is the sum of the first i + 1 of s_k -
// start_k, plus (i + 2) c_i.  Memory rises from one completion to the next, so a request (s, o) may start in round t
// iff the completion rounds among t + 1 .. t + o, and round t + o, have room for it.
//
// One pass over the completions, from the earliest on, finds the start.  Where c_i lies within t + 1 .. t + o it rules out every start
// before min(c_i, b_i + s - M).  Where it is the first behind that, the last round t + o has to have room beside the first i + 1
// requests; if it has not, no start has whose last round comes before c_i or with it, as memory only rises until then, and the
// start moves to c_i + 1 - o, where c_i is within its rounds and rules out what it does (no less than round t + o did).  Later
// completions find more room in that round, as fewer requests are left, so none of them moves a start that fits; and a start that an
// earlier one has been passed for does not come back to it.  With x = c_i - o one comparison serves all cases: the room that round t + o
// has beside the first i + 1 requests, also where c_i comes before it (it only seems less then, and max(x + 1, min(c_i, b_i + s - M)) is
// beyond t only if that completion is in the way).
//
// The ids are read as whole rows and the completion rounds written by request id through LDS; that an order is a
// permutation comes out on the way.  So there is no second pass over the rows.
//
// Bound by the chain of its vector instructions: ten for each completion, three of them behind the one before, and seven to keep
// them in order.  With a look at all completions after each move of the start, and one more (as many as there are completions, if the
// memory is tight), 8 and 16 requests a row and 65536 rows were 7.7 and 17.0 us a call, 7.0 and 14.5 now, 24 and 32 34.6 and 59.0, now 28.0
// and 41.2; 16384 rows of 16 that wait more 26.5, now 13.1; every order of 8 in a budget of 3 requests 7.8, now 6.4 (the launch alone takes 6).
// The time hardly depends on the lengths.  Where many short requests wait for long ones the timeline kernel
// looks at many more rounds: 16 requests of 1 or 4096 tokens and rounds, 8192 orders 13 us (2116).
#include "kvsched_internal.h"
#include "device_util.h"

#include <climits>

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

    int c[N];       // completion rounds placed so far, latest first
    unsigned b[N];  // the memory reserved for round c[i], and c[i] once more
#pragma unroll
    for (int i = 0; i < N; ++i) c[i] = -1, b[i] = 0;  // none placed
    int t = 0, tel = 0, met = 0;
    bool permutation = true, valid = true;
    const int *ids = row + lane * PITCH;  // (lanes without an order place what is there, of no account)
    const int longest = min(p.o_bound, M);
    int raw = ids[0], id = min(max(raw, 0), n - 1), s_next = len_s[id], o_next = len_o[id];
    for (int k = 0; k < n; ++k) {
        permutation &= raw == id && ((met >> id) & 1) == 0;
        met |= 1 << id;
        const int here = id;
        // (1 <= o <= longest <= M, hence M - o >= 0, and 1 <= s <= M - o)
        const bool good = (unsigned)o_next - 1u < (unsigned)longest && (unsigned)s_next - 1u < (unsigned)M - (unsigned)o_next;
        valid &= good;  // a request that cannot be scheduled ends in the round it is reached in and holds nothing
        const int s = good ? s_next : 0, o = good ? o_next : 0;
        raw = ids[min(k + 1, n - 1)];  // (the next one's lengths are on their way meanwhile)
        id = min(max(raw, 0), n - 1);
        s_next = len_s[id];
        o_next = len_o[id];
        // (it is looked at as one round without a token, s + 1 = 0, which no completion moves; as no rounds a completion in round t
        // itself could be in its way)
        const int rounds = good ? o : 1;
        const unsigned over = (unsigned)((good ? s : -1) - M);
#pragma unroll
        for (int f = N - 4; f >= 0; f -= 4) {
            if (k <= f) continue;  // (uniform: four places that are empty yet)
#pragma unroll
            for (int i = f + 3; i >= f; --i) {
                const int bound = (int)(b[i] + over), x = c[i] - rounds;
                const int least = max(x + 1, min(c[i], bound));
                const int at_x = bound - __mul24(x, i + 2);
                t = at_x + __mul24(t, i + 2) > t ? max(t, least) : t;
            }
        }
        const int c_new = t + o;
        const unsigned a_new = (unsigned)(s - t);
        tel += c_new;
        done[lane * PITCH + here] = c_new;
#pragma unroll
        for (int f = N - 4; f >= 0; f -= 4) {  // to its place among the completions
            if (k < f) continue;
#pragma unroll
            for (int i = f + 3; i >= f; --i) {
                const bool keep = c[i] >= c_new;
                const int c_left = i > 0 ? c[i > 0 ? i - 1 : 0] : INT_MAX;
                const unsigned b_in = i > 0 ? b[i > 0 ? i - 1 : 0] + (unsigned)c_left + a_new + (unsigned)__mul24(min(c_new - c_left, 0), i + 2)
                                            : a_new + 2u * (unsigned)c_new;
                c[i] = keep ? c[i] : min(c_left, c_new);
                b[i] = keep ? b[i] : b_in;
            }
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

// Are `rows` orders of n requests placed a lane each?  The chain grows with the square of the requests and does not shrink with the
// orders: 9 chat requests 7.2 us (timeline kernel: 4096 orders 6.8, 8192 8.8), 12 9.3 (8.2, 11.4), 16 13 (10.7, 15.3), 24 24 (8192 18.5,
// 16384 31.1), 32 36 (21.7, 36.4).
bool kvs_short_rows(int32_t rows, int32_t n)
{
    return n <= 32 && (n <= 8 || rows >= 512 * n);
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
