// Phase 2 of Algorithm 1 for explicit orders, one 64-lane wavefront per order, ONE LANE PER COMPLETION ROUND.
//
// The timeline kernel (timeline_reg.hip) keeps the reserved memory of every future round and pays for each request by the rounds
// it runs.  Here a lane keeps a round c at which requests complete, the memory P(c) reserved for it and the number N(c) of requests that
// still run in it; between two of these rounds the memory rises by one token a round and running request, so they say all there is to
// know, and a request costs the same whether it runs one round or fourteen thousand.  The lanes are in no order; those with c <= t are
// free.  A row whose requests complete in more than 64 different rounds ahead gives up and says so in todo[]; the timeline kernel places
// it.  Orders of up to 64 requests never do.  Orders are taken here where the decode lengths are few (KVS_FEW_LENGTHS of them among 64
// requests), and then mostly a handful of lanes is in use: 4 on average and 18 at most for an order of 100000 requests of 1 or 4096 tokens
// with 64 exchanges.
//
// Start of a request (s, o) at t or later.  Completion c_i <= t + o rules out every start before min(c_i, P(c_i) + s + c_i - M): started
// later the request is smaller at c_i, or no longer overlaps it.  c_i > t + o: round t + o has P(c_i) - N(c_i) (c_i - t - o) tokens
// reserved if c_i is the first completion behind it, and less is reserved beside any later one alone; where that and s + o exceed M,
// no start has its last round before c_i, as memory only rises until then, and the bound of c_i as above holds too.  All lanes test
// at once, the start moves to the largest of these, until none moves it.
//
// Requests that start together (a burst): as long as the next ones' memory, added up, stays within what every round behind t has left, all of
// them start in t.  Two stretches are told apart, the rounds up to t + a and those behind, with a the least decode length of the requests
// looked at: a request of up to a rounds is in the first stretch only, so a mixture of long and short ones is taken at once as
// well.  GROUP positions are looked at together, four consecutive ones a lane.  The request behind those that fit is placed alone, and so are
// the next few (`patience`) where looking has found next to nothing; what a burst adds is entered length by length.
//
// Bound: the latency of one wavefront's chain of dependent instructions, some nine cycles each (1000 orders of 100000: 125 k vector and 70 k
// scalar ones a row, a quarter of the vector issue slots, half of the time in waits for the lane moves and for the scattered stores).
// The row's ids and lengths therefore come a chunk ahead through LDS, its completion rounds leave together behind the wait for the next
// chunk's lengths, so that no wait is for a store of less than a chunk ago, and a bit per request met, in LDS, checks the row on the way.
// Per call, the timeline kernel and here (us; bimodal lengths unless said otherwise): 1025 orders of 100000, 64 exchanges 2786 and 1060,
// 400 of 6042 748 and 230, 8000 of 3000 1570 and 705, 7791 of 942 1630 and 630, 32768 of 203 2130 and 744, one of 1384 327 and 120, two of
// 131 82 and 47, one of 26 18.4 and 12.2; 1000 of 2000 with four lengths up to 4096 790 and 610, of 10000 3700 and 3400.
#include "kvsched_internal.h"
#include "device_util.h"

#include <climits>

namespace {

constexpr int GROUP = 4 * WAVE;  // positions looked at together, four consecutive ones a lane
constexpr int BLOCKS = 2;        // ... in a chunk
// How many requests are placed one by one after a look for a burst has found less than four: more each time, and from PATIENT on also if the
// round moves meanwhile.  (32768 orders of 203 in a budget of one and a half requests 756 us with 7, 677 with 31; but one in a hundred
// orders of 100000 with a burst in every round is then placed one by one to its end, 1025 of them 1270 and 1156.)
constexpr int MOST_PATIENCE = 7, PATIENT = 3;

template <int CTRL, int ROWS>
__device__ __forceinline__ int from_lane(int old, int v)
{
    return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false);
}

// Largest of the 64 lanes' numbers.
__device__ __forceinline__ int lanes_max(int v)
{
    v = max(v, from_lane<0xB1, 0xf>(INT_MIN, v));
    v = max(v, from_lane<0x4E, 0xf>(INT_MIN, v));
    v = max(v, from_lane<0x141, 0xf>(INT_MIN, v));
    v = max(v, from_lane<0x140, 0xf>(INT_MIN, v));
    v = max(v, from_lane<0x142, 0xa>(INT_MIN, v));
    v = max(v, from_lane<0x143, 0xc>(INT_MIN, v));
    return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ int lanes_min(int v) { return ~lanes_max(~v); }

// Lane l: the sum over lanes 0 .. l.
__device__ __forceinline__ int lanes_prefix(int v)
{
    v += from_lane<0x111, 0xf>(0, v);
    v += from_lane<0x112, 0xf>(0, v);
    v += from_lane<0x114, 0xf>(0, v);
    v += from_lane<0x118, 0xf>(0, v);
    v += from_lane<0x142, 0xa>(0, v);
    v += from_lane<0x143, 0xc>(0, v);
    return v;
}

__device__ __forceinline__ int lane_of(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ bool in_mask(unsigned long long m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
__device__ __forceinline__ unsigned long long ballot(bool v) { return __builtin_amdgcn_ballot_w64(v); }
// max(a - b, 0) of numbers from 0 on
__device__ __forceinline__ int beyond(int a, int b) { return (int)__builtin_elementwise_sub_sat((unsigned)a, (unsigned)b); }

__device__ __forceinline__ void wave_sync()
{
    // LDS traffic of one wavefront is served in order; this keeps the compiler from moving accesses across a point where lanes
    // read what other lanes wrote, or write where they have read
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The completion rounds ahead, a lane each.
struct Events {
    int t = 0;  // start round of the last request
    int c = 0;  // completion round (free lane: c <= t)
    int b = 0;  // P(c) + c (of a free lane: anything; sums are modulo 2^32)
    int n = 0;  // N(c)
    bool full = false;

    // what is reserved for round `at` (t < at) beside the lane's completion and later ones: exact in the first lane from `at` on
    __device__ __forceinline__ int reserved(int at) const
    {
        return (int)((unsigned)b - (unsigned)c - (unsigned)n * (unsigned)beyond(c, at));
    }

    // g requests of s tokens together, started in round t, that end in round t + o
    __device__ __forceinline__ void enter(int s, int g, int o)
    {
        const int end = t + o;
        const bool le = c <= end;
        b = le ? (int)((unsigned)b + (unsigned)s + (unsigned)g * (unsigned)(c - t)) : b;
        n += le ? g : 0;
        if (ballot(c == end) != 0) return;
        const unsigned long long free_lanes = ballot(c <= t);
        if (free_lanes == 0) {
            full = true;
            return;
        }
        int p = 0, m = 0;
        const unsigned long long behind = ballot(c > end);
        if (behind != 0) {
            const int next = lanes_min(c > end ? c : INT_MAX);
            const int l = __builtin_ctzll(ballot(c == next));
            m = lane_of(n, l);
            p = lane_of(b, l) - next - m * (next - end);
        }
        const bool mine = in_mask(free_lanes & (0 - free_lanes));
        c = mine ? end : c;
        b = mine ? p + s + g * o + end : b;
        n = mine ? m + g : n;
    }
};

typedef int four __attribute__((ext_vector_type(4)));

// Of the GROUP positions, four a lane, number k (the same in all lanes).
__device__ __forceinline__ int pick(four v, int k)
{
    const int l = k >> 2;
    const int v0 = lane_of(v[0], l), v1 = lane_of(v[1], l), v2 = lane_of(v[2], l), v3 = lane_of(v[3], l);
    const int low = (k & 1) != 0 ? v1 : v0, high = (k & 1) != 0 ? v3 : v2;
    return (k & 2) != 0 ? high : low;
}

constexpr int CHUNK = BLOCKS * GROUP, PIECES = CHUNK / WAVE;

__global__ __launch_bounds__(WAVE) void event_rows_kernel(SimParams p)
{
    extern __shared__ unsigned met[];  // a bit per request id
    __shared__ __align__(16) int kept_s[CHUNK], kept_o[CHUNK], kept_id[CHUNK];
    const int lane = threadIdx.x, cand = blockIdx.x, n = p.n, M = p.M;
    const int words = (n + 31) >> 5;
    const int32_t *row = p.src.orders + (size_t)cand * (size_t)n;
    int32_t *crow = p.completion_out ? p.completion_out + (size_t)cand * (size_t)n : nullptr;

    // The ids and lengths of a chunk, position 64 q + lane of it in number q.  (Past the end the last position's, or the shortest.)
    // No length is read by an id that has not been clamped.
    int id[PIECES], sv[PIECES], ov[PIECES], id_next[PIECES];
#pragma unroll
    for (int q = 0; q < PIECES; ++q) id[q] = id_next[q] = 0, sv[q] = ov[q] = 1;
    auto fetch_ids = [&](int (&to)[PIECES], int first) __attribute__((always_inline)) {
        if (first + CHUNK <= n) {
#pragma unroll
            for (int q = 0; q < PIECES; ++q) to[q] = row[first + WAVE * q + lane];
        } else {
#pragma unroll
            for (int q = 0; q < PIECES; ++q)
                if (first + WAVE * q < n) to[q] = row[min(first + WAVE * q + lane, n - 1)];
        }
    };
    bool strange = false;  // an id that there is not
    for (int w = lane; w < words; w += WAVE) met[w] = 0;
    wave_sync();
    auto clamped = [&](int raw) __attribute__((always_inline)) -> int { return min(max(raw, 0), n - 1); };
    auto meet = [&](int raw) __attribute__((always_inline)) -> int {
        const int r = clamped(raw);
        strange |= raw != r;
        atomicOr(&met[r >> 5], 1u << (r & 31));
        return r;
    };
    auto length_of = [&](int q) __attribute__((always_inline)) {
        const unsigned at = (unsigned)id[q] * 4u;
        sv[q] = *(const int32_t *)((const char *)p.s + at);
        ov[q] = *(const int32_t *)((const char *)p.o + at);
    };
    auto fetch_lengths = [&](int first) __attribute__((always_inline)) {
        if (first + CHUNK <= n) {
#pragma unroll
            for (int q = 0; q < PIECES; ++q) {
                id[q] = meet(id[q]);
                length_of(q);
            }
        } else {
#pragma unroll
            for (int q = 0; q < PIECES; ++q) {
                if (first + WAVE * q >= n) continue;
                // (the lanes past the end hold the last id as it stands, which may be none; met they are not: lanes that mean one word take turns)
                id[q] = first + WAVE * q + lane < n ? meet(id[q]) : clamped(id[q]);
                length_of(q);
            }
        }
    };
    fetch_ids(id, 0);
    const int sample = p.o[sampled(lane, n)];
    fetch_ids(id_next, CHUNK);
    fetch_lengths(0);
    if (p.gate && *p.gate > p.o_bound) return;
    if (p.scan_here) {
        int longest = 0, flags = 0;
        for (int k = lane; k < n; k += WAVE) {
            const int o = p.o[k];
            longest = max(longest, o);
            if (cand == 0) flags |= length_flags(p.s[k], o, M, p.scan_bound);
        }
        longest = lanes_max(longest);
        if (cand == 0) {
            const int all = lanes_max(flags & KVSCHED_DEV_BAD_LENGTH) | lanes_max(flags & KVSCHED_DEV_O_MAX);
            if (lane == 0) report_lengths(p, longest, all);
        }
        if (longest > p.scan_limit) {
            if (p.todo && lane == 0) p.todo[cand] = 0;
            return;
        }
    }
    const bool few = few_lengths(sample);
    if (p.scan_here && cand == 0 && lane == 0) report_few(p, few);
    if (p.todo && !few) {
        if (lane == 0) p.todo[cand] = 1;
        return;
    }
    const int longest_o = min(p.o_bound, M);
    const int shift = max(0, 10 - __builtin_clz(M));  // sums of GROUP sizes (and one more each) in units of 2^shift stay below 2^31
    const unsigned up = shift > 0 ? 1u : 0u;

    Events e;
    long long tel = 0;
    int patience = 0, look = 0;       // requests to be placed one by one before a burst is looked for
    bool known = false;               // what every round behind t has left is at least:
    int a = 0, room1 = 0, room2 = 0;  // in rounds t + 1 .. t + a, and behind
    bool bad_length = false;

    for (int chunk = 0; chunk < n; chunk += CHUNK) {
#pragma unroll
        for (int q = 0; q < PIECES; ++q) {
            kept_s[WAVE * q + lane] = sv[q];
            kept_o[WAVE * q + lane] = ov[q];
            kept_id[WAVE * q + lane] = id[q];
            id[q] = id_next[q];
        }
        wave_sync();
        fetch_lengths(chunk + CHUNK);
        fetch_ids(id_next, chunk + 2 * CHUNK);
        for (int q = 0; q < BLOCKS && chunk + GROUP * q < n; ++q) {
            const int cnt = min(GROUP, n - chunk - GROUP * q);
            four s = *(const four *)&kept_s[GROUP * q + 4 * lane], o = *(const four *)&kept_o[GROUP * q + 4 * lane];
            // (o <= longest and s + o <= M, both from 1 on)
            unsigned longest = 0, largest = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                longest = max(longest, (unsigned)o[j] - 1u);
                largest = max(largest, __builtin_elementwise_add_sat((unsigned)s[j] - 1u, (unsigned)o[j]));
            }
            if ((ballot(longest >= (unsigned)longest_o) | ballot(largest >= (unsigned)M)) != 0) {
                bad_length = true;
                break;
            }
            four done;
#pragma unroll
            for (int j = 0; j < 4; ++j) done[j] = e.t + o[j];  // (unless the round moves before)
            if (cnt < GROUP) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const bool in = 4 * lane + j < cnt;
                    s[j] = in ? s[j] : 0;
                    o[j] = in ? o[j] : 0;
                }
            }
            int first = 0, cleared = 0;
            for (;;) {
                if (look == 0) {
                    if (first > cleared) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const bool placed = 4 * lane + j < first;
                            s[j] = placed ? 0 : s[j];
                            o[j] = placed ? 0 : o[j];
                        }
                        cleared = first;
                    }
                    const int most = max(max(o[0], o[1]), max(o[2], o[3]));
                    const bool fresh = !known;
                    if (fresh) {
                        unsigned least = (unsigned)o[0] - 1u;
#pragma unroll
                        for (int j = 1; j < 4; ++j) least = min(least, (unsigned)o[j] - 1u);
                        a = lanes_min((int)min(least, (unsigned)INT_MAX - 1u)) + 1;
                        room1 = M - lanes_max(e.c > e.t ? e.reserved(e.t + a) : 0);
                        room2 = M - lanes_max(e.c > e.t + a ? e.b - e.c : 0);
                        known = true;
                    }
                    // what the requests hold at most in the rounds up to t + a, and behind
                    unsigned up_to1[4], up_to2[4] = {0, 0, 0, 0};
#pragma unroll
                    for (int j = 0; j < 4; ++j) up_to1[j] = (unsigned)(s[j] + min(o[j], a)) + (j > 0 ? up_to1[j > 0 ? j - 1 : 0] : 0u);
                    const int sum1 = lanes_prefix((int)((up_to1[3] >> shift) + up));
                    unsigned long long over = ballot(sum1 > room1 >> shift);
                    int sum2 = 0;
                    const bool longer = ballot(most > a) != 0;
                    if (longer) {
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            up_to2[j] = (o[j] > a ? (unsigned)(s[j] + o[j]) : 0u) + (j > 0 ? up_to2[j > 0 ? j - 1 : 0] : 0u);
                        sum2 = lanes_prefix((int)((up_to2[3] >> shift) + up));
                        over |= ballot(sum2 > room2 >> shift);
                    }
                    int to = cnt, taken = 0;  // (taken: if shift == 0)
                    four os = o, ss = s;
                    if (over == 0) {
                        taken = lane_of(sum1, WAVE - 1);
                        room1 -= taken << shift;
                        room2 -= longer ? lane_of(sum2, WAVE - 1) << shift : 0;
                    } else {  // the lanes before that one whole, and of its four as many as fit
                        const int l = __builtin_ctzll(over);
                        int fits = 0, held = 0;
                        if (shift == 0) {
                            const int left1 = room1 - (sum1 - (int)up_to1[3]), left2 = room2 - (sum2 - (int)up_to2[3]);
#pragma unroll
                            for (int j = 0; j < 3; ++j) {
                                const bool fit = (int)up_to1[j] <= left1 && (int)up_to2[j] <= left2;
                                held = fit ? (int)up_to1[j] : held;
                                fits += fit ? 1 : 0;
                            }
                            held += sum1 - (int)up_to1[3];
                        }
                        to = max(4 * l + lane_of(fits, l), first);
                        taken = lane_of(held, l);
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const bool now = 4 * lane + j < to;
                            os[j] = now ? o[j] : 0;
                            ss[j] = now ? s[j] : 0;
                        }
                    }
                    const int g = to - first;
                    for (int left = g; left > 0;) {  // length by length
                        const int longest_left = max(max(os[0], os[1]), max(os[2], os[3]));
                        const int length = lane_of(longest_left, __builtin_ctzll(ballot(longest_left != 0)));
                        int tokens = 0, count = 0;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const bool same = os[j] == length;
                            count += __popcll(ballot(same));
                            tokens += same ? ss[j] : 0;
                            os[j] = same ? 0 : os[j];
                        }
                        const bool all = count == g && shift == 0;  // (then what was taken tells)
                        e.enter(all ? taken - g * min(length, a) : lane_of(lanes_prefix(tokens), WAVE - 1), count, length);
                        left -= count;
                    }
                    first = to;
                    if (first == cnt) break;
                    // the next one is placed alone
                    patience = g >= 4 ? 0 : fresh ? min(2 * patience + 1, MOST_PATIENCE) : patience;
                    look = fresh ? max(patience, 1) : 1;
                }
                // one request
                const int s1 = pick(s, first), o1 = pick(o, first);
                const int bound = (int)((unsigned)e.b + (unsigned)(s1 - M));
                const int least = max(e.c - o1 + 1, min(e.c, bound));  // the start that the lane's completion asks for if it is in the way
                known = false;
                --look;
                const int before = e.t;
                for (;;) {
                    const int late = (int)((unsigned)bound - (unsigned)(e.n + 1) * (unsigned)beyond(e.c, e.t + o1));
                    const int ask = min(late, least) > e.t ? least : 0;
                    if (ballot(ask > e.t) == 0) break;
                    e.t = lanes_max(ask);
                }
                if (e.t != before) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) done[j] = 4 * lane + j >= first ? e.t + o[j] : done[j];
                    look = patience <= PATIENT ? 0 : look;
                }
                e.enter(s1, 1, o1);
                if (++first == cnt) break;
            }
            if (e.full) break;
            unsigned sum = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) sum += cnt == GROUP || 4 * lane + j < cnt ? (unsigned)done[j] : 0u;
            tel += sum;
            *(four *)&kept_s[GROUP * q + 4 * lane] = done;
        }
        if (e.full || bad_length) break;
        wave_sync();
        if (crow) {
            // what the next chunk takes has arrived before the stores are issued
#pragma unroll
            for (int q = 0; q < PIECES; ++q) asm volatile("" : "+v"(sv[q]), "+v"(ov[q]), "+v"(id_next[q]));
#pragma unroll
            for (int q = 0; q < PIECES; ++q) {
                const int k = chunk + WAVE * q + lane;
                if (k < n) crow[kept_id[WAVE * q + lane]] = kept_s[WAVE * q + lane];
            }
            wave_sync();
        }
    }
    if (p.todo && lane == 0) p.todo[cand] = e.full;
    if (e.full) return;
    if (bad_length) {  // (the ids behind have not all been looked at)
        for (int k = lane; k < n; k += WAVE) meet(row[k]);
    }
    wave_sync();
    // n ids that there are set n bits exactly if none is there twice
    bool missing = false;
    for (int w = lane; w < words; w += WAVE) missing |= met[w] != (32 * w + 32 <= n ? ~0u : (1u << (n & 31)) - 1u);
    const bool is_order = (ballot(strange) | ballot(missing)) == 0;
    for (int d = 32; d > 0; d >>= 1) tel += __shfl_down(tel, d);
    if (lane == 0) {
        p.tel_out[cand] = is_order && !bad_length ? tel : -1;
        if (!is_order) atomicOr(&p.d_words[p.status_word], KVSCHED_DEV_BAD_ORDER);
    }
    if (!is_order && crow)  // (requests that do not occur)
        for (int k = lane; k < n; k += WAVE)
            if (((met[k >> 5] >> (k & 31)) & 1u) == 0) crow[k] = -1;
}

}  // namespace

// p.tel_out and p.completion_out (by request id) of the rows whose requests complete in few enough different rounds, checked;
// p.todo[c] = 1 for the others (without p.todo, n <= 64: every row).  n <= KVS_EVENTS_MAX_N.
int kvs_launch_event_rows(const SimParams &p, hipStream_t st)
{
    hipLaunchKernelGGL(event_rows_kernel, dim3((unsigned)p.C), dim3(WAVE), sizeof(int32_t) * (((size_t)p.n + 31) >> 5), st, p);
    return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}
