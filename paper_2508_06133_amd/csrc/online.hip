// Scheduling under online arrivals (Section 6, "Heuristics under Online Arrival"; Section 7,
// "Experiment under Online Poisson Arrivals"): many independent request streams at once, ONE
// 64-lane WAVEFRONT PER STREAM, the whole policy on the device.
//
// Per stream, iteration t = 0, 1, 2, ...:
//   1. requests with a_i <= t join the backlog and the end of the cached priority list;
//   2. when a refresh is due the planner re-orders the whole backlog into a new cached list;
//   3. list entries are admitted from the front while Eq. (1) holds beside the running requests,
//      stopping at the first that does not fit.
// Iterations that cannot change anything are not executed one by one: with an empty backlog the
// stream moves to the next arrival, and when the head of the list does not fit, to the earliest of
// the first round at which it might, the next arrival and the next refresh that could change the
// list (refreshes of an unchanged backlog reproduce the list and are only counted).
//
// A stream is a chain of small dependent steps (a whole plan in the paper's setting is some
// twenty batches and a hundred exchanges on fifty requests), so nothing is gained by putting
// more lanes on one stream; the chip is filled by running thousands of streams side by side.
// One wavefront per stream needs no workgroup barrier anywhere: every decision is a ballot or a
// wave reduction, and the LDS a stream needs (24 KB in the smallest size class) lets six
// streams share a compute unit.
//
// State of a stream, all in LDS:
//   * the backlog as an array of 64-bit keys sorted in the planner's order; a key packs
//     (s+o, o, id) so that sorting, the fallback order and the lengths needed at admission all
//     come from the one word.  Arrivals are merged in (rank among the newcomers + binary search
//     in the backlog), admitted requests are struck out by a compaction; two copies alternate;
//   * the cached list: a circular buffer of the same keys;
//   * the running requests' future memory P(tau) for the next H rounds in a ring of H slots
//     (H = power of two >= longest decode length; the slot of round t is cleared at iteration t
//     before anything is admitted, so it can stand for round t + H); an attempt checks its o rounds 64 at
//     a time and ends in one ballot;
//   * the look-ahead window of the Sorted-F-Online planner: Phase 1 of Algorithm 1 with Local
//     Swap Search batches, sorted place 64 r + lane in row r of the lane's registers (greedy fill
//     = longest prefix by a saturating wave scan; an exchange step = each member's first partner from a
//     mask of who has less o, or, beyond 64 requests, the records of the prefix minimum of o over non-members
//     against all members at once).
#include "kvsched_internal.h"
#include "lane_mask.h"
#include "phase1_util.h"

#include <limits.h>

namespace {

typedef unsigned long long u64;

constexpr int OMAXW = KVSCHED_ONLINE_MAX_WINDOW;
constexpr int OMAXCOUNT = 1 << 20;  // ids are 20-bit fields of the keys

template <int QCAP, int HCAP>
struct StreamLds {
    static constexpr int WCAP = QCAP < OMAXW ? QCAP : OMAXW;
    u64 qa[QCAP];
    u64 qb[QCAP];
    u64 list[QCAP];
    u64 wk[WCAP];  // the planner's window, compacted after every batch
    int ring[HCAP];
    unsigned dead[QCAP / 32];
};

// (s+o, o, id) <-> key.  Fields: s+o < 2^30 (30 bits), o <= 2^13 (14 bits), id < 2^20; the planner's
// sort order decides which field is most significant.
struct Codec {
    int w_shift, o_shift, id_shift;
    __device__ explicit Codec(int planner)
    {
        if (planner == KVSCHED_PLANNER_ARRIVAL) { id_shift = 44; w_shift = 14; o_shift = 0; }        // (id)
        else if (planner == KVSCHED_PLANNER_SHORTEST_DECODE) { o_shift = 50; id_shift = 30; w_shift = 0; }  // (o, id)
        else { w_shift = 34; o_shift = 20; id_shift = 0; }                                           // (s+o, o, id)
    }
    __device__ __forceinline__ u64 make(int w, int o, int id) const
    {
        return ((u64)w << w_shift) | ((u64)o << o_shift) | ((u64)id << id_shift);
    }
    __device__ __forceinline__ int size(u64 k) const { return (int)((k >> w_shift) & 0x3fffffffu); }
    __device__ __forceinline__ int decode(u64 k) const { return (int)((k >> o_shift) & 0x3fffu); }
    __device__ __forceinline__ int id(u64 k) const { return (int)((k >> id_shift) & 0xfffffu); }
};

// ------------------------------------------------------------------ wavefront primitives
// All 64 lanes are active wherever these are called (control flow is uniform per stream).

__device__ __forceinline__ void wave_sync()
{
    // LDS traffic of one wavefront is served in order; this keeps the compiler from moving
    // accesses across a point where lanes read what other lanes wrote
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ u64 uni64(u64 v)
{
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32));
    return ((u64)hi << 32) | lo;
}

__device__ __forceinline__ u64 lane_u64(u64 v, int lane)  // lane is uniform
{
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), lane);
    return ((u64)hi << 32) | lo;
}

// DPP moves: lanes whose source lies outside the pattern (or whose row is masked off) get `idle`.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ int dpp(int idle, int v)
{
    return __builtin_amdgcn_update_dpp(idle, v, CTRL, ROW_MASK, 0xf, false);
}
constexpr int DPP_QUAD_1032 = 0xB1, DPP_QUAD_2301 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140;
constexpr int DPP_ROW_SHR1 = 0x111, DPP_ROW_SHR2 = 0x112, DPP_ROW_SHR4 = 0x114, DPP_ROW_SHR8 = 0x118;
constexpr int DPP_BCAST15 = 0x142, DPP_BCAST31 = 0x143;  // last lane of a row -> the next row(s)
constexpr int DPP_WAVE_SHR1 = 0x138;                      // every lane from the lane below, across rows

// (lanes that receive nothing take the operation's neutral value, which lets the exchange be part of the operation)
__device__ __forceinline__ int wave_min(int v)
{
    v = min(v, dpp<DPP_QUAD_1032>(INT_MAX, v));
    v = min(v, dpp<DPP_QUAD_2301>(INT_MAX, v));
    v = min(v, dpp<DPP_HALF_MIRROR>(INT_MAX, v));
    v = min(v, dpp<DPP_MIRROR>(INT_MAX, v));
    v = min(v, dpp<DPP_BCAST15, 0xa>(INT_MAX, v));
    v = min(v, dpp<DPP_BCAST31, 0xc>(INT_MAX, v));
    return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ long long wave_sum64(long long v)
{
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
    return (long long)uni64((u64)v);
}

__device__ __forceinline__ int wave_max(int v)
{
    v = max(v, dpp<DPP_QUAD_1032>(INT_MIN, v));
    v = max(v, dpp<DPP_QUAD_2301>(INT_MIN, v));
    v = max(v, dpp<DPP_HALF_MIRROR>(INT_MIN, v));
    v = max(v, dpp<DPP_MIRROR>(INT_MIN, v));
    v = max(v, dpp<DPP_BCAST15, 0xa>(INT_MIN, v));
    v = max(v, dpp<DPP_BCAST31, 0xc>(INT_MIN, v));
    return __builtin_amdgcn_readlane(v, 63);
}

// Inclusive prefix scans over the 64 lanes: within rows by shifts of 1, 2, 4, 8, then the last
// lane of row 0 / 2 into rows 1 / 3 and the last lane of row 1 into rows 2 and 3.

// sums of non-negative values, saturating at cap (cap <= 2^30)
__device__ __forceinline__ unsigned wave_incl_add_sat(unsigned v, unsigned cap)
{
    v = min(v + (unsigned)dpp<DPP_ROW_SHR1>(0, (int)v), cap);
    v = min(v + (unsigned)dpp<DPP_ROW_SHR2>(0, (int)v), cap);
    v = min(v + (unsigned)dpp<DPP_ROW_SHR4>(0, (int)v), cap);
    v = min(v + (unsigned)dpp<DPP_ROW_SHR8>(0, (int)v), cap);
    v = min(v + (unsigned)dpp<DPP_BCAST15, 0xa>(0, (int)v), cap);
    v = min(v + (unsigned)dpp<DPP_BCAST31, 0xc>(0, (int)v), cap);
    return v;
}

// inclusive prefix minimum
__device__ __forceinline__ int wave_incl_min(int v)
{
    v = min(v, dpp<DPP_ROW_SHR1>(INT_MAX, v));
    v = min(v, dpp<DPP_ROW_SHR2>(INT_MAX, v));
    v = min(v, dpp<DPP_ROW_SHR4>(INT_MAX, v));
    v = min(v, dpp<DPP_ROW_SHR8>(INT_MAX, v));
    v = min(v, dpp<DPP_BCAST15, 0xa>(INT_MAX, v));
    v = min(v, dpp<DPP_BCAST31, 0xc>(INT_MAX, v));
    return v;
}

__device__ __forceinline__ int first_lane(u64 ballot) { return __ffsll((long long)ballot) - 1; }

// number of entries of the ascending array a[0..n) that are < key (n >= 1; the same number of steps in every lane)
__device__ __forceinline__ int lower_bound_u64(const u64 *a, int n, u64 key)
{
    int lo = 0;
    for (int w = 1 << (31 - __builtin_clz(n)); w > 0; w >>= 1) {
        const bool less = lo + w <= n && a[min(lo + w, n) - 1] < key;
        lo = less ? lo + w : lo;
    }
    return lo;
}

__device__ __forceinline__ u64 lanes_from(int first) { return first >= 64 ? 0ull : ~0ull << first; }
__device__ __forceinline__ u64 lanes_upto(int count) { return count >= 64 ? ~0ull : ~(~0ull << count); }  // count >= 0
__device__ __forceinline__ int rank_in(u64 mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0));
}

// ------------------------------------------------- Sorted-F-Online's look-ahead window
//
// The window: backlog keys in (s+o, o, id) order.  Phase 1 of Algorithm 1 with every batch
// chosen by Local Swap Search over these requests alone (budget M): greedy fill in that
// order, then the first improving exchange (members and non-members scanned in the sorted
// order; |X| is fixed, so F falls exactly when o_in < o_out) until none is left; the batch is
// emitted by (o, id) and removed.
//
// The plan is made batch by batch, as far as admission asks for it: a batch depends on what the batches
// before it left over (wk), not on anything that happens meanwhile, and at the next refresh
// all that has not been asked for is planned anew (in the paper's setting twenty to thirty batches, of which
// admission looks at one or two: 600 streams of it, 23.0 -> 4.9 ms).
//
// Mostly the members and all that they could be exchanged for are the window's first 64 requests, a lane each: exchange_in_lanes makes the
// exchanges there from masks of who has less o than whom, and the batch stays in the lanes (`batch`): admission takes one or two
// requests of a batch before the next refresh, so the batch is not sorted but the least (o, id) looked for when it is asked for,
// and wk is closed up when a next batch is.  (The listed grid of 600 streams 1.72 -> 1.45 ms with masks instead of records, below, and
// 1.41 with the batches of windows beyond 64 requests in the lanes too.)
//
// Beyond, all rows of the window take part, from registers alone: the first non-member with a smaller o than a member's is always a
// record, a non-member with less o than every non-member before it, and of some fifty requests four or five
// are, most of which are too large for every member or have more o than any.  A member has a partner iff a record that
// still fits has less o than it, so all members are tested against one record after the other (a prefix minimum in LDS with a binary search per
// member took three times as long).  An exchange on two rows takes 1250 cycles so.
//
// plan_batch chooses the next batch among wk[0..m); it is in the lanes or, removed from wk, in list[0..K).  Returns K.
// bkey: an idle array of >= m keys, an even number.  m <= 64 RMAX.  One and two rows, where the paper's backlogs fit, keep the whole state
// in scalar and vector registers without a test per row.
struct Batch {
    u64 key;     // this lane's request of the window ...
    unsigned o;  // ... and its o while it is in the batch and has not been asked for (else NO_O)
    u64 others;  // the lanes whose requests are not in the batch
    bool here;   // the batch is in the lanes (else in the list)
};
constexpr unsigned NO_O = 0x7fffffffu;

// The batch's next request: least (o, id) of those not asked for yet (there is one).
__device__ __forceinline__ u64 take_next(Batch &b)
{
    const unsigned least = (unsigned)wave_min((int)b.o);
    u64 who = __builtin_amdgcn_ballot_w64(b.o == least);
    if ((who & (who - 1)) != 0) {
        const int id = __builtin_amdgcn_inverse_ballot_w64(who) ? (int)(b.key & 0xfffffu) : INT_MAX;
        who = __builtin_amdgcn_ballot_w64(id == wave_min(id)) & who;
    }
    const int l = first_lane(who) & 63;
    b.o = lane_id() == l ? NO_O : b.o;
    return lane_u64(b.key, l);
}

// Four more bits of a mask, those of lanes B + 3 ... B: does the lane have less o than this one?  (Written out because a scalar that a
// vector instruction has written may be read by one only two instructions later, and so may its mask.)
template <int B>
__device__ __forceinline__ void four_below(unsigned &mask, unsigned o)
{
    unsigned r0, r1, r2, r3;
    u64 m0, m1, m2, m3;
    asm("s_nop 1\n"
        "v_readlane_b32 %1, %9, %10\n"
        "v_readlane_b32 %2, %9, %11\n"
        "v_readlane_b32 %3, %9, %12\n"
        "v_readlane_b32 %4, %9, %13\n"
        "v_cmp_lt_u32 %5, %1, %9\n"
        "v_cmp_lt_u32 %6, %2, %9\n"
        "v_cmp_lt_u32 %7, %3, %9\n"
        "v_cmp_lt_u32 %8, %4, %9\n"
        "v_addc_co_u32 %0, vcc, %0, %0, %5\n"
        "v_addc_co_u32 %0, vcc, %0, %0, %6\n"
        "v_addc_co_u32 %0, vcc, %0, %0, %7\n"
        "v_addc_co_u32 %0, vcc, %0, %0, %8\n"
        : "+&v"(mask), "=&s"(r0), "=&s"(r1), "=&s"(r2), "=&s"(r3), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3)
        : "v"(o), "n"(B + 3), "n"(B + 2), "n"(B + 1), "n"(B)
        : "vcc");
}

// Lanes B + 31 ... B, of which `count` hold a request at most.
template <int B>
__device__ __forceinline__ unsigned below(unsigned o, int count)
{
    unsigned mask = 0;
    if (count > 24) four_below<B + 28>(mask, o), four_below<B + 24>(mask, o);
    if (count > 16) four_below<B + 20>(mask, o), four_below<B + 16>(mask, o);
    if (count > 8) four_below<B + 12>(mask, o), four_below<B + 8>(mask, o);
    four_below<B + 4>(mask, o);
    four_below<B>(mask, o);
    return mask;
}

// The exchanges of a batch among the lanes' requests, as long as no request from w_limit on (the size of the first that `count` lanes do
// not cover) has room: w_most + slack, what the largest member could be exchanged for, tells.  Returns whether none is left.
// Who has less o than whom does not change with an exchange, so each lane keeps that as a mask of 64 bits; its first partner is then the
// lowest bit of it that is no member's, one lane move brings that one's size, and a ballot says which members have a
// partner with room: 300 cycles an exchange, and up to 850 for the masks of a batch.
__device__ __forceinline__ bool exchange_in_lanes(int w, unsigned o, int count, int w_limit, int &slack, int &w_most, u64 &members,
                                                  u64 &others)
{
    const unsigned less_lo = below<0>(o, count), less_hi = count > 32 ? below<32>(o, count - 32) : 0u;
    while (w_most + slack < w_limit) {
        const unsigned lo = less_lo & (unsigned)others, hi = less_hi & (unsigned)(others >> 32);
        // (no bit: all ones, which is no lane)
        const unsigned first_lo = lo != 0 ? (unsigned)__builtin_ctz(lo) : ~0u, first_hi = hi != 0 ? (unsigned)__builtin_ctz(hi) | 32u : ~0u;
        const unsigned partner = min(first_lo, first_hi);
        const int w_in = __builtin_amdgcn_ds_bpermute((int)(partner << 2), w);
        const u64 has = __builtin_amdgcn_ballot_w64(w_in - w <= slack) & __builtin_amdgcn_ballot_w64((lo | hi) != 0) & members;
        if (has == 0) return true;
        const int a = __builtin_ctzll(has);
        const int b = __builtin_amdgcn_readlane((int)partner, a), w_b = __builtin_amdgcn_readlane(w_in, a);
        slack -= w_b - __builtin_amdgcn_readlane(w, a);
        w_most = max(w_most, w_b);
        const u64 both = 1ull << a | 1ull << b;
        members ^= both;
        others ^= both;
    }
    return false;
}

// The batch (members: v with the sign bit) goes to list[0..), in nondecreasing (o, id), and out of wk[0..m); returns its size.
template <int RMAX>
__device__ __forceinline__ int emit_batch(u64 *wk, int m, int R, const unsigned (&v)[RMAX], u64 *bkey, u64 *list)
{
    constexpr u64 LOW34 = (1ull << 34) - 1;  // (o, id) of a key
    constexpr unsigned IN = 0x80000000u, NONE = 0x7fffffffu;
    const int lane = lane_id();
    // the batch in nondecreasing o, ties by id: rank of each member among the members
    int nmem = 0;
#pragma unroll
    for (int r = 0; r < RMAX; ++r) {
        if (r < R) {
            const u64 bal = __builtin_amdgcn_ballot_w64(v[r] >= IN);
            put_b64(bal, bkey + nmem + rank_in(bal), wk[min(64 * r + lane, m - 1)]);
            nmem += __popcll(bal);
        }
    }
    if (nmem & 1) put_b64(1, bkey + nmem, ~0ull);  // (the loop below takes them two by two)
    wave_sync();
    for (int i0 = 0; i0 < nmem; i0 += 64) {
        const u64 mine = bkey[min(i0 + lane, nmem - 1)];
        const u64 me = mine & LOW34;
        int rank = 0;
#pragma unroll 4
        for (int j = 0; j < nmem; j += 2) rank += ((bkey[j] & LOW34) < me ? 1 : 0) + ((bkey[j + 1] & LOW34) < me ? 1 : 0);
        put_b64(lanes_upto(nmem - i0), list + rank, mine);
    }
    wave_sync();
    // what remains closes up in place, still sorted: row by row, each row read before it is
    // written, and never written beyond itself
    int kept = 0;
#pragma unroll
    for (int r = 0; r < RMAX; ++r) {
        if (r < R) {
            const u64 k = wk[min(64 * r + lane, m - 1)];
            const u64 bal = __builtin_amdgcn_ballot_w64(v[r] < NONE);
            wave_sync();
            put_b64(bal, wk + kept + rank_in(bal), k);
            kept += __popcll(bal);
            wave_sync();
        }
    }
    return nmem;
}

template <int RMAX>
__device__ __forceinline__ int plan_batch(u64 *wk, int m, int M, u64 *bkey, u64 *list, Batch &batch)
{
    constexpr unsigned IN = 0x80000000u, NONE = 0x7fffffffu;
    constexpr int G = RMAX <= 2 ? 2 : 1;  // records tested at a time: what each waits for overlaps
    const int lane = lane_id();
    const int R = RMAX <= 2 ? RMAX : (m + 63) >> 6;
    // this lane's places 64 r + lane: size, and o with the sign bit set in a member (no place: NONE)
    int w[RMAX];
    unsigned v[RMAX];
#pragma unroll
    for (int r = 0; r < RMAX; ++r) {
        if (r < R) {
            const bool is = 64 * r + lane < m;
            const u64 k = wk[min(64 * r + lane, m - 1)];
            if (r == 0) batch.key = k;
            w[r] = is ? (int)(k >> 34) : 0;
            v[r] = is ? (unsigned)(k >> 20) & 0x3fffu : NONE;
        }
    }
    // greedy fill: sizes ascend, so "add while it fits" is the longest prefix within M
    const unsigned cap = (unsigned)M + 1u;
    unsigned carry = 0;
    int K = 0, slack = M;
    int w_most = 0;       // no member is larger than this, and none has more o than this
    unsigned o_most = 0;
#pragma unroll
    for (int r = 0; r < RMAX; ++r) {
        if (r < R && K == 64 * r) {
            const unsigned incl = min(wave_incl_add_sat((unsigned)w[r], cap) + carry, cap);
            const bool in = v[r] != NONE && incl <= (unsigned)M;
            o_most = max(o_most, in ? v[r] : 0u);
            v[r] |= in ? IN : 0u;
            const int c = __popcll(__builtin_amdgcn_ballot_w64(in));
            K += c;
            if (c > 0) {
                slack = M - __builtin_amdgcn_readlane((int)incl, c - 1);
                w_most = __builtin_amdgcn_readlane(w[r], c - 1);
            }
            carry = (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
        }
    }

    // Mostly members and all that they could be exchanged for lie in the first row.
    if (RMAX == 1 || K <= 64) {
        const unsigned of = v[0] & ~IN;
        u64 members = __builtin_amdgcn_ballot_w64(v[0] >= IN), others = __builtin_amdgcn_ballot_w64(v[0] < NONE);
        const u64 room = __builtin_amdgcn_ballot_w64(w[0] <= w_most + slack);
        const int reach = __popcll(room & (members | others));
        const int behind = RMAX > 1 && m > 64 ? __builtin_amdgcn_readlane(w[RMAX > 1 ? 1 : 0], 0) : INT_MAX;  // the next row's first
        bool none_left = (room & others) == 0 && behind > w_most + slack;  // (no masks where the budget holds all of the window)
        for (int count = max((reach + 7) & ~7, 8); !none_left && count <= 64; count = count < 64 ? 64 : 65)
            none_left = exchange_in_lanes(w[0], of, count, count >= 64 ? behind : count < m ? __builtin_amdgcn_readlane(w[0], count & 63) : INT_MAX,
                                          slack, w_most, members, others);
        if (RMAX == 1 || none_left) {
            batch.o = __builtin_amdgcn_inverse_ballot_w64(members) ? of : NO_O;
            batch.others = others;
            batch.here = true;
            return K;
        }
        v[0] = __builtin_amdgcn_inverse_ballot_w64(members) ? of | IN : of;
        o_most = __builtin_amdgcn_inverse_ballot_w64(members) ? of : 0u;  // (K <= 64: of all members)
    }
    o_most = (unsigned)wave_max((int)o_most);

    for (;;) {  // one exchange per turn; every exchange lowers the batch's sum of o
        u64 records[RMAX];
        int upto[RMAX];
        unsigned least[RMAX];  // least o of a record for which this lane's member has room
#pragma unroll
        for (int r = 0; r < RMAX; ++r) {
            least[r] = ~0u;
            if (r < R) upto[r] = wave_incl_min((int)min(v[r], NONE));
        }
        unsigned low = NONE;  // least o of a non-member in the rows before
#pragma unroll
        for (int r = 0; r < RMAX; ++r) {
            if (r < R) {
                const unsigned before = min(min((unsigned)dpp<DPP_WAVE_SHR1>(INT_MAX, upto[r]), low), o_most);
                records[r] = __builtin_amdgcn_ballot_w64(v[r] < before) & __builtin_amdgcn_ballot_w64(w[r] <= w_most + slack);
                low = min(low, (unsigned)__builtin_amdgcn_readlane(upto[r], 63));
            }
        }
#pragma unroll
        for (int r = 0; r < RMAX; ++r) {
            if (r < R) {
                while (records[r] != 0) {
                    int w_in[G];
                    unsigned o_in[G];
#pragma unroll
                    for (int u = 0; u < G; ++u) {  // (past the last record: lane 63 or the record itself, taken for nothing)
                        const int l = first_lane(records[r]) & 63;
                        const unsigned none = records[r] != 0 ? 0u : ~0u;
                        w_in[u] = __builtin_amdgcn_readlane(w[r], l) - slack;  // members of at least this size have room for it
                        o_in[u] = (unsigned)__builtin_amdgcn_readlane((int)v[r], l) | none;
                        records[r] &= records[r] - 1;
                    }
#pragma unroll
                    for (int u = 0; u < G; ++u) {
#pragma unroll
                        for (int rr = 0; rr < RMAX; ++rr)  // in vector registers: a mask in a scalar one would be waited for
                            if (rr < R) least[rr] = min(least[rr], (unsigned)((w[rr] - w_in[u]) >> 31) | o_in[u]);
                    }
                }
            }
        }
        int ra = -1;
        u64 who = 0;
#pragma unroll
        for (int r = RMAX - 1; r >= 0; --r) {
            if (r < R) {
                const u64 has = __builtin_amdgcn_ballot_w64(v[r] > min(least[r], NONE) + IN);
                ra = has != 0 ? r : ra;
                who = has != 0 ? has : who;
            }
        }
        if (ra < 0) break;
        const int la = first_lane(who) & 63;
        unsigned o_out = 0;
        int w_out = 0;
#pragma unroll
        for (int r = 0; r < RMAX; ++r) {
            if (r < R) {
                const unsigned x = (unsigned)__builtin_amdgcn_readlane((int)v[r], la) & ~IN;
                const int y = __builtin_amdgcn_readlane(w[r], la);
                o_out = r == ra ? x : o_out;
                w_out = r == ra ? y : w_out;
            }
        }
        int rb = -1;  // always found: a record said so
#pragma unroll
        for (int r = RMAX - 1; r >= 0; --r) {
            if (r < R) {
                const u64 bal = __builtin_amdgcn_ballot_w64(v[r] < o_out);
                rb = bal != 0 ? r : rb;
                who = bal != 0 ? bal : who;
            }
        }
        const int lb = first_lane(who) & 63;
        slack += w_out;
        int w_in = 0;
#pragma unroll
        for (int r = 0; r < RMAX; ++r) {
            if (r < R) {
                const int y = __builtin_amdgcn_readlane(w[r], lb);
                w_in = r == rb ? y : w_in;
                v[r] ^= (lane == (r == ra ? la : -1)) != (lane == (r == rb ? lb : -1)) ? IN : 0u;
            }
        }
        slack -= w_in;
        w_most = max(w_most, w_in);
    }

    batch.here = false;
    return emit_batch<RMAX>(wk, m, R, v, bkey, list);
}

// ------------------------------------------------------------------------ the stream kernel

struct OnlineParams {
    int32_t B;
    const int32_t *streams;  // [B][8]
    int32_t N;
    const int32_t *a, *s, *o;
    int32_t M;
    int32_t H;    // ring slots: power of two >= longest decode length
    int32_t cap;  // the caller's bound on the backlog of a stream
    int32_t out_len;
    int32_t *completion_out;
    int64_t *stats_out;  // [B][4]
    int32_t *d_words;
    const int32_t *by_cost;  // [B] stream numbers in ascending order of estimated work, or NULL
};

// A batch takes as long as its longest stream, which should therefore not start last: the streams are
// taken in descending order of a rough measure of their work, requests x 8 for Sorted-F-Online (every
// refresh plans a window by Local Swap Search), requests x 1 for the planners that only sort.
// One workgroup: stable 8-bit radix passes on that measure.
__global__ __launch_bounds__(1024) void online_order_kernel(const int32_t *streams, int32_t B, int32_t *tmp, int32_t *sorted)
{
    __shared__ RadixLds<1024> L;
    __shared__ int sh_max[16];
    auto cost = [streams](int b) {
        const int count = streams[8 * (size_t)b + 1], planner = streams[8 * (size_t)b + 2];
        const int c = min(max(count, 0), 1 << 27);
        return planner == KVSCHED_PLANNER_SORTED_F ? 8 * c : c;
    };
    int mx = 0;
    for (int i = threadIdx.x; i < B; i += 1024) mx = max(mx, cost(i));
    for (int d = 32; d > 0; d >>= 1) mx = max(mx, __shfl_xor(mx, d));
    if ((threadIdx.x & 63) == 0) sh_max[threadIdx.x >> 6] = mx;
    __syncthreads();
    for (int w = 0; w < 16; ++w) mx = max(mx, sh_max[w]);
    const int passes = (bits_of(mx) + 7) / 8;
    int *src = (passes & 1) ? tmp : sorted, *dst = (passes & 1) ? sorted : tmp;  // the last pass lands in `sorted`
    for (int i = threadIdx.x; i < B; i += 1024) src[i] = i;
    __threadfence_block();
    __syncthreads();
    for (int pass = 0; pass < passes; ++pass) {
        radix_pass<1024>(src, dst, B, 8 * pass, cost, L);
        __threadfence_block();
        __syncthreads();
        int *sw = src; src = dst; dst = sw;
    }
}

template <int QCAP, int HCAP>
__global__ __launch_bounds__(64) void online_kernel(OnlineParams p)
{
    typedef StreamLds<QCAP, HCAP> Lds;
    __shared__ Lds L;
    constexpr int QM = QCAP - 1;
    const int lane = lane_id();
    const int b = p.by_cost ? uni(p.by_cost[p.B - 1 - (int)blockIdx.x]) : (int)blockIdx.x;  // most work first
    const int32_t *d = p.streams + 8 * (size_t)b;
    const int begin = uni(d[0]), count = uni(d[1]), planner = uni(d[2]), period = uni(d[3]), window = uni(d[4]);
    const int rnum = uni(d[5]), rden = uni(d[6]), outb = uni(d[7]);
    int64_t *stats = p.stats_out + 4 * (size_t)b;
    const bool bad_desc = begin < 0 || count < 0 || count > OMAXCOUNT || (long long)begin + count > p.N ||
                          planner < 0 || planner > KVSCHED_PLANNER_SORTED_F || period < 1 || window < 0 ||
                          window > OMAXW || rnum < 0 || rden < 0 || outb < 0 ||
                          (long long)outb + count > p.out_len;
    if (bad_desc) {
        if (lane == 0) {
            atomicOr(&p.d_words[KVS_W_STATUS], KVSCHED_DEV_BAD_STREAM);
            stats[0] = stats[1] = stats[2] = stats[3] = -1;
        }
        return;
    }
    if (count == 0) {
        if (lane == 0) stats[0] = stats[1] = stats[2] = stats[3] = 0;
        return;
    }
    const int H = p.H, HM = max(H, 256) - 1, M = p.M;  // (the ring has 256 slots or more)
    const Codec codec(planner);

    for (int i = lane; i <= HM; i += 64) L.ring[i] = 0;
    for (int i = lane; i < QCAP / 32; i += 64) L.dead[i] = 0;
    wave_sync();

    u64 *cur = L.qa, *oth = L.qb;
    int t = 0;
    int q = 0;             // backlog size = entries of the cached list
    int head = 0;          // list entries are list[(head + i) & QM], i < q
    int planned_left = 0;  // leading list entries that were placed by the last refresh
    int known = 0, started = 0;
    int wn = 0, planned = 0;  // window of the last refresh, and how many of its entries are planned ...
    int listed = 0;           // ... and of these in list[0 ... listed); the others are still in `batch`
    int rows = 0;             // lanes of it that hold a request of the window
    Batch batch = {0, NO_O, 0, false};
    int t_plan = 0, backlog_at_plan = 0;
    u64 blocked = ~0ull;   // the last request that did not fit, and a round before which it cannot start
    int blocked_to = 0;
    // What is seldom looked at lives in vector registers, though it is the same in all lanes: there are not scalar registers enough
    // for everything, and the compiler would move others to and fro.
    int zero;
    asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
    long long refreshes = zero, sum_c = zero, sum_a = zero;  // sum_a: this lane's share
    int last_c = zero, max_backlog = zero;
    const int32_t *a = p.a + begin + zero, *s = p.s + begin + zero, *o = p.o + begin + zero;
    int32_t *cout = p.completion_out + outb + zero;
    // the next up to 64 requests, one per lane (arrivals find them without waiting for memory)
    struct { int a, bad; u64 key; } ahead;
    int ahead_at = 0;
    auto read_ahead = [&]() __attribute__((always_inline)) {
        ahead_at = known;
        const int idx = known + lane, at = min(idx, count - 1);
        const int av = a[at], earlier = a[max(at - 1, 0)], sv = s[at], ov = o[at];
        ahead.bad = sv < 1 || ov < 1 || (long long)sv + ov > (long long)M ? KVSCHED_DEV_BAD_LENGTH : 0;
        ahead.bad |= ov > H ? KVSCHED_DEV_O_MAX : 0;
        ahead.bad |= av < 0 || (idx > 0 && earlier > av) ? KVSCHED_DEV_BAD_ARRIVAL : 0;
        ahead.a = idx < count ? av : INT_MAX;
        ahead.key = codec.make(sv + ov, ov, idx);  // (of a request with a fault: not looked at)
    };
    read_ahead();
    int next_a = uni(ahead.a);
    int fault = 0;
    // has the backlog grown since the last refresh so much that the list is due?  (Mostly in 32 bits: q <= 4096.)
    const bool short_ratio = (rnum | rden) < (1 << 18);
    auto grown = [&]() __attribute__((always_inline)) {
        if (short_ratio) return (q - planned_left) * rden >= rnum * backlog_at_plan;
        return (long long)(q - planned_left) * rden >= (long long)rnum * backlog_at_plan;
    };
    const float per_round = 1.0f / (float)period;
    // No admission for H iterations in a row with a backlog is impossible (every running request
    // has left by then and a single request always fits), idle stretches are skipped in one step:
    // the budget below is never reached by well-formed input and bounds the loop otherwise.
    // (An iteration passes a round, and rounds are 32-bit numbers.)
    int budget = (int)min((long long)count * (H + 2) + 16, (long long)INT_MAX);
    t = max(next_a, 0);  // nothing waits before (the ring is empty)

    while (started < count) {
        if (--budget < 0) { fault = KVSCHED_DEV_BAD_STREAM; break; }
        // ---- 1. arrivals, up to 64 at a time
        while (known < count && next_a <= t) {
            const int off = known - ahead_at;  // the newcomers are lanes off ... off + kc - 1 of the requests read ahead
            const u64 newly = __builtin_amdgcn_ballot_w64(ahead.a <= t) & lanes_from(off) & lanes_upto(count - ahead_at);
            const int kc = __popcll(newly);
            if ((__builtin_amdgcn_ballot_w64(ahead.bad != 0) & newly) != 0) {
                int bad = __builtin_amdgcn_inverse_ballot_w64(newly) ? ahead.bad : 0;
                for (int dlt = 32; dlt >= 1; dlt >>= 1) bad |= __shfl_xor(bad, dlt);
                fault = uni(bad);
            }
            if (q + kc > p.cap) fault |= KVSCHED_DEV_BACKLOG;
            if (fault) break;
            put_b64(newly, L.list + ((head + q + lane - off) & QM), ahead.key);  // arrival order
            sum_a += __builtin_amdgcn_inverse_ballot_w64(newly) ? ahead.a : 0;
            if (kc <= 2) {
                // each newcomer moves the entries behind it up by one, the last tile first
                for (int j = 0; j < kc; ++j) {
                    const u64 key = lane_u64(ahead.key, off + j);
                    int at = 0;
                    for (int i0 = (q - 1) & ~63; i0 >= 0; i0 -= 64) {
                        const u64 k = cur[min(i0 + lane, q - 1)];
                        const u64 there = lanes_upto(q - i0);
                        const u64 up = __builtin_amdgcn_ballot_w64(key < k) & there;
                        put_b64(up, cur + i0 + lane + 1, k);
                        if (up != there) {
                            at = i0 + __popcll(there & ~up);
                            break;
                        }
                    }
                    put_b64(1, cur + at, key);
                    ++q;
                }
            } else {
                // merge: a newcomer lands at (entries of the backlog before it) + (newcomers before it);
                // an entry of the backlog moves up by the newcomers before it
                const u64 key = ahead.key;
                int at = 0;
                for (int j = 0; j < kc; ++j) at += (lane_u64(key, off + j) < key) ? 1 : 0;
                for (int i0 = 0; i0 < q; i0 += 64) {
                    const u64 there = lanes_upto(q - i0);
                    const u64 k = cur[min(i0 + lane, q - 1)];
                    int nb = 0;
                    for (int j = 0; j < kc; ++j) {
                        const u64 before = __builtin_amdgcn_ballot_w64(k < lane_u64(key, off + j)) & there;
                        nb += __builtin_amdgcn_inverse_ballot_w64(before) ? 0 : 1;
                        at += lane == off + j ? __popcll(before) : 0;
                    }
                    put_b64(there, oth + i0 + lane + nb, k);
                }
                put_b64(newly, oth + at, key);
                u64 *sw = cur; cur = oth; oth = sw;
                q += kc;
            }
            known += kc;
            next_a = INT_MAX;
            if (known < count) {
                if (known - ahead_at == 64) read_ahead();
                next_a = __builtin_amdgcn_readlane(ahead.a, known - ahead_at);
            }
        }
        if (fault) break;
        max_backlog = max(max_backlog, q);

        // ---- 2. refresh of the cached order
        bool refreshed = false;
        if (q > 0 && (planned_left == 0 || t - t_plan >= period || (rden > 0 && grown()))) {
            wn = planner == KVSCHED_PLANNER_SORTED_F ? min(window, q) : 0;
            planned = listed = 0;
            if (wn > 64)  // (a window of one row is read from the backlog itself, below)
                for (int i0 = 0; i0 < wn; i0 += 64) put_b64(lanes_upto(wn - i0), L.wk + i0 + lane, cur[min(i0 + lane, q - 1)]);
            for (int i0 = wn; i0 < q; i0 += 64) put_b64(lanes_upto(q - i0), L.list + i0 + lane, cur[min(i0 + lane, q - 1)]);
            head = 0;
            planned_left = q;
            t_plan = t;
            backlog_at_plan = q;
            ++refreshes;
            refreshed = true;
        }

        // ---- 3. admission of the longest feasible prefix of the list (the ring's slot of round t is empty)
        int adm = 0;
        u64 taken = 0;  // the request admitted last
        int wait_to = t + 1;  // when the loop stops at a request: a round before which it cannot start
        while (adm < q) {
            // (the window's entries are never wrapped: head counts from the refresh)
            if (head + adm == planned && planned < wn) {
                const int left = wn - planned;
                u64 *from = L.wk;
                if (planned == 0) {
                    if (left <= 64) from = cur;  // (in the iteration of the refresh)
                } else if (batch.here) {  // what the batch has left in the lanes, and the rows behind, close up
                    put_b64(batch.others, L.wk + rank_in(batch.others), batch.key);
                    const int kept = __popcll(batch.others), gone = rows - kept;
                    for (int i0 = rows; i0 < left + gone; i0 += 64) {
                        const u64 k = L.wk[min(i0 + lane, left + gone - 1)];
                        wave_sync();
                        put_b64(lanes_upto(left + gone - i0), L.wk + i0 - gone + lane, k);
                        wave_sync();
                    }
                }
                rows = min(left, 64);
                if (left <= 64) planned += plan_batch<1>(from, left, M, oth, L.list + planned, batch);
                else planned += left <= 128 ? plan_batch<2>(L.wk, left, M, oth, L.list + planned, batch)
                                            : plan_batch<Lds::WCAP / 64>(L.wk, left, M, oth, L.list + planned, batch);
                if (!batch.here) listed = planned;
            }
            u64 key;
            if (head + adm == listed && listed < planned) {
                key = take_next(batch);
                put_b64(1, L.list + listed, key);
                ++listed;
            } else {
                key = uni64(L.list[(head + adm) & QM]);
            }
            if (key == blocked && t < blocked_to) {  // found not to start before then (memory only grows by what is admitted)
                wait_to = blocked_to;
                break;
            }
            const int oo = codec.decode(key), id = codec.id(key);
            const int sr = codec.size(key) - oo;
            // (The rounds last read are written from registers when the request is admitted, mostly all of them: a second
            // reading was a third of an admission, 600 streams 2.56 -> 2.39 ms.)
            // round t + j rules out every start before t + min(excess, j): started later the request is
            // smaller at that round by as much, or no longer overlaps it
            int excess = 0;
            int have[4], *at[4];  // four reads at a time; those of the last ones are kept
            const int peak = sr + lane + 1, limit = oo - lane - 1;
            auto read4 = [&](int from) __attribute__((always_inline)) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    at[u] = L.ring + ((t + lane + 1 + from + 64 * u) & HM);
                    have[u] = *at[u];
                }
            };
            for (int from = 0; from < oo; from += 256) {
                read4(from);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = from + 64 * u;  // (less lane + 1)
                    const int over = min(have[u] + (peak + j) - M, j + lane + 1);
                    excess = max(excess, j <= limit ? over : 0);
                }
            }
            if (__builtin_amdgcn_ballot_w64(excess > 0) != 0) {
                wait_to = t + wave_max(excess);
                blocked = key;
                blocked_to = wait_to;
                break;
            }
            // (all 256 rounds of a turn are written, those behind the last with what they hold: the ring has 256 slots or more)
            for (int from = (oo - 1) & ~255; ; from -= 256, read4(from)) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = from + 64 * u;
                    *at[u] = have[u] + (j <= limit ? peak + j : 0);
                }
                if (from == 0) break;
            }
            put_global(1, cout + id, t + oo);
            sum_c += t + oo;
            last_c = max(last_c, t + oo);
            taken = key;
            ++adm;
        }
        // ---- the admitted requests leave the backlog
        if (adm > 0) {
            if (adm < q) {
                if (adm == 1) {
                    for (int i0 = 0; i0 < q; i0 += 64) {
                        const u64 k = cur[min(i0 + lane, q - 1)];
                        put_b64(__builtin_amdgcn_ballot_w64(taken < k) & lanes_upto(q - i0), cur + i0 + lane - 1, k);
                    }
                } else if (adm <= 8) {  // (in place: an entry moves down by as many as went before it)
                    const u64 gone = L.list[(head + min(lane, adm - 1)) & QM];
                    for (int i0 = 0; i0 < q; i0 += 64) {
                        const u64 k = cur[min(i0 + lane, q - 1)];
                        u64 stay = lanes_upto(q - i0);
                        int before = 0;
                        for (int j = 0; j < adm; ++j) {
                            const u64 g = lane_u64(gone, j);
                            before += g < k ? 1 : 0;
                            stay &= ~__builtin_amdgcn_ballot_w64(k == g);
                        }
                        put_b64(stay, cur + i0 + lane - before, k);
                    }
                } else {
                    for (int j0 = 0; j0 < adm; j0 += 64) {
                        const u64 g = L.list[(head + min(j0 + lane, adm - 1)) & QM];
                        const int pos = lower_bound_u64(cur, q, g);
                        or_b32(lanes_upto(adm - j0), L.dead + (pos >> 5), 1u << (pos & 31));
                    }
                    int kept = 0;
                    for (int i0 = 0; i0 < q; i0 += 64) {
                        const int i = min(i0 + lane, q - 1);
                        const u64 k = cur[i];
                        const u64 stay = __builtin_amdgcn_ballot_w64(((L.dead[i >> 5] >> (i & 31)) & 1u) == 0) & lanes_upto(q - i0);
                        put_b64(stay, cur + kept + rank_in(stay), k);
                        kept += __popcll(stay);
                    }
                    for (int i0 = 0; i0 < QCAP / 32; i0 += 64) put_b32(lanes_upto(QCAP / 32 - i0), L.dead + i0 + lane, 0);
                }
            }
            head = (head + adm) & QM;
            q -= adm;
            started += adm;
            planned_left = max(planned_left - adm, 0);
        }
        // ---- the rounds at which nothing can happen are passed in one step.  Until the request at
        // the head of the list can start (wait_to at the earliest), an iteration changes something
        // only if requests arrive or the list is re-planned.  Re-planning an unchanged backlog gives
        // the same list, so where the list is the plan of the present backlog (a refresh in this
        // iteration, and nothing admitted since unless the planner is a plain sort) the refreshes
        // of the rounds passed are only counted; otherwise the step ends at the next refresh due.
        int t_next = t + 1;
        if (q > 0) {
            t_next = min(wait_to, next_a);
            bool quiet = short_ratio;
            if (refreshed && (wn == 0 || adm == 0)) {
                const bool each = rden > 0 && rnum == 0;
                const int rounds = t_next - 1 - t;  // (fewer than 2^14: wait_to lies within the ring)
                if (rounds >= (each ? 1 : period)) {
                    int passed = rounds;
                    if (!each) {  // rounds / period, the quotient in fp32 off by one at most
                        passed = uni((int)((float)rounds * per_round));
                        passed += (passed + 1) * period <= rounds ? 1 : 0;
                        passed -= passed * period > rounds ? 1 : 0;
                    }
                    refreshes += passed;
                    t_plan = t + passed * (each ? 1 : period);
                    backlog_at_plan = q;
                }
                quiet = quiet && !each;
            } else if (planned_left == 0 || (rden > 0 && grown())) {
                t_next = t + 1;
                quiet = false;
            } else {
                t_next = (int)min((long long)t_next, max((long long)t + 1, (long long)t_plan + period));
            }
            // Nor does an arrival change anything but the backlog and the list's end, until the one that makes the backlog grown
            // enough for a refresh: arrivals before it wait for the next iteration there is (as far as they have been read).  600
            // streams 2.10 -> 1.90 ms.
            if (quiet && t_next == next_a && __builtin_amdgcn_ballot_w64(ahead.bad != 0) == 0) {
                const int off = known - ahead_at;
                const u64 enough = rden > 0 ? __builtin_amdgcn_ballot_w64((q - planned_left + lane - off + 1) * rden >= rnum * backlog_at_plan) & lanes_from(off) : 0;
                const int last = min(count - 1 - ahead_at, 63);  // (read so far; behind the last request of all none arrives)
                const int l = min(enough != 0 ? first_lane(enough) : 64, last);
                int grows = __builtin_amdgcn_readlane(ahead.a, l);
                if (enough == 0 && ahead_at + last == count - 1) grows = INT_MAX;
                t_next = (int)min((long long)min(wait_to, grows), max((long long)t + 1, (long long)t_plan + period));
            }
        } else if (known < count) {
            t_next = max(t_next, next_a);  // nothing waits: on to the next arrival
        }
        // the rounds up to t_next are behind every check from now on: their slots stand for the rounds H later
        const int span = min(t_next - t, H);
        for (int i0 = 1; i0 <= span; i0 += 64) put_b32(lanes_upto(span + 1 - i0), L.ring + ((t + i0 + lane) & HM), 0);
        t = t_next;
    }

    const long long sa = wave_sum64(sum_a);
    if (lane == 0) {
        if (fault) {
            atomicOr(&p.d_words[KVS_W_STATUS], fault);
            stats[0] = stats[1] = stats[2] = stats[3] = -1;
        } else {
            stats[0] = sum_c - sa;
            stats[1] = refreshes;
            stats[2] = last_c;
            stats[3] = max_backlog;
        }
    }
}

template <int QCAP, int HCAP>
int launch_online(const OnlineParams &p, hipStream_t st)
{
    hipLaunchKernelGGL((online_kernel<QCAP, HCAP>), dim3((unsigned)p.B), dim3(64), 0, st, p);
    return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}

}  // namespace

// Size classes (backlog capacity, ring slots) and the LDS a stream takes in each: 24 KB, 48 KB,
// 136 KB; the smallest that holds the caller's backlog bound and the longest decode is used.
int kvs_launch_online(int32_t B, const int32_t *streams, int32_t N, const int32_t *a, const int32_t *s,
                      const int32_t *o, int32_t M, int32_t backlog_cap, int32_t ring_slots, int32_t *completion_out,
                      int32_t out_len, int64_t *stats_out, int32_t *order_scratch, int32_t *d_words, hipStream_t st)
{
    if (ring_slots < 2 || (ring_slots & (ring_slots - 1)) || backlog_cap < 1) return KVSCHED_ERANGE;
    OnlineParams p;
    p.by_cost = nullptr;
    if (order_scratch) {  // [2 B]: the order, and the other buffer of the sort
        hipLaunchKernelGGL(online_order_kernel, dim3(1), dim3(1024), 0, st, streams, B, order_scratch + B, order_scratch);
        if (hipGetLastError() != hipSuccess) return KVSCHED_EHIP;
        p.by_cost = order_scratch;
    }
    p.B = B;
    p.streams = streams;
    p.N = N;
    p.a = a;
    p.s = s;
    p.o = o;
    p.M = M;
    p.H = ring_slots;
    p.cap = backlog_cap;
    p.out_len = out_len;
    p.completion_out = completion_out;
    p.stats_out = stats_out;
    p.d_words = d_words;
    if (backlog_cap <= 512 && ring_slots <= 2048) return launch_online<512, 2048>(p, st);
    if (backlog_cap <= 1024 && ring_slots <= 4096) return launch_online<1024, 4096>(p, st);
    if (backlog_cap <= KVSCHED_ONLINE_MAX_BACKLOG && ring_slots <= KVSCHED_ONLINE_MAX_O)
        return launch_online<KVSCHED_ONLINE_MAX_BACKLOG, KVSCHED_ONLINE_MAX_O>(p, st);
    return KVSCHED_ERANGE;
}
