// Phase 1 of Algorithm 1 ("Batch Construction") with every batch chosen by Local Swap Search
// (the appendix algorithm of that name): fill greedily in ascending s+o, then repeat the first
// improving single exchange (r_out in X, r_in not in X) that keeps sum(s+o) <= M, scanning
// members and non-members in the sorted order (s+o, o, id).
//
// An exchange keeps |X|, so it lowers F = sum o / |X|^2 exactly when o_in < o_out.  With the
// remaining requests in sorted order (w = s+o ascending) and slack = M - mem, r_in fits against
// r_out iff w_in <= w_out + slack, i.e. iff r_in lies before ub(out) = first place with
// w > w_out + slack.  Hence, with pm[j] = least o among the non-members before place j,
//     r_out has an improving partner   <=>   pm[ub(out)] < o_out,
// the pair the double scan meets first is the first such member, and its partner is the first
// non-member with o < o_out (it lies before ub(out) because one such non-member does).
// One step = one exclusive prefix-minimum scan, one ub() per member, two block-wide reductions.
//
// The step is a chain of dependent wave operations and barriers, so the whole construction runs in
// ONE small workgroup (LS_T threads = one wavefront per SIMD of a compute unit: with more waves the
// instructions every wave repeats share the issue ports and the step gets slower), each thread
// owning LS_E consecutive places of a tile and keeping its places of the first tile in registers.
// Once at most LS_CAP requests remain the working set lives in LDS, and while the sizes stay below
// LS_TABLE ub() is one read of a table rank[v] = number of remaining requests with w <= v (the
// arrangement is fixed within a batch, so the table is built once per batch); otherwise ub() is a
// binary search.
//
// Up to LSR_N - 1 requests of sizes below LS_TABLE (the second half of this file) the values are
// replaced by their ranks beforehand, by a kernel over the whole chip, so that a whole backlog fits in
// LDS, and the exchanges of a batch are made by a single wavefront where its places are few.
#include "phase1_util.h"
#include "sort_util.h"

namespace {

constexpr int LS_T = 256;                // threads of the workgroup
constexpr int LS_E = 4;                  // consecutive places per thread in a tile
constexpr int LS_TILE = LS_T * LS_E;
constexpr int LS_NW = LS_T / 64;
constexpr int LS_CAP = 10240;            // remaining requests held in LDS (3 x 40 KB + the 32 KB table)
constexpr int LS_TABLE = 16384;          // sizes covered by the rank table
constexpr int LS_SMALL_VALUE = 1 << 15;  // values (o, or a s + b o) the straight-line steps can carry
constexpr int LS_INF = 0x7fffffff;
constexpr unsigned LS_MEMBER = 0x80000000u;  // membership flag kept in the sign bit of the o entry
constexpr int LS_NONE = 0x7fffffff;
constexpr unsigned long long LS_NO_KEY = ~0ull;

typedef __attribute__((address_space(3))) int lds_int;
typedef __attribute__((address_space(3))) const unsigned short lds_rank;

// LDS words read and written at other widths than they are declared with
typedef unsigned __attribute__((may_alias)) any_u32;
typedef unsigned short __attribute__((may_alias)) any_u16;
typedef unsigned any_u32x2 __attribute__((ext_vector_type(2), may_alias));
typedef unsigned any_u32x4 __attribute__((ext_vector_type(4), may_alias));

struct SwapLds {
    int wave_min[LS_NW];
    unsigned long long first_out[2];  // alternating slots: (place << 32 | o) of the first member that has a partner
    unsigned first_key[2];            // the same as place << 15 | o (small case)
    int first_in[2][4];               //                    {place, o, w} of that partner
    long long scan_w[LS_NW];
    long long scan_o[LS_NW];
    int scan_c[LS_NW];
    long long fill_mem, fill_S;
};

struct WorkLds {
    int w[LS_CAP];
    int o[LS_CAP];
    int pm[LS_CAP + LS_E];  // LS_CAP is a multiple of the tile: whole-tile stores of a tile that holds place m - 1 < LS_CAP stay inside
    unsigned short rank[LS_TABLE];
};

union PhaseLds {
    RadixLds<LS_T> radix;
    WorkLds work;
};

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_else(int keep, int v)
{
    return __builtin_amdgcn_update_dpp(keep, v, CTRL, ROW_MASK, 0xf, false);
}

// inclusive prefix minimum (MAX: maximum of non-negative values) over the 64 lanes, all active
template <bool MAX>
__device__ __forceinline__ int wave_scan(int v)
{
    constexpr int ID = MAX ? 0 : LS_INF;
    auto op = [](int x, int y) { return MAX ? max(x, y) : min(x, y); };
    v = op(v, dpp_else<0x111, 0xf>(ID, v));  // row_shr:1
    v = op(v, dpp_else<0x112, 0xf>(ID, v));  // row_shr:2
    v = op(v, dpp_else<0x114, 0xf>(ID, v));  // row_shr:4
    v = op(v, dpp_else<0x118, 0xf>(ID, v));  // row_shr:8
    v = op(v, dpp_else<0x142, 0xa>(ID, v));  // row_bcast15 into rows 1 and 3
    v = op(v, dpp_else<0x143, 0xc>(ID, v));  // row_bcast31 into rows 2 and 3
    return v;
}

// the value of the lane below (the identity in lane 0)
template <bool MAX>
__device__ __forceinline__ int wave_prev(int v)
{
    return dpp_else<0x138, 0xf>(MAX ? 0 : LS_INF, v);  // wave_shr:1
}

// first place in [lo, hi) whose w exceeds lim (hi if none); W ascending
template <class IntPtr>
__device__ __forceinline__ int upper_bound_w(IntPtr W, int lo, int hi, int lim)
{
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (W[mid] <= lim) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Greedy fill over W[0..m): the longest prefix with sum of w <= M.  Marks it in O, returns its
// length K; mem and S receive its sums.  (Sizes ascend, so nothing after the first request that
// does not fit can fit either: the fill of the algorithm is this prefix.)
__device__ int greedy_fill(const int *W, int *O, int m, int M, long long &mem, long long &S, SwapLds &L)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) { L.fill_mem = 0; L.fill_S = 0; }
    long long carry_w = 0, carry_o = 0;
    int K = 0;
    for (int tile = 0; tile < m; tile += LS_T) {
        const int i = tile + tid;
        const int ov = i < m ? O[i] : 0;
        long long w = i < m ? (long long)W[i] : 0, q = ov;
        for (int d = 1; d < 64; d <<= 1) {
            const long long uw = __shfl_up(w, d), uq = __shfl_up(q, d);
            if (lane >= d) { w += uw; q += uq; }
        }
        if (lane == 63) { L.scan_w[wave] = w; L.scan_o[wave] = q; }
        __syncthreads();
        long long off_w = carry_w, off_o = carry_o, tot_w = carry_w, tot_o = carry_o;
        for (int v = 0; v < LS_NW; ++v) {
            const long long xw = L.scan_w[v], xo = L.scan_o[v];
            if (v < wave) { off_w += xw; off_o += xo; }
            tot_w += xw;
            tot_o += xo;
        }
        const long long pre = w + off_w;
        const bool fit = i < m && pre <= (long long)M;
        if (fit) {
            O[i] = (int)((unsigned)ov | LS_MEMBER);
            if (i + 1 >= m || pre + (long long)W[i + 1] > (long long)M) {  // the last one that fits
                L.fill_mem = pre;
                L.fill_S = q + off_o;
            }
        }
        const int c = __syncthreads_count(fit);
        K += c;
        carry_w = tot_w;
        carry_o = tot_o;
        if (c < LS_T) break;  // uniform: c is the same in every thread
    }
    __syncthreads();
    mem = L.fill_mem;
    S = L.fill_S;
    return K;
}

// rank[v] = number of the m sorted entries with w <= v, for v = 0..W[m-1] < LS_TABLE:
// boundaries of the runs of equal w are scattered into a zeroed table, then a running maximum
// fills the gaps (each thread owns a contiguous chunk, chunk totals scanned across the block).
__device__ void build_rank(const int *W, int m, unsigned short *rank, SwapLds &L)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int w_last = W[m - 1];
    for (int v = tid; v <= w_last; v += LS_T) rank[v] = 0;
    __syncthreads();
    for (int j = tid; j < m; j += LS_T) {
        const int wj = W[j];
        if (j + 1 == m || W[j + 1] != wj) rank[wj] = (unsigned short)(j + 1);
    }
    __syncthreads();
    const int chunk = (w_last + LS_T) / LS_T;
    const int lo = tid * chunk, hi = min(lo + chunk, w_last + 1);
    int run = 0;
    for (int v = lo; v < hi; ++v) run = max(run, (int)rank[v]);
    const int incl = wave_scan<true>(run);
    if (lane == 63) L.wave_min[wave] = incl;
    int before = wave_prev<true>(incl);
    __syncthreads();
    for (int u = 0; u < LS_NW; ++u)
        if (u < wave) before = max(before, L.wave_min[u]);
    for (int v = lo; v < hi; ++v) {
        before = max(before, (int)rank[v]);
        rank[v] = (unsigned short)before;
    }
    __syncthreads();
}

// One tile of the prefix-minimum scan: ov[e] = entries of places base + tid*LS_E + e (members and
// places past the end count as "none"); pm[e] receives the least o among non-members before each
// place (carry = the same over all earlier tiles, updated) and is stored to PM[base + ...] for
// places <= m.  Two barriers; PM is complete after the second.
template <class IntPtr>
__device__ __forceinline__ void scan_tile(const int (&ov)[LS_E], int (&pm)[LS_E], int &carry, SwapLds &L, IntPtr PM,
                                          int base, int m)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int run = LS_INF;
#pragma unroll
    for (int e = 0; e < LS_E; ++e) {
        pm[e] = run;
        if (ov[e] >= 0) run = min(run, ov[e]);
    }
    const int incl = wave_scan<false>(run);
    if (lane == 63) L.wave_min[wave] = incl;
    int before = wave_prev<false>(incl);
    __syncthreads();
    int total = carry;
    before = min(before, carry);
#pragma unroll
    for (int u = 0; u < LS_NW; ++u) {
        const int x = L.wave_min[u];
        if (u < wave) before = min(before, x);
        total = min(total, x);
    }
#pragma unroll
    for (int e = 0; e < LS_E; ++e) {
        pm[e] = min(pm[e], before);
        const int i = base + (int)threadIdx.x * LS_E + e;
        if (i <= m) PM[i] = pm[e];
    }
    carry = total;
    __syncthreads();
}

// Running state of one batch's exchanges, the same in every thread.
struct SwapState {
    long long mem, S;  // sum of s+o and of o over the members
    int hi;            // every member lies before place hi
    int w_hi;          // no member is larger than this
    int swaps;
};

// The exchanges of one batch, any size.  W, O, PM: m sorted entries (LDS or global memory; PM
// holds m + 1), members flagged in O's sign bit.  rank: table of build_rank or null.
template <class IntPtr, class RankPtr>
__device__ __forceinline__ void swap_loop(IntPtr W, IntPtr O, IntPtr PM, RankPtr rank, int m, int M, SwapState &st,
                                          SwapLds &L)
{
    long long mem = st.mem, S = st.S;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w_last = W[m - 1];
    // number of places whose w is at most lim; needs W[from - 1] <= lim and the answer <= to
    auto ub = [&](int from, int to, int lim) {
        if (rank) return (int)rank[min(lim, w_last)];  // rank[w_last] = m
        return upper_bound_w(W, from, to, lim);
    };
    // this thread's places of the first tile, in registers (LS_INF = a non-member that never helps)
    int own_o[LS_E], own_w[LS_E], own_pm[LS_E];
#pragma unroll
    for (int e = 0; e < LS_E; ++e) {
        const int i = tid * LS_E + e;
        own_o[e] = i < m ? O[i] : LS_INF;
        own_w[e] = i < m ? W[i] : 0;
    }
    if (tid < 2) { L.first_out[tid] = LS_NO_KEY; L.first_in[tid][0] = LS_NONE; }
    __syncthreads();
    int hi = st.hi, swaps = st.swaps, w_hi = st.w_hi;
    for (int it = 0;; ++it) {
        const int slot = it & 1;
        const int slack = (int)((long long)M - mem);
        const int U = ub(hi, m, w_hi + slack);  // places from U on fit against no member

        // ---- pm[j] = least o among non-members before place j, for j = 0..U (entries past U may
        //      be written too; nothing reads them)
        int carry = LS_INF;
        scan_tile(own_o, own_pm, carry, L, PM, 0, m);
        for (int tile = LS_TILE; tile <= U; tile += LS_TILE) {
            int ov[LS_E], pm[LS_E];
#pragma unroll
            for (int e = 0; e < LS_E; ++e) {
                const int i = tile + tid * LS_E + e;
                ov[e] = i < m ? O[i] : LS_INF;
            }
            scan_tile(ov, pm, carry, L, PM, tile, m);
        }

        // ---- first member with an improving partner that fits: per wave the lowest lane of the
        //      first tile that has one; waves combined by a minimum in LDS; the key carries its o
        unsigned long long cand = LS_NO_KEY;
        for (int tile = 0; tile < hi; tile += LS_TILE) {
            unsigned long long mine = LS_NO_KEY;
            int ov[LS_E], wv[LS_E];
#pragma unroll
            for (int e = 0; e < LS_E; ++e) {
                const int a = tile + tid * LS_E + e;
                if (tile == 0) { ov[e] = own_o[e]; wv[e] = own_w[e]; }
                else { ov[e] = a < hi ? O[a] : LS_INF; wv[e] = a < hi ? W[a] : 0; }
            }
            if (rank) {  // loads issued for all places at once; non-members read rank[0] = 0, pm[0] = none
                int j[LS_E], p[LS_E];
#pragma unroll
                for (int e = 0; e < LS_E; ++e) j[e] = rank[ov[e] < 0 ? min(wv[e] + slack, w_last) : 0];
#pragma unroll
                for (int e = 0; e < LS_E; ++e) p[e] = PM[j[e]];
#pragma unroll
                for (int e = LS_E - 1; e >= 0; --e) {
                    const int oo = (int)((unsigned)ov[e] & ~LS_MEMBER);
                    if (ov[e] < 0 && p[e] < oo)
                        mine = ((unsigned long long)(tile + tid * LS_E + e) << 32) | (unsigned)oo;
                }
            } else {
#pragma unroll
                for (int e = LS_E - 1; e >= 0; --e) {
                    const int a = tile + tid * LS_E + e;
                    if (ov[e] < 0) {  // a member
                        const int oo = (int)((unsigned)ov[e] & ~LS_MEMBER);
                        if (PM[upper_bound_w(W, a + 1, U, wv[e] + slack)] < oo)
                            mine = ((unsigned long long)a << 32) | (unsigned)oo;
                    }
                }
            }
            const unsigned long long bal = __builtin_amdgcn_ballot_w64(mine != LS_NO_KEY);
            if (bal != 0 && cand == LS_NO_KEY) {
                const int l = (int)__builtin_ctzll(bal);
                const unsigned lo32 = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)mine, l);
                const unsigned hi32 = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(mine >> 32), l);
                cand = ((unsigned long long)hi32 << 32) | lo32;
            }
        }
        if (lane == 0 && cand != LS_NO_KEY) atomicMin(&L.first_out[slot], cand);
        __syncthreads();
        const unsigned long long key = L.first_out[slot];
        if (key == LS_NO_KEY) break;  // uniform
        const int a_star = (int)(key >> 32), o_a = (int)(unsigned)key;
        const int w_a = W[a_star];

        // ---- its partner: the first non-member with smaller o, i.e. the one place where the
        //      prefix minimum is still >= o_out and the entry itself is below it
        {
            int fb = LS_NONE, fo = 0, fw = 0;
#pragma unroll
            for (int e = 0; e < LS_E; ++e) {
                const bool is = own_o[e] >= 0 && own_o[e] < o_a && own_pm[e] >= o_a;
                fb = is ? tid * LS_E + e : fb;
                fo = is ? own_o[e] : fo;
                fw = is ? own_w[e] : fw;
            }
            if (fb != LS_NONE) {
                L.first_in[slot][0] = fb;
                L.first_in[slot][1] = fo;
                L.first_in[slot][2] = fw;
            }
        }
        for (int tile = LS_TILE; tile < U; tile += LS_TILE) {
#pragma unroll
            for (int e = 0; e < LS_E; ++e) {
                const int b = tile + tid * LS_E + e;
                if (b < U) {
                    const int ov = O[b];
                    if (ov >= 0 && ov < o_a && PM[b] >= o_a) {
                        L.first_in[slot][0] = b;
                        L.first_in[slot][1] = ov;
                        L.first_in[slot][2] = W[b];
                    }
                }
            }
        }
        __syncthreads();
        const int b_star = L.first_in[slot][0], o_b = L.first_in[slot][1], w_b = L.first_in[slot][2];
        if (b_star == LS_NONE) break;  // cannot happen: pm said a partner exists; never spin

        // ---- exchange; every thread keeps the running sums, the owners rewrite the flags
        mem += (long long)w_b - (long long)w_a;
        S += (long long)o_b - (long long)o_a;
        if (b_star >= hi) { hi = b_star + 1; w_hi = w_b; }
        ++swaps;
        const int in_flag = (int)((unsigned)o_b | LS_MEMBER);
        if (((a_star & (LS_TILE - 1)) / LS_E) == tid) O[a_star] = o_a;
        if (((b_star & (LS_TILE - 1)) / LS_E) == tid) O[b_star] = in_flag;
#pragma unroll
        for (int e = 0; e < LS_E; ++e) {
            if (tid * LS_E + e == a_star) own_o[e] = o_a;
            if (tid * LS_E + e == b_star) own_o[e] = in_flag;
        }
        if (tid == 0) {  // the other slot was last read two barriers ago; ready it for the next step
            L.first_out[slot ^ 1] = LS_NO_KEY;
            L.first_in[slot ^ 1][0] = LS_NONE;
        }
    }
    st.mem = mem;
    st.S = S;
    st.hi = hi;
    st.w_hi = w_hi;
    st.swaps = swaps;
}

// The same steps for the common small case, straight-line: working set in LDS, rank table present,
// and every place that matters (U, see above) inside the first tile, so each thread works on the
// LS_E places it keeps in registers and nothing is conditional but the two block-wide decisions.
// Runs until no exchange is left (returns true) or the case no longer applies (returns false with
// st and the flags in O consistent, for swap_loop to continue).
__device__ __forceinline__ bool swap_steps_small(lds_int *W, lds_int *O, lds_int *PM, lds_rank *rank, int m, int M,
                                                 SwapState &st, SwapLds &L)
{
    constexpr unsigned NO_KEY = 0xffffffffu;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int w_last = W[m - 1];
    int own_o[LS_E], own_w[LS_E];
#pragma unroll
    for (int e = 0; e < LS_E; ++e) {
        const int i = tid * LS_E + e;
        own_o[e] = i < m ? O[i] : LS_INF;
        own_w[e] = i < m ? W[i] : 0;
    }
    if (tid < 2) { L.first_key[tid] = NO_KEY; L.first_in[tid][0] = LS_NONE; }
    __syncthreads();
    int slack = (int)((long long)M - st.mem), hi = st.hi, w_hi = st.w_hi, swaps = st.swaps;
    long long S = st.S;
    bool done = false;
    for (int it = 0;; ++it) {
        const int slot = it & 1;
        const int U = rank[min(w_hi + slack, w_last)];
        if (U >= LS_TILE) break;  // uniform

        // ---- prefix minimum of o over the non-members (a member reads as "none": its sign bit
        //      makes it the largest unsigned value)
        int pm[LS_E];
        int run = LS_INF;
#pragma unroll
        for (int e = 0; e < LS_E; ++e) {
            pm[e] = run;
            run = (int)min((unsigned)run, (unsigned)own_o[e]);
        }
        const int incl = wave_scan<false>(run);
        if (lane == 63) L.wave_min[wave] = incl;
        int before = wave_prev<false>(incl);
        __syncthreads();
#pragma unroll
        for (int u = 0; u < LS_NW; ++u) before = u < wave ? min(before, L.wave_min[u]) : before;
#pragma unroll
        for (int e = 0; e < LS_E; ++e) {
            pm[e] = min(pm[e], before);
            PM[tid * LS_E + e] = pm[e];  // the table has room for the whole tile
        }
        __syncthreads();

        // ---- first member with an improving partner that fits; key = place << 15 | o
        unsigned key = NO_KEY;
        {
            int j[LS_E], p[LS_E];
#pragma unroll
            for (int e = 0; e < LS_E; ++e) j[e] = rank[own_o[e] < 0 ? min(own_w[e] + slack, w_last) : 0];
#pragma unroll
            for (int e = 0; e < LS_E; ++e) p[e] = PM[j[e]];
#pragma unroll
            for (int e = LS_E - 1; e >= 0; --e) {
                const int oo = (int)((unsigned)own_o[e] & ~LS_MEMBER);
                key = (own_o[e] < 0 && p[e] < oo) ? (unsigned)(((tid * LS_E + e) << 15) | oo) : key;
            }
        }
        const unsigned long long bal = __builtin_amdgcn_ballot_w64(key != NO_KEY);
        if (bal != 0) {
            const unsigned k = (unsigned)__builtin_amdgcn_readlane((int)key, (int)__builtin_ctzll(bal));
            if (lane == 0) atomicMin(&L.first_key[slot], k);
        }
        __syncthreads();
        const unsigned best = L.first_key[slot];
        if (best == NO_KEY) { done = true; break; }  // uniform
        const int a_star = (int)(best >> 15), o_a = (int)(best & 0x7fffu);
        const int w_a = W[a_star];

        // ---- its partner: the one non-member below o_out whose prefix minimum is not
        {
            int fb = LS_NONE, fo = 0, fw = 0;
#pragma unroll
            for (int e = 0; e < LS_E; ++e) {
                const bool is = (unsigned)own_o[e] < (unsigned)o_a && pm[e] >= o_a;
                fb = is ? tid * LS_E + e : fb;
                fo = is ? own_o[e] : fo;
                fw = is ? own_w[e] : fw;
            }
            if (fb != LS_NONE) {
                L.first_in[slot][0] = fb;
                L.first_in[slot][1] = fo;
                L.first_in[slot][2] = fw;
            }
        }
        __syncthreads();
        const int b_star = L.first_in[slot][0], o_b = L.first_in[slot][1], w_b = L.first_in[slot][2];
        if (b_star == LS_NONE) { done = true; break; }  // cannot happen; never spin

        // ---- exchange
        slack -= w_b - w_a;
        S += (long long)(o_b - o_a);
        if (b_star >= hi) { hi = b_star + 1; w_hi = w_b; }
        ++swaps;
        const int in_flag = (int)((unsigned)o_b | LS_MEMBER);
#pragma unroll
        for (int e = 0; e < LS_E; ++e) {
            own_o[e] = (tid * LS_E + e == a_star) ? o_a : own_o[e];
            own_o[e] = (tid * LS_E + e == b_star) ? in_flag : own_o[e];
        }
        if ((a_star / LS_E) == tid) O[a_star] = o_a;
        if ((b_star / LS_E) == tid) O[b_star] = in_flag;
        if (tid == 0) {  // the other slot was last read two barriers ago; ready it for the next step
            L.first_key[slot ^ 1] = NO_KEY;
            L.first_in[slot ^ 1][0] = LS_NONE;
        }
    }
    st.mem = (long long)M - slack;
    st.S = S;
    st.hi = hi;
    st.w_hi = w_hi;
    st.swaps = swaps;
    return done;
}

__global__ __launch_bounds__(LS_T) void local_swap_kernel(int32_t n, const int32_t *s, const int32_t *o, int32_t M,
                                                          int32_t ga, int32_t gb, int32_t *order_out, int32_t *batch_end_out, double *F_out,
                                                          int32_t *swaps_out, int32_t *num_batches_out, int *gw, int *go,
                                                          int *gid, int *alt_o, int *buf0, int *buf1, int *by_o,
                                                          int *batch_of, int32_t *words, const int *ranked,
                                                          int32_t pad)
{
    __shared__ PhaseLds P;
    __shared__ SwapLds L;
    __shared__ int sh[4];
    if (ranked && *ranked != 0) return;  // done by ranked_swap_kernel
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    // ---- well-formedness and key widths
    int omax = 0, wmax = 0, vmax = 0, bad = 0;
    for (int i = tid; i < n; i += LS_T) {
        const int sv = s[i], ov = o[i];
        const bool ok = sv >= 1 && ov >= 1 && (long long)sv + ov <= (long long)M;
        if (!ok) bad = 1;
        omax = max(omax, ov);
        wmax = max(wmax, (sv < 1 || ov < 1) ? 0 : (int)min((long long)sv + ov, (long long)M));
        vmax = max(vmax, ok ? ga * sv + gb * ov : 0);
    }
    if (tid < 4) sh[tid] = 0;
    __syncthreads();
    if (bad) atomicOr(&sh[2], 1);
    atomicMax(&sh[0], omax);
    atomicMax(&sh[1], wmax);
    atomicMax(&sh[3], vmax);
    __syncthreads();
    omax = sh[0];
    wmax = sh[1];
    vmax = sh[3];  // largest value an exchange compares: o, or the effective length of the G metric
    if (sh[2] != 0) {  // a request that can never run: report, emit no batches
        if (tid == 0) {
            atomicOr(&words[KVS_W_STATUS], KVSCHED_DEV_BAD_LENGTH);
            *num_batches_out = 0;
        }
        if (pad)
            for (int i = tid; i < n; i += LS_T) {
                batch_end_out[i] = 0;
                F_out[i] = 0.0;
                if (swaps_out) swaps_out[i] = 0;
            }
        return;
    }

    // ---- key sorts: ids by (o, id), kept for the emission order, then on by s+o
    for (int i = tid; i < n; i += LS_T) buf0[i] = i;
    __syncthreads();
    int *cur = buf0, *alt = buf1;
    auto key_o = [o](int id) { return o[id]; };
    auto key_w = [s, o](int id) { return s[id] + o[id]; };
    for (int shift = 0; shift < bits_of(omax); shift += 8) {
        radix_pass(cur, alt, n, shift, key_o, P.radix);
        int *t = cur; cur = alt; alt = t;
    }
    for (int i = tid; i < n; i += LS_T) by_o[i] = cur[i];
    __syncthreads();
    for (int shift = 0; shift < bits_of(wmax); shift += 8) {
        radix_pass(cur, alt, n, shift, key_w, P.radix);
        int *t = cur; cur = alt; alt = t;
    }
    for (int i = tid; i < n; i += LS_T) {
        const int id = cur[i];
        gid[i] = id;
        go[i] = ga * s[id] + gb * o[id];  // what an exchange must lower: o, or the effective length of the G metric
        gw[i] = s[id] + o[id];
    }
    __threadfence_block();
    __syncthreads();
    int *alt_w = buf0, *alt_id = buf1;  // the sort buffers are free until the last step

    // ---- batches
    int a = 0, nb = 0;
    while (a < n) {
        const int m = n - a;
        const bool in_lds = m <= LS_CAP;
        const int *W = gw + a;
        int *O = go + a;
        if (in_lds) {
            for (int i = tid; i < m; i += LS_T) {
                P.work.w[i] = gw[a + i];
                P.work.o[i] = go[a + i];
            }
            __syncthreads();
            W = P.work.w;
            O = P.work.o;
        }
        long long mem = 0, S = 0;
        int hi = 0, swaps = 0;
        const int K = greedy_fill(W, O, m, M, mem, S, L);
        if (K < 1) {  // cannot happen for well-formed input; never spin
            if (tid == 0) atomicOr(&words[KVS_W_STATUS], KVSCHED_DEV_BAD_LENGTH);
            break;
        }
        SwapState st;
        st.mem = mem;
        st.S = S;
        st.hi = K;
        st.w_hi = W[K - 1];
        st.swaps = 0;
        if (in_lds) {  // the same loop, compiled for LDS addresses
            lds_rank *rank = nullptr;
            bool done = false;
            if (W[m - 1] < LS_TABLE) {
                build_rank(W, m, P.work.rank, L);
                rank = (lds_rank *)P.work.rank;
                if (vmax < LS_SMALL_VALUE)  // the straight-line steps pack (place, value) into 32 bits
                    done = swap_steps_small((lds_int *)P.work.w, (lds_int *)P.work.o, (lds_int *)P.work.pm, rank, m, M, st, L);
            }
            if (!done) swap_loop((lds_int *)P.work.w, (lds_int *)P.work.o, (lds_int *)P.work.pm, rank, m, M, st, L);
        } else {
            swap_loop(gw + a, go + a, alt_o, (const unsigned short *)nullptr, m, M, st, L);
        }
        S = st.S;
        hi = st.hi;
        swaps = st.swaps;
        __syncthreads();
        if (tid == 0) {
            batch_end_out[nb] = a + K;
            F_out[nb] = (double)S / ((double)gb * (double)K * (double)K);
            if (swaps_out) swaps_out[nb] = swaps;
        }
        // members get the batch number; non-members of [0, hi) close up behind the K removed
        // places (stable), through the spare arrays
        int carry = 0;
        for (int tile = 0; tile < hi; tile += LS_T) {
            const int i = tile + tid;
            int keep = 0, ov = 0;
            if (i < hi) {
                ov = O[i];
                if (ov < 0) batch_of[gid[a + i]] = nb;
                else keep = 1;
            }
            int c = keep;
            for (int d = 1; d < 64; d <<= 1) {
                const int u = __shfl_up(c, d);
                if (lane >= d) c += u;
            }
            if (lane == 63) L.scan_c[wave] = c;
            __syncthreads();
            int off = carry, total = carry;
            for (int u = 0; u < LS_NW; ++u) {
                const int x = L.scan_c[u];
                if (u < wave) off += x;
                total += x;
            }
            if (keep) {
                const int dst = K + off + c - 1;
                alt_w[dst] = W[i];
                alt_o[dst] = ov;
                alt_id[dst] = gid[a + i];
            }
            carry = total;
            __syncthreads();
        }
        __threadfence_block();
        __syncthreads();
        for (int i = K + tid; i < hi; i += LS_T) {
            gw[a + i] = alt_w[i];
            go[a + i] = alt_o[i];
            gid[a + i] = alt_id[i];
        }
        __threadfence_block();
        __syncthreads();
        a += K;
        ++nb;
    }
    if (tid == 0) *num_batches_out = nb;
    if (pad)
        for (int i = nb + tid; i < n; i += LS_T) {
            batch_end_out[i] = 0;
            F_out[i] = 0.0;
            if (swaps_out) swaps_out[i] = 0;
        }
    __threadfence_block();
    __syncthreads();

    // ---- order the (o, id)-sorted ids by batch number (stable): each batch in nondecreasing o
    int *src = by_o, *dst = buf0, *other = buf1;
    auto key_b = [batch_of](int id) { return batch_of[id]; };
    bool first = true;
    for (int shift = 0; shift < bits_of(nb - 1); shift += 8) {
        radix_pass(src, dst, n, shift, key_b, P.radix);
        if (first) { src = dst; dst = other; first = false; }
        else { int *t = src; src = dst; dst = t; }
    }
    for (int i = tid; i < n; i += LS_T) order_out[i] = src[i];
}

// ---------------------------------------------------------------------------------------------
// Fewer than LSR_N requests, all of sizes below LS_TABLE.
//
// Exchanges only compare values, so a value is replaced by the number of requests of smaller values
// (equal ones stay equal).  Then size, value and membership of a request fit in one LDS word, and with
// its rank by (o, id) two bytes more; nothing is read from memory between the batches.
//
// rank_requests_kernel sorts by counting: a request's place in an order is the number of requests
// before it, three counts of n comparisons each, which the whole chip shares (2000 requests: 125
// workgroups; the radix passes that one workgroup made took 95 us).
//
// What a step costs is its chain of dependent operations and, to a lone wavefront, some 7 cycles an instruction.  Up to
// 1024 places it is therefore the work of ONE wavefront, without a barrier: lane l holds places E l ...
// E l + E - 1 of the arrangement in registers, and which of them are members in the bits of one more.  Cycles per
// exchange, 2 / 4 / 8 / 16 places per lane: 700 / 800 / 1050 / 1700 (with a flag put into two of the registers for each exchange, the
// lanes looked up with a case for none, and the last member's place kept up: 4 / 8 / 16 places 880 / 1150 / 1880); by
// eight wavefronts with four barriers, 4 / 16 places per lane: 2100 / 4000 (so 1024 places are the line:
// with 2 places per lane the workgroup takes 2290).  The rest of the workgroup takes part between the exchanges
// (greedy fill, table of ub(), closing up: three microseconds per batch) and writes the batch before out
// during them.
// 2000 mixed requests, 31 batches, 848 exchanges: 460 -> 427 us a call; 8000 chat requests, 8 batches, 1720 exchanges over up to
// 6000 places: 1.99 -> 1.83 ms; 600 mixed ones 217 -> 193.
// A bound for each member on its partner's size instead of the table, kept up with every exchange, is no gain: the exchange takes as many
// instructions, and a fifth to a third of the members that a bound does not rule out have no partner after all (2000 mixed
// requests 506 us; 64 places, a lane each, no difference).

constexpr int LSR_N = 8192;
constexpr int LSR_T = 512;  // threads of the workgroup
constexpr int LSR_NW = LSR_T / 64;
constexpr int LSR_OWN = 16;        // requests ranked by a workgroup
// The word of a place: LSR_IN for a member | value << 18 | size << 4 | (in registers only) number of the register.
// Comparing words compares values, and a member's is larger than any non-member's.
constexpr unsigned LSR_IN = 0x80000000u;
constexpr unsigned LSR_VALUE = 0x7ffc0000u;  // as a word, a place without a request: larger than every value
constexpr unsigned LSR_REST = 0x3ffffu;
__device__ __forceinline__ int size_of(unsigned word) { return (int)(word >> 4) & (LS_TABLE - 1); }
static_assert(LS_TABLE <= 1 << 14 && LSR_N <= 1 << 13, "words of RankedLds");

// What the ranking kernel leaves behind.
struct RankedArrays {
    int *state;            // 1: the arrays hold the ranked requests; 0: a size does not fit; -1: malformed lengths
    unsigned *word;        // [n] by (size, o, id): value rank << 18 | size << 4
    unsigned short *by_w;  // [n] rank by (o, id) of the same requests
    unsigned short *by_o;  // [n] id at a rank by (o, id)
    int *value;            // [n] value of the request at a rank by (o, id)
};

// Each workgroup ranks LSR_OWN requests: lane 16 g + r of wavefront v compares request r with the keys of
// part 4 v + g.  Keys of a quad that lies before the request count when equal, those behind it when
// smaller; the quad that holds the request itself is corrected afterwards.
__global__ __launch_bounds__(1024) void rank_requests_kernel(int32_t n, const int32_t *s, const int32_t *o, int32_t M,
                                                             int32_t ga, int32_t gb, RankedArrays r, int32_t *words,
                                                             int32_t *num_batches_out)
{
    __shared__ __align__(16) unsigned key_w[LSR_N];  // size << 14 | o
    __shared__ __align__(16) unsigned key_v[LSR_N];
    __shared__ unsigned part[16][3][LSR_OWN];
    __shared__ int sh[3];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < 3) sh[tid] = 0;
    __syncthreads();
    int omax = 0, wide = 0, bad = 0;
    for (int j = tid; j < ((n + 3) & ~3); j += 1024) {
        unsigned kw = ~0u, kv = ~0u;  // (padding: below no key, and o < size < 0x3fff)
        if (j < n) {
            const int sv = s[j], ov = o[j];
            if (sv < 1 || ov < 1 || (long long)sv + ov > (long long)M) bad = 1;
            else if (sv + ov >= LS_TABLE) wide = 1;
            omax = max(omax, ov);
            kw = ((unsigned)(sv + ov) << 14) | ((unsigned)ov & 0x3fffu);
            kv = (unsigned)(ga * sv + gb * ov);
        }
        key_w[j] = kw;
        key_v[j] = kv;
    }
    for (int d = 32; d > 0; d >>= 1) omax = max(omax, __shfl_xor(omax, d));
    if (lane == 0) atomicMax(&sh[0], omax);
    if (bad) atomicOr(&sh[1], 1);
    if (wide) atomicOr(&sh[2], 1);
    __syncthreads();
    bad = sh[1];
    wide = sh[2];
    if (blockIdx.x == 0 && tid == 0) {
        words[KVS_W_STATUS] = bad ? KVSCHED_DEV_BAD_LENGTH : 0;
        words[KVS_W_STATUS_AT] = KVS_W_STATUS;
        words[KVS_W_OMAX] = sh[0];
        words[KVS_W_MINPOS] = 0x7fffffff;
        words[KVS_W_MAXPOS] = -1;
        *r.state = bad ? -1 : (wide ? 0 : 1);
        if (bad) *num_batches_out = 0;
    }
    if (bad || wide) return;

    const int i = (int)blockIdx.x * LSR_OWN + (lane & 15);
    const int ii = min(i, n - 1), group = 4 * wave + (lane >> 4);
    const unsigned kw = key_w[ii], kv = key_v[ii], ko = kw & 0x3fffu;
    const int quads = (n + 3) >> 2, per = (quads + 63) >> 6;
    const int q1 = min(quads, (group + 1) * per);
    unsigned cw = 0, co = 0, cv = 0;
    for (int q = group * per; q < q1; ++q) {
        const any_u32x4 a = reinterpret_cast<const any_u32x4 *>(key_w)[q], b = reinterpret_cast<const any_u32x4 *>(key_v)[q];
        const unsigned tie = 4 * q + 3 < ii ? 1u : 0u, tw = kw + tie, to = ko + tie;
        cw += (a.x < tw) + (a.y < tw) + (a.z < tw) + (a.w < tw);
        co += ((a.x & 0x3fffu) < to) + ((a.y & 0x3fffu) < to) + ((a.z & 0x3fffu) < to) + ((a.w & 0x3fffu) < to);
        cv += (b.x < kv) + (b.y < kv) + (b.z < kv) + (b.w < kv);
    }
    if (group == 0) {
        for (int j = ii & ~3; j < ii; ++j) {
            cw += key_w[j] == kw;
            co += (key_w[j] & 0x3fffu) == ko;
        }
    }
    for (int d = 16; d < 64; d <<= 1) {
        cw += __shfl_xor((int)cw, d);
        co += __shfl_xor((int)co, d);
        cv += __shfl_xor((int)cv, d);
    }
    if (lane < LSR_OWN) {
        part[wave][0][lane] = cw;
        part[wave][1][lane] = co;
        part[wave][2][lane] = cv;
    }
    __syncthreads();
    if (tid < LSR_OWN && i < n) {
        cw = co = cv = 0;
        for (int u = 0; u < 16; ++u) {
            cw += part[u][0][tid];
            co += part[u][1][tid];
            cv += part[u][2][tid];
        }
        r.word[cw] = (cv << 18) | ((kw >> 14) << 4);
        r.by_w[cw] = (unsigned short)co;
        r.by_o[co] = (unsigned short)i;
        r.value[co] = (int)kv;
    }
}

// (the two arrays of the dependent look-ups come first: their offsets fit in an LDS instruction)
struct alignas(16) RankedLds {
    unsigned short rank[LS_TABLE];   // twice the number of places of at most a size
    unsigned short pm[LSR_N];        // upper half of the least word of a non-member before a place
    unsigned word[LSR_N];            // by place
    unsigned short by_w[LSR_N];      // by place: rank by (o, id)
    unsigned short by_o[LSR_N];
    int value[LSR_N];
    unsigned bits[2][LSR_N / 32];    // a batch by rank by (o, id): a bit per request; two batches in turn
    unsigned wave_sum[LSR_NW];
    unsigned wave_top[LSR_NW];
    unsigned wave_min[LSR_NW];
    unsigned out[LSR_NW], in[LSR_NW];  // each wavefront's first member that has a partner, and first one of a smaller value
    int fill_end, fill_mem, fill_w;
    int slack, w_hi, swaps, done;
    int hi;                          // no member lies behind this place, from the batch's first group of eight on
    u64 S;                           // sum of values of the batch that is written out
    int parts;                       // wavefronts that have added theirs
};

// x = from[e] of the least e with a[e] < b[e], or with from[e] < below (x if there is none): written out because a
// comparison's mask may be read only two instructions later, and the compiler fills the gap with idle ones
// when it takes one mask at a time (an exchange of four places per lane: 942 -> 740 cycles).
template <int E>
__device__ __forceinline__ void first_less(unsigned &x, const unsigned (&a)[E], const unsigned (&b)[E])
{
    u64 m0, m1, m2, m3;
    if constexpr (E == 2) {
        asm("v_cmp_lt_u32 %2, %4, %6\n\tv_cmp_lt_u32 %1, %3, %5\n\ts_nop 0\n\tv_cndmask_b32 %0, %0, %6, %2\n\tv_cndmask_b32 %0, %0, %5, %1"
            : "+&v"(x), "=&s"(m0), "=&s"(m1) : "v"(a[0]), "v"(a[1]), "v"(b[0]), "v"(b[1]));
    } else {
#pragma unroll
        for (int e = E - 4; e >= 0; e -= 4)
            asm("v_cmp_lt_u32 %4, %8, %12\n\tv_cmp_lt_u32 %3, %7, %11\n\tv_cmp_lt_u32 %2, %6, %10\n\tv_cmp_lt_u32 %1, %5, %9\n\t"
                "v_cndmask_b32 %0, %0, %12, %4\n\tv_cndmask_b32 %0, %0, %11, %3\n\tv_cndmask_b32 %0, %0, %10, %2\n\tv_cndmask_b32 %0, %0, %9, %1"
                : "+&v"(x), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3)
                : "v"(a[e]), "v"(a[e + 1]), "v"(a[e + 2]), "v"(a[e + 3]), "v"(b[e]), "v"(b[e + 1]), "v"(b[e + 2]), "v"(b[e + 3]));
    }
}

template <int E>
__device__ __forceinline__ void first_below(unsigned &x, unsigned below, const unsigned (&from)[E])
{
    u64 m0, m1, m2, m3;
    if constexpr (E == 2) {
        asm("v_cmp_gt_u32 %2, %3, %5\n\tv_cmp_gt_u32 %1, %3, %4\n\ts_nop 0\n\tv_cndmask_b32 %0, %0, %5, %2\n\tv_cndmask_b32 %0, %0, %4, %1"
            : "+&v"(x), "=&s"(m0), "=&s"(m1) : "s"(below), "v"(from[0]), "v"(from[1]));
    } else {
#pragma unroll
        for (int e = E - 4; e >= 0; e -= 4)
            asm("v_cmp_gt_u32 %4, %5, %9\n\tv_cmp_gt_u32 %3, %5, %8\n\tv_cmp_gt_u32 %2, %5, %7\n\tv_cmp_gt_u32 %1, %5, %6\n\t"
                "v_cndmask_b32 %0, %0, %9, %4\n\tv_cndmask_b32 %0, %0, %8, %3\n\tv_cndmask_b32 %0, %0, %7, %2\n\tv_cndmask_b32 %0, %0, %6, %1"
                : "+&v"(x), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3)
                : "s"(below), "v"(from[e]), "v"(from[e + 1]), "v"(from[e + 2]), "v"(from[e + 3]));
    }
}

// The lowest lane of a mask (some lane, if there is none).
__device__ __forceinline__ int first_lane(u64 mask)
{
    int l;
    asm("s_ff1_i32_b64 %0, %1" : "=s"(l) : "s"(mask));
    return l & 63;
}

// State of a batch's exchanges, the same in every thread.  Places count from the batch's first group of eight.
struct RankedState {
    int slack, w_hi, swaps;  // (w_hi: no member is larger)
};

// Exchanges of one batch while no place from NW 64 E - 1 on can fit, by NW wavefronts (1: without
// barriers, called by one wavefront; or all of the workgroup).  Returns true when none is left.
template <int NW, int E>
__device__ __forceinline__ bool ranked_steps(RankedLds &L, int p0, int n, int w_last, int fill_from, int fill_to,
                                             RankedState &st)
{
    static_assert(E >= 2 && E <= 16, "numbers of registers in the words");
    constexpr int PLACES = NW * 64 * E;
    const int lane = threadIdx.x & 63, wave = NW == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int q = (wave * 64 + lane) * E;
    asm volatile("" : "+v"(q));  // (keeps what each split derives from it out of the batches' loop, where it fills the registers)
    unsigned v[E];  // the words of this thread's places
    int w2[E];      // twice their sizes
#pragma unroll
    for (int e = 0; e < E; e += 2) {
        const any_u32x2 x = *reinterpret_cast<const any_u32x2 *>(&L.word[min(p0 + q + e, LSR_N - 2)]);
        v[e] = p0 + q + e < LSR_N ? x.x : LSR_VALUE;
        v[e + 1] = p0 + q + e < LSR_N ? x.y : LSR_VALUE;
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        w2[e] = 2 * size_of(v[e]);
        v[e] |= (unsigned)e | ((q + e >= fill_from && q + e < fill_to) ? LSR_IN : 0u);
    }
    unsigned in = 0;  // which of them are members, the first one highest
#pragma unroll
    for (int e = 0; e < E; ++e) in |= (v[e] & LSR_IN) >> e;
    // no place from PLACES - 1 on fits against a member while w_hi + slack stays below this
    const int w_limit = n - p0 < PLACES ? LS_INF : __builtin_amdgcn_readfirstlane(size_of(L.word[p0 + PLACES - 1]));
    int slack = __builtin_amdgcn_readfirstlane(st.slack), w_hi = __builtin_amdgcn_readfirstlane(st.w_hi);
    int swaps = __builtin_amdgcn_readfirstlane(st.swaps);
    bool done = false;
    while (w_hi + slack < w_limit) {
        // ---- how far each place would reach as a member (what non-members find is never used)
        unsigned p[E];
        const bool members = NW == 1 || __builtin_amdgcn_ballot_w64(in != 0) != 0;  // (without members nothing is looked up)
        if (members) {
            const int reach = 2 * min(slack, w_last), top = 2 * w_last;
#pragma unroll
            for (int e = 0; e < E; ++e)
                p[e] = *reinterpret_cast<const any_u16 *>(reinterpret_cast<const char *>(L.rank) + min(w2[e] + reach, top));
        }
        // ---- least word of a non-member before each place (as unsigned numbers the members are the largest)
        unsigned pm[E], run = LS_INF;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            pm[e] = run;
            run = min(run, v[e]);
        }
        const int incl = wave_scan<false>((int)run);
        unsigned before = (unsigned)wave_prev<false>(incl);
        if (NW > 1) {
            if (lane == 63) L.wave_min[wave] = (unsigned)incl;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < NW - 1; ++u) before = u < wave ? min(before, L.wave_min[u]) : before;
        }
        {
            any_u32 *to = reinterpret_cast<any_u32 *>(&L.pm[q]);
            unsigned two[E / 2];
#pragma unroll
            for (int e = 0; e < E; e += 2)
                two[e / 2] = __builtin_amdgcn_perm(min(pm[e + 1], before), e == 0 ? before : min(pm[e], before), 0x07060302);
#pragma unroll
            for (int e = 0; e < E / 2; ++e) to[e] = two[e];
        }
        if (NW > 1) __syncthreads();

        // ---- first member with an improving partner that fits
        unsigned x_a = 0, x_b = ~0u;
        if (members) {
#pragma unroll
            for (int e = 0; e < E; ++e)
                p[e] = *reinterpret_cast<const any_u16 *>(reinterpret_cast<const char *>(L.pm) + p[e]) << 16 | (LSR_IN | LSR_REST);
            first_less<E>(x_a, p, v);
        }
        int l_a = first_lane(__builtin_amdgcn_ballot_w64(x_a != 0)), l_b;  // their lanes, elsewhere none
        x_a = (unsigned)__builtin_amdgcn_readlane((int)x_a, l_a);
        if (NW > 1) {
            if (lane == 0) L.out[wave] = x_a;  // (0: none)
            __syncthreads();
            const unsigned each = L.out[lane & (NW - 1)];
            const int u = first_lane(__builtin_amdgcn_ballot_w64(each != 0));
            x_a = (unsigned)__builtin_amdgcn_readlane((int)each, u);
            l_a = u == wave ? l_a : 64;
        }
        if (x_a == 0) {  // none left
            done = true;
            break;
        }

        // ---- its partner: the first non-member of a smaller value
        first_below<E>(x_b, x_a & LSR_VALUE, v);
        l_b = first_lane(__builtin_amdgcn_ballot_w64(x_b != ~0u));
        x_b = (unsigned)__builtin_amdgcn_readlane((int)x_b, l_b);
        if (NW > 1) {
            if (lane == 0) L.in[wave] = x_b;  // (~0: none)
            __syncthreads();
            const unsigned each = L.in[lane & (NW - 1)];
            const int u = first_lane(__builtin_amdgcn_ballot_w64(each != ~0u));
            x_b = (unsigned)__builtin_amdgcn_readlane((int)each, u);
            l_b = u == wave ? l_b : 64;
        }

        // ---- exchange
        const int w_b = size_of(x_b);
        slack -= w_b - size_of(x_a);
        w_hi = max(w_hi, w_b);
        ++swaps;
        in ^= lane == l_a ? LSR_IN >> (x_a & 15) : 0u;
        in ^= lane == l_b ? LSR_IN >> (x_b & 15) : 0u;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const unsigned up = in << e;
            asm("v_bfi_b32 %0, %1, %0, %2" : "+v"(v[e]) : "s"(~LSR_IN), "v"(up));
        }
    }
#pragma unroll
    for (int e = 0; e < E; e += 2)
        if (p0 + q + e < LSR_N) *reinterpret_cast<any_u32x2 *>(&L.word[p0 + q + e]) = any_u32x2{v[e] & ~15u, v[e + 1] & ~15u};
    const u64 with = __builtin_amdgcn_ballot_w64(in != 0);  // lanes with members
    if (with != 0 && lane == 63 - __clzll((long long)with)) atomicMax(&L.hi, q + 33 - __ffs((int)in));
    st.slack = slack;
    st.w_hi = w_hi;
    st.swaps = swaps;
    return done;
}

// A batch that has left, from its bits, by four wavefronts (part 0 ... 3): the order, from place `first` on, and
// its ratio.
__device__ __forceinline__ void ranked_emit(RankedLds &L, int part, const unsigned *bits, int first, double scale,
                                            int *order_out, double *F_out)
{
    static_assert(LSR_N / 32 == 4 * 64, "a word per lane");
    const int lane = threadIdx.x & 63;
    unsigned ahead = 0, mine = 0;
    for (int u = 0; u < 4; ++u) {
        const unsigned x = bits[64 * u + lane];
        if (u < part) ahead += (unsigned)__popc(x);
        if (u == part) mine = x;
    }
    const unsigned c = (unsigned)__popc(mine);
    const unsigned incl = wave_scan_u32(c);
    int at = first + (int)(incl - c) + (int)__builtin_amdgcn_readlane((int)wave_scan_u32(ahead), 63);
    u64 S = 0;
    while (mine != 0) {
        const int k = 32 * (64 * part + lane) + __ffs((int)mine) - 1;
        order_out[at++] = L.by_o[k];
        S += (u64)(unsigned)L.value[k];
        mine &= mine - 1;
    }
    S = wave_scan_u64(S);
    if (lane == 63) {
        atomicAdd(&L.S, S);
        __threadfence_block();
        if (atomicAdd(&L.parts, 1) == 3) *F_out = (double)(long long)atomicAdd(&L.S, 0ull) / scale;
    }
}

__device__ int ranked_construction(RankedLds &L, int n, int M, int gb, const RankedArrays &r, int *order_out,
                                   int *batch_end_out, double *F_out, int *swaps_out, int *num_batches_out, int *words)
{
    constexpr int ROWS = (LS_TABLE / 512 + LSR_NW - 1) / LSR_NW;  // rows of the table per wavefront, at most
    constexpr int OWN = LSR_N / (4 * LSR_T);                     // groups of four places per thread, at most
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int i = tid; i < LSR_N; i += LSR_T) {
        L.word[i] = i < n ? r.word[i] : LSR_VALUE;
        if (i < n) {
            L.by_w[i] = r.by_w[i];
            L.by_o[i] = r.by_o[i];
            L.value[i] = r.value[i];
        }
    }
    for (int i = 8 * tid; i < LS_TABLE; i += 8 * LSR_T) *reinterpret_cast<any_u32x4 *>(&L.rank[i]) = any_u32x4{0, 0, 0, 0};
    for (int i = tid; i < 2 * (LSR_N / 32); i += LSR_T) L.bits[0][i] = 0;
    __syncthreads();
    int a = 0, nb = 0;
    int left = 0, left_K = 0;  // where the batch before starts, and its size
    auto emit_left = [&](int part) {
        if (nb == 0) return;
        ranked_emit(L, part, L.bits[(nb - 1) & 1], left, (double)gb * (double)left_K * (double)left_K, order_out, F_out + nb - 1);
    };
    while (a < n) {
        const int p0 = a & ~7;
        const int groups = (n - p0 + 4 * LSR_T - 1) / (4 * LSR_T);  // of four places, per thread
        const int i0 = p0 + 4 * groups * tid;

        // ---- greedy fill (the longest run of places whose sizes add up to at most M) and the table of ub(), which is
        //      zero here: the last place of each size enters its number, a running maximum fills the gaps
        unsigned sum = 0;
        for (int g = 0; g < groups; ++g) {
            const int i = i0 + 4 * g;
            const any_u32x4 y = *reinterpret_cast<const any_u32x4 *>(&L.word[min(i, LSR_N - 4)]);
            const int next = size_of(L.word[min(i + 4, LSR_N - 1)]);
            const int ws[5] = {size_of(y.x), size_of(y.y), size_of(y.z), size_of(y.w), i + 4 < n ? next : -1};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (i + e < n) {
                    sum += (unsigned)ws[e];
                    if (ws[e] != ws[e + 1]) L.rank[ws[e]] = (unsigned short)(2 * (i + e + 1 - p0));  // (past the last place: size 0)
                }
            }
        }
        const unsigned incl = wave_scan_u32(sum);
        if (lane == 63) L.wave_sum[wave] = incl;
        if (tid == 0) {
            L.S = 0;
            L.parts = 0;
            L.hi = 0;
        }
        const int w_last = __builtin_amdgcn_readfirstlane(size_of(L.word[n - 1]));
        // (rows of 512 entries, eight per lane, from the first size on)
        const int first_row = __builtin_amdgcn_readfirstlane(size_of(L.word[a])) >> 9;
        const int rows = (w_last >> 9) + 1, per = (rows - first_row + LSR_NW - 1) / LSR_NW;
        const int r0 = first_row + wave * per, r1 = min(rows, r0 + per);
        __syncthreads();
        unsigned h[ROWS][8], top = 0;
#pragma unroll
        for (int k = 0; k < ROWS; ++k) {  // (rows past r1 are computed for nothing)
            if (k >= per) break;
            const any_u32x4 y = *reinterpret_cast<const any_u32x4 *>(&L.rank[512 * min(r0 + k, LS_TABLE / 512 - 1) + 8 * lane]);
            h[k][0] = y.x & 0xffffu, h[k][1] = y.x >> 16, h[k][2] = y.y & 0xffffu, h[k][3] = y.y >> 16;
            h[k][4] = y.z & 0xffffu, h[k][5] = y.z >> 16, h[k][6] = y.w & 0xffffu, h[k][7] = y.w >> 16;
        }
        unsigned pre = incl - sum;
#pragma unroll
        for (int u = 0; u < LSR_NW; ++u)
            if (u < wave) pre += L.wave_sum[u];
        // the one thread in whose places the run ends
        if (pre <= (unsigned)M && i0 < n && (pre + sum > (unsigned)M || n <= i0 + 4 * groups)) {
            int i = i0;
            for (bool more = true; more;) {  // four places a turn; it ends in them or at n
                const any_u32x4 y = *reinterpret_cast<const any_u32x4 *>(&L.word[i]);
                const unsigned ws[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned next = pre + (unsigned)size_of(ws[e]);
                    more = more && i < n && next <= (unsigned)M;
                    pre = more ? next : pre;
                    i += more;
                }
            }
            L.fill_end = i;
            L.fill_mem = (int)pre;
            L.fill_w = size_of(L.word[max(i - 1, 0)]);
        }
#pragma unroll
        for (int k = 0; k < ROWS; ++k) {
            if (k >= per) break;
#pragma unroll
            for (int e = 1; e < 8; ++e) h[k][e] = max(h[k][e], h[k][e - 1]);
            const int m = wave_scan<true>((int)h[k][7]);
            const unsigned lower = (unsigned)max(wave_prev<true>(m), (int)top);
            if (r0 + k < r1) top = (unsigned)max((int)top, __builtin_amdgcn_readlane(m, 63));
#pragma unroll
            for (int e = 0; e < 8; ++e) h[k][e] = max(h[k][e], lower);
        }
        if (lane == 0) L.wave_top[wave] = top;
        __syncthreads();
        {
            unsigned lower = 0;
#pragma unroll
            for (int u = 0; u < LSR_NW; ++u)
                if (u < wave) lower = max(lower, L.wave_top[u]);
#pragma unroll
            for (int k = 0; k < ROWS; ++k) {
                if (r0 + k < r1) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) h[k][e] = max(h[k][e], lower);
                    *reinterpret_cast<any_u32x4 *>(&L.rank[512 * (r0 + k) + 8 * lane]) =
                        any_u32x4{h[k][0] | h[k][1] << 16, h[k][2] | h[k][3] << 16, h[k][4] | h[k][5] << 16, h[k][6] | h[k][7] << 16};
                }
            }
        }
        RankedState st;
        st.slack = M - __builtin_amdgcn_readfirstlane(L.fill_mem);
        st.w_hi = __builtin_amdgcn_readfirstlane(L.fill_w);
        st.swaps = 0;
        const int K = __builtin_amdgcn_readfirstlane(L.fill_end) - a;
        if (K < 1) {  // cannot happen for well-formed input; never spin
            if (tid == 0) atomicOr(&words[KVS_W_STATUS], KVSCHED_DEV_BAD_LENGTH);
            break;
        }
        __syncthreads();

        // ---- exchanges; meanwhile the batch before is written out
        bool emitted = false;
        const bool all = a + K == n;  // the batch has taken everything
        int from = a - p0, to = a - p0 + K;  // places that become members when they are first read
        while (!all) {
            const int U = L.rank[min(st.w_hi + st.slack, w_last)] >> 1;  // places from U on fit against no member
            bool done = false;
            if (U < 1024) {
                if (wave == 0) {
                    done = U < 128   ? ranked_steps<1, 2>(L, p0, n, w_last, from, to, st)
                           : U < 256 ? ranked_steps<1, 4>(L, p0, n, w_last, from, to, st)
                           : U < 512 ? ranked_steps<1, 8>(L, p0, n, w_last, from, to, st)
                                     : ranked_steps<1, 16>(L, p0, n, w_last, from, to, st);
                    if (lane == 0) {
                        L.slack = st.slack;
                        L.w_hi = st.w_hi;
                        L.swaps = st.swaps;
                        L.done = done;
                    }
                } else if (wave <= 4 && !emitted) emit_left(wave - 1);
                emitted = true;
                __syncthreads();
                st.slack = __builtin_amdgcn_readfirstlane(L.slack);
                st.w_hi = __builtin_amdgcn_readfirstlane(L.w_hi);
                st.swaps = __builtin_amdgcn_readfirstlane(L.swaps);
                done = __builtin_amdgcn_readfirstlane(L.done) != 0;
            } else if (U < 2048) done = ranked_steps<LSR_NW, 2048 / LSR_T>(L, p0, n, w_last, from, to, st);
            else if (U < 4096) done = ranked_steps<LSR_NW, 4096 / LSR_T>(L, p0, n, w_last, from, to, st);
            else done = ranked_steps<LSR_NW, 8192 / LSR_T>(L, p0, n, w_last, from, to, st);
            __syncthreads();
            if (done) break;  // uniform
            to = from;
        }
        if (!emitted && wave < 4) emit_left(wave);
        if (tid == 0) {
            batch_end_out[nb] = a + K;
            if (swaps_out) swaps_out[nb] = st.swaps;
        }
        const int hi = all ? n : p0 + L.hi;

        // ---- members leave; non-members of [a, hi) close up behind the K removed places.  The table is zeroed.
        unsigned x[OWN][4];
        unsigned short at[OWN][4];
        unsigned stay = 0;
#pragma unroll
        for (int g = 0; g < OWN; ++g) {
            if (g < groups) {
                const int i = i0 + 4 * g;
                const int at_i = min(i, LSR_N - 4);
                const any_u32x4 y = *reinterpret_cast<const any_u32x4 *>(&L.word[at_i]);
                const any_u32x2 z = *reinterpret_cast<const any_u32x2 *>(&L.by_w[at_i]);
                x[g][0] = y.x, x[g][1] = y.y, x[g][2] = y.z, x[g][3] = y.w;
                at[g][0] = (unsigned short)z.x, at[g][1] = (unsigned short)(z.x >> 16);
                at[g][2] = (unsigned short)z.y, at[g][3] = (unsigned short)(z.y >> 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (i + e >= a && i + e < hi) {
                        if (all || (x[g][e] & LSR_IN)) atomicOr(&L.bits[nb & 1][at[g][e] >> 5], 1u << (at[g][e] & 31));
                        else stay |= 1u << (4 * g + e);
                    }
                }
            }
        }
        const unsigned count = (unsigned)__popc(stay);
        const unsigned upto = wave_scan_u32(count);
        if (lane == 63) L.wave_min[wave] = upto;
        for (int i = 8 * tid; i <= w_last; i += 8 * LSR_T) *reinterpret_cast<any_u32x4 *>(&L.rank[i]) = any_u32x4{0, 0, 0, 0};
        __syncthreads();
        {
            int place = a + K + (int)(upto - count);
#pragma unroll
            for (int u = 0; u < LSR_NW; ++u)
                if (u < wave) place += (int)L.wave_min[u];
            if (stay != 0) {
#pragma unroll
                for (int g = 0; g < OWN; ++g) {
                    if (g < groups) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (stay & (1u << (4 * g + e))) {
                                L.word[place] = x[g][e];
                                L.by_w[place] = at[g][e];
                                ++place;
                            }
                        }
                    }
                }
            }
        }
        left = a;
        left_K = K;
        a += K;
        ++nb;
        if (tid < 8 && (a & ~7) + tid < a) L.word[(a & ~7) + tid] = LSR_VALUE;
        if (tid < LSR_N / 32) L.bits[nb & 1][tid] = 0;  // of the batch before the one that has just left
        __syncthreads();
    }
    if (tid == 0) {
        *num_batches_out = nb;
        L.S = 0;
        L.parts = 0;
    }
    __syncthreads();
    if (wave < 4) emit_left(wave);
    return nb;
}

__global__ __launch_bounds__(LSR_T) void ranked_swap_kernel(int32_t n, int32_t M, int32_t gb, RankedArrays r,
                                                            int32_t *order_out, int32_t *batch_end_out, double *F_out,
                                                            int32_t *swaps_out, int32_t *num_batches_out, int32_t pad,
                                                            int32_t *words)
{
    __shared__ RankedLds L;
    const int state = *r.state;
    int nb = 0;
    if (state == 1)
        nb = ranked_construction(L, n, M, gb, r, order_out, batch_end_out, F_out, swaps_out, num_batches_out, words);
    if (state != 0 && pad) {
        for (int i = nb + (int)threadIdx.x; i < n; i += LSR_T) {
            batch_end_out[i] = 0;
            F_out[i] = 0.0;
            if (swaps_out) swaps_out[i] = 0;
        }
    }
}

}  // namespace


size_t kvs_local_swap_scratch_bytes(int32_t n)
{
    const size_t np = ((size_t)n + 64) & ~(size_t)63;
    return np * 8 * sizeof(int) + 256;
}

int kvs_launch_local_swap(int32_t n, const int32_t *s, const int32_t *o, int32_t M, int32_t ga, int32_t gb, int32_t pad,
                          int32_t *order_out,
                          int32_t *batch_end_out, double *F_out, int32_t *swaps_out, int32_t *num_batches_out,
                          void *scratch, int32_t *d_words, hipStream_t st)
{
    const size_t np = ((size_t)n + 64) & ~(size_t)63;
    int *gw = (int *)scratch;
    int *go = gw + np;
    int *gid = go + np;
    int *alt_o = gid + np;
    int *buf0 = alt_o + np;
    int *buf1 = buf0 + np;
    int *by_o = buf1 + np;
    int *batch_of = by_o + np;
    int *state = nullptr;
    if (n < LSR_N) {
        RankedArrays r;
        r.state = state = batch_of + np;
        r.word = (unsigned *)gw;
        r.value = go;
        r.by_w = (unsigned short *)gid;
        r.by_o = (unsigned short *)alt_o;
        hipLaunchKernelGGL(rank_requests_kernel, dim3((unsigned)((n + LSR_OWN - 1) / LSR_OWN)), dim3(1024), 0, st, n, s, o,
                           M, ga, gb, r, d_words, num_batches_out);
        hipLaunchKernelGGL(ranked_swap_kernel, dim3(1), dim3(LSR_T), 0, st, n, M, gb, r, order_out, batch_end_out, F_out,
                           swaps_out, num_batches_out, pad, d_words);
        if (M < LS_TABLE) return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;  // then every size is below it
    } else {
        const int rc = kvs_launch_scan_lengths(s, o, n, M, 0, d_words, st);
        if (rc != KVSCHED_OK) return rc;
    }
    hipLaunchKernelGGL(local_swap_kernel, dim3(1), dim3(LS_T), 0, st, n, s, o, M, ga, gb, order_out, batch_end_out, F_out,
                       swaps_out, num_batches_out, gw, go, gid, alt_o, buf0, buf1, by_o, batch_of, d_words, state, pad);
    return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}
