// Phase 1 of Algorithm 1 ("Batch Construction") with every batch the exact minimiser of
// (F, -|X|), found by Algorithm 2 ("Exact Optimal Request Selection via Dynamic Programming"):
//   dp[k][m] = least sum of o over sets of k requests whose load is exactly m,
// requests taken one by one, k running downward, a state replaced only by a strictly smaller
// value; at the end every state is scored F = dp[k][m] / k^2.
//
// On the GPU a launch offers four requests to the states at once, reading the table before them and writing a second
// one: the value of (k, m) behind four requests depends on the sixteen states before them that lack a part of the four
// (row k - |part|, load m - its load), combined one request after the other, which is what "k downward" achieves in
// place.  One wavefront covers 64 consecutive loads m of one cardinality k, and its ballots of "this state was
// improved by request t" are the only record kept of the chosen sets (bits[t][k][m / 64]).  The set
// of the best state is recovered by walking those records backwards: at state (k, m) the last
// request that improved it is a member, and the walk continues at (k - 1, m - load) among the
// earlier requests.  That is the set Algorithm 2 carries in path[k][m].
//
// Only states that can be part of the answer are kept up to date.  Let kmin be the least k at which the k smallest
// values could sum to as good a metric as a batch known to be feasible (the best prefix in ascending cost).  A chosen set
// has at least kmin members, so after t of r requests a state needs k >= kmin - (r - t), and its load lies between the sum
// of the k smallest loads and M minus that of the kmin - k smallest.  Every state on the way to the answer satisfies
// this, and so does every state its value or its record depends on; the others hold values that are too large at worst.
//
// feas_mode 0: load = sum (s+o) <= M, requests in input order (Algorithm 2 as printed).
// feas_mode 1: the constraint of Algorithm 1's Phase 1 (all of X started together stays within M
//   at every completion time): requests in order of decreasing o, load = sum s, and request j may
//   join k - 1 others only if load + o_j k <= M (j then has the least o, so this is the memory at
//   its completion; the constraints at later completions are not touched by j).
#include "phase1_util.h"
#include "sort_util.h"

namespace {

constexpr int DP_T = 1024;  // threads of the single-workgroup helper kernels
constexpr int DP_NW = DP_T / 64;
constexpr unsigned DP_NONE = 0x80000000u; // no set: above every value (< 2^31), and still below 2^32 with one more added
constexpr int DP_STEP_T = 256;
constexpr int DP_STEP_M = 512;            // loads per workgroup of a step launch, two per thread
constexpr int DP_G = 4;                   // requests per step launch

struct HelperLds {
    RadixLds<DP_T> radix;
    long long scan[DP_NW];
    int scan_c[DP_NW];
    int sh[4];
    long long red_S[DP_NW];
    int red_k[DP_NW];
    int red_m[DP_NW];
};

__device__ __forceinline__ int cost_of(int sv, int ov, int feas_mode)
{
    return feas_mode ? sv + 1 : sv + ov;  // every feasible set of k requests has sum of cost <= M
}

// Length of the longest prefix of list[0..r) (ascending cost) whose costs sum to at most M: no
// feasible set is larger.  All threads return the same value.
__device__ int prefix_fit(const int *list, int r, const int *s, const int *o, int feas_mode, int M, HelperLds &L)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    long long carry = 0;
    int K = 0;
    for (int tile = 0; tile < r; tile += DP_T) {
        const int i = tile + tid;
        long long w = 0;
        if (i < r) {
            const int id = list[i];
            w = cost_of(s[id], o[id], feas_mode);
        }
        for (int d = 1; d < 64; d <<= 1) {
            const long long u = __shfl_up(w, d);
            if (lane >= d) w += u;
        }
        if (lane == 63) L.scan[wave] = w;
        __syncthreads();
        long long off = carry, total = carry;
        for (int v = 0; v < DP_NW; ++v) {
            const long long x = L.scan[v];
            if (v < wave) off += x;
            total += x;
        }
        const int c = __syncthreads_count(i < r && w + off <= (long long)M);
        K += c;
        carry = total;
        if (c < DP_T) break;  // uniform
    }
    __syncthreads();
    return K;
}

// out = the ids of in[0..n) in ascending (key, place), n <= DP_T: a thread counts the keys before its own.  (200 ids:
// 11 us less than the two passes of a radix sort.  Up to a quarter of DP_T ids have four threads each: 3 us less again.)
template <class KeyFn>
__device__ void rank_sort(const int *in, int *out, int n, KeyFn key, HelperLds &L)
{
    typedef int keys4 __attribute__((ext_vector_type(4), may_alias));
    static_assert(sizeof(L.radix.wcount) >= DP_T * sizeof(int), "room for the keys");
    int *k = &L.radix.wcount[0][0];
    const int tid = threadIdx.x;
    const int id = tid < n ? in[tid] : 0;
    const int mine = tid < n ? key(id) : INT_MAX;  // (keys are below INT_MAX)
    __syncthreads();
    k[tid] = mine;
    __syncthreads();
    // (parts: threads for each id, which share the quads; their counts are added up)
    const int parts = 4 * n <= DP_T ? 4 : 1, at = tid / parts, part = tid % parts;
    const int own = parts == 1 ? mine : k[at];
    int rank = 0;
    for (int q = part; 4 * q < n; q += parts) {
        const keys4 v = reinterpret_cast<const keys4 *>(k)[q];
        const int limit = 4 * q + 3 < at && at < n ? own + 1 : own;  // equal keys count when the whole quad lies before this one
        rank += (v.x < limit) + (v.y < limit) + (v.z < limit) + (v.w < limit);
    }
    if (part == 0)
        for (int j = at & ~3; j < at; ++j) rank += k[j] == own;
    if (parts == 4) {
        rank += __shfl_xor(rank, 1);
        rank += __shfl_xor(rank, 2);
    }
    if (at < n && part == 0) out[rank] = parts == 1 ? id : in[at];
    __syncthreads();
}

// Validation, the three orders of the ids (emission order (o, id); processing order; ascending
// cost), the first bound on the batch size.
// Returns that bound, or -1 for malformed lengths (reported; no batches).  costs: without it neither the order by cost nor
// the bound are made (0 is returned).
__device__ int prepare_body(int32_t n, const int32_t *s, const int32_t *o, int32_t M, int32_t feas_mode, int *proc,
                            int *by_o, int *by_cost, int *buf0, int *buf1, int *batch_of, int32_t *words,
                            int32_t *num_batches_out, HelperLds &L, bool costs = true)
{
    const int tid = threadIdx.x;
    int omax = 0, cmax = 0, bad = 0;
    for (int i = tid; i < n; i += DP_T) {
        const int sv = s[i], ov = o[i];
        if (sv < 1 || ov < 1 || (long long)sv + ov > (long long)M) bad = 1;
        else {
            omax = max(omax, ov);
            cmax = max(cmax, cost_of(sv, ov, feas_mode));
        }
        batch_of[i] = -1;
    }
    if (tid < 4) L.sh[tid] = 0;
    __syncthreads();
    if (bad) atomicOr(&L.sh[2], 1);
    atomicMax(&L.sh[0], omax);
    atomicMax(&L.sh[1], cmax);
    __syncthreads();
    omax = L.sh[0];
    cmax = L.sh[1];
    if (tid == 0) {  // (the first kernel of the call: as the length scan leaves them)
        words[KVS_W_STATUS] = L.sh[2] != 0 ? KVSCHED_DEV_BAD_LENGTH : 0;
        words[KVS_W_STATUS_AT] = KVS_W_STATUS;
        words[KVS_W_OMAX] = omax;
        words[KVS_W_MINPOS] = INT_MAX;
        words[KVS_W_MAXPOS] = -1;
    }
    if (L.sh[2] != 0) {  // a request that can never run: report, emit no batches
        if (tid == 0) {
            words[KVS_W_REMAIN] = 0;
            words[KVS_W_KMAX] = 0;
            *num_batches_out = 0;
        }
        return -1;
    }
    auto sort_by = [&](int *out, auto key, int kmax_key) {
        for (int i = tid; i < n; i += DP_T) buf0[i] = i;
        __syncthreads();
        if (n <= DP_T) {
            rank_sort(buf0, out, n, key, L);
            return;
        }
        int *cur = buf0, *alt = buf1;
        for (int shift = 0; shift < bits_of(kmax_key); shift += 8) {
            radix_pass(cur, alt, n, shift, key, L.radix);
            int *t = cur; cur = alt; alt = t;
        }
        for (int i = tid; i < n; i += DP_T) out[i] = cur[i];
        __syncthreads();
    };
    sort_by(by_o, [o](int id) { return o[id]; }, omax);
    if (feas_mode) sort_by(proc, [o, omax](int id) { return omax - o[id]; }, omax);
    else {
        for (int i = tid; i < n; i += DP_T) proc[i] = i;
        __syncthreads();
    }
    if (!costs) {
        __threadfence_block();
        __syncthreads();
        return 0;
    }
    sort_by(by_cost, [s, o, feas_mode](int id) { return cost_of(s[id], o[id], feas_mode); }, cmax);
    __threadfence_block();
    __syncthreads();
    return prefix_fit(by_cost, n, s, o, feas_mode, M, L);
}

// The entry for "no set", which the states before row 0 and load 0 are read from (DP_FRONT words of it), and both tables.
constexpr int DP_FRONT = 64;
__global__ __launch_bounds__(DP_STEP_T) void dp_init_kernel(unsigned *a, size_t count, size_t table)
{
    const size_t i = (size_t)blockIdx.x * DP_STEP_T + threadIdx.x;
    if (i < count) a[i] = i >= DP_FRONT && (i - DP_FRONT) % table == 0 ? 0u : DP_NONE;  // dp[0][0] = 0
}

// What the step launches read, laid out so that one round trip brings it: per request in processing order its load,
// decode length and value; per row k the loads a chosen set can pass through (see the top of the file).
struct DpPlan {
    const int4 *req;
    const int2 *range;
};

// Requests proc[t0 .. t0 + DP_G) offered to row k = k_first + blockIdx.y, loads blockIdx.x * DP_STEP_M ...
// Bound by the launch and by L2 reads (16 per state and four requests, where one request a launch took 2 reads and a
// write each): 200 requests, M = 16384: 497 launches of 4.5 us become 126 of 5.6 us (two dependent reads and a write take 4 of them).
template <int MODE>
__global__ __launch_bounds__(DP_STEP_T) void dp_step_kernel(DpPlan plan, int t0, int r, int32_t M, const unsigned *none,
                                                            const unsigned *src, unsigned *dst, unsigned long long *bits,
                                                            size_t per_t, int Mp, int k_first)
{
    const int k = k_first + (int)blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int m0 = (int)blockIdx.x * DP_STEP_M + 128 * __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int2 range = plan.range[k];
    const int lo = range.x, hi = range.y;
    unsigned load[DP_G], gain[DP_G];
    int len[DP_G];
#pragma unroll
    for (int g = 0; g < DP_G; ++g) {  // (behind the last request: entries that join nothing)
        const int4 q = plan.req[t0 + g];
        load[g] = (unsigned)q.x;
        len[g] = q.y;
        gain[g] = (unsigned)q.z;
    }
    if (m0 > hi || m0 + 127 < lo) return;
    unsigned off[1 << DP_G];
    off[0] = 0;
#pragma unroll
    for (int h = 1; h < (1 << DP_G); ++h) off[h] = off[h & (h - 1)] + load[__builtin_ctz(h)];
    if (k < DP_G) {  // no set has fewer than no members: such a state reads as one of negative load does
#pragma unroll
        for (int h = 1; h < (1 << DP_G); ++h)
            if (__builtin_popcount(h) > k) off[h] = ~0u;
    }
    const unsigned *row = src + (size_t)k * Mp;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int mc = m0 + 64 * c;
        if (mc > hi || mc + 63 < lo) continue;
        const unsigned m = (unsigned)(mc + lane);
        unsigned f[1 << DP_G];  // f[h]: the state that lacks the requests of h, behind those below h's lowest
#pragma unroll
        for (int h = 0; h < (1 << DP_G); ++h)
            f[h] = *(off[h] <= m ? row + ((long long)m - off[h] - (long long)__builtin_popcount(h) * Mp) : none);
        static_assert(DP_G == 4, "sixteen states");
        // all sixteen reads are in flight before the first is waited for
        asm volatile("" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "+v"(f[4]), "+v"(f[5]), "+v"(f[6]), "+v"(f[7]),
                     "+v"(f[8]), "+v"(f[9]), "+v"(f[10]), "+v"(f[11]), "+v"(f[12]), "+v"(f[13]), "+v"(f[14]), "+v"(f[15]));
        unsigned long long took[DP_G];
#pragma unroll
        for (int g = 0; g < DP_G; ++g) {
#pragma unroll
            for (int h = 0; h < (1 << DP_G); h += 2 << g) {
                unsigned with = f[h | (1 << g)] + gain[g];
                if (MODE && (long long)m - (long long)off[h] + (long long)len[g] * (k - __builtin_popcount(h)) > (long long)M) with = DP_NONE;
                if (h == 0) took[g] = __builtin_amdgcn_ballot_w64(with < f[0]);
                f[h] = min(f[h], with);
            }
        }
        dst[(size_t)k * Mp + m] = f[0];
        if (lane == 0) {
            unsigned long long *b = bits + (size_t)t0 * per_t + (size_t)k * (Mp >> 6) + (mc >> 6);
#pragma unroll
            for (int g = 0; g < DP_G; ++g)
                if (t0 + g < r) b[(size_t)g * per_t] = took[g];
        }
    }
}

// sign of Sa/ka^2 - Sb/kb^2 (S < 2^31, k <= 4096: the products stay below 2^55)
__device__ __forceinline__ int dp_cmp_F(long long Sa, int ka, long long Sb, int kb)
{
    const long long l = Sa * (long long)kb * (long long)kb, r = Sb * (long long)ka * (long long)ka;
    return l < r ? -1 : (l > r ? 1 : 0);
}

// Is state a a better final choice than state b?  Least F; among equal F the larger k
// (KVSCHED_TIE_LARGER) or the smaller; then the smaller load (the first met scanning m upward).
__device__ __forceinline__ bool dp_better(long long Sa, int ka, int ma, long long Sb, int kb, int mb, int tie_rule)
{
    if (ka == 0) return false;
    if (kb == 0) return true;
    const int c = dp_cmp_F(Sa, ka, Sb, kb);
    if (c != 0) return c < 0;
    if (ka != kb) return tie_rule == KVSCHED_TIE_LARGER ? ka > kb : ka < kb;
    return ma < mb;
}

// Block-wide best of per-thread candidates; every thread receives it.
__device__ void reduce_best(int32_t tie_rule, HelperLds &L, long long &bS, int &bk, int &bm)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int d = 32; d > 0; d >>= 1) {
        const long long oS = __shfl_down(bS, d);
        const int ok = __shfl_down(bk, d), om = __shfl_down(bm, d);
        if (dp_better(oS, ok, om, bS, bk, bm, tie_rule)) { bS = oS; bk = ok; bm = om; }
    }
    __syncthreads();  // the reduction slots may still be read from an earlier call
    if (lane == 0) { L.red_S[wave] = bS; L.red_k[wave] = bk; L.red_m[wave] = bm; }
    __syncthreads();
    if (wave == 0) {  // (a total order)
        bS = L.red_S[lane & (DP_NW - 1)];
        bk = L.red_k[lane & (DP_NW - 1)];
        bm = L.red_m[lane & (DP_NW - 1)];
        for (int d = DP_NW / 2; d > 0; d >>= 1) {
            const long long oS = __shfl_xor(bS, d);
            const int ok = __shfl_xor(bk, d), om = __shfl_xor(bm, d);
            if (dp_better(oS, ok, om, bS, bk, bm, tie_rule)) { bS = oS; bk = ok; bm = om; }
        }
        if (lane == 0) { L.red_S[0] = bS; L.red_k[0] = bk; L.red_m[0] = bm; }
    }
    __syncthreads();
    bS = L.red_S[0];
    bk = L.red_k[0];
    bm = L.red_m[0];
}

// Best final state among rows 1 ... kmax of a table of rows of 2^lg loads; every thread receives it (bk = 0: none).
__device__ void argmin_body(const unsigned *dp, int kmax, int32_t M, int lg, int32_t tie_rule, HelperLds &L, long long &bS, int &bk,
                            int &bm)
{
    bS = 0;
    bk = 0;
    bm = 0;
    for (int i = threadIdx.x; i < kmax << lg; i += DP_T) {
        const int k = 1 + (i >> lg), m = i & ((1 << lg) - 1);
        const unsigned v = dp[i + (1 << lg)];
        if (m <= M && v != DP_NONE && dp_better(v, k, m, bS, bk, bm, tie_rule)) { bS = v; bk = k; bm = m; }
    }
    reduce_best(tie_rule, L, bS, bk, bm);
}

// Thread 0: the outputs of batch nb (or the report that no state exists, which cannot happen for
// well-formed input: a single request always fits).
__device__ void publish_batch(long long bS, int bk, int32_t gb, int32_t done, int32_t nb, int32_t *batch_end_out,
                              double *F_out, int32_t *words)
{
    if (bk >= 1) {
        batch_end_out[nb] = done + bk;
        F_out[nb] = (double)bS / ((double)gb * (double)bk * (double)bk);
    } else {
        atomicOr(&words[KVS_W_STATUS], KVSCHED_DEV_BAD_LENGTH);
    }
}

// Row k = kmin + blockIdx.x of the last table: its least value and the least load that has it, as value << 32 | load.
__global__ __launch_bounds__(DP_T) void dp_argmin_rows_kernel(const unsigned *dp, int kmin, int Mp, DpPlan plan,
                                                              unsigned long long *partial)
{
    __shared__ unsigned long long red[DP_NW];
    const int k = kmin + (int)blockIdx.x;
    const int lo = plan.range[k].x, hi = plan.range[k].y;
    unsigned long long best = ~0ull;
    for (int m = max(lo, 0) + threadIdx.x; m <= hi; m += DP_T) {
        const unsigned v = dp[(size_t)k * Mp + m];
        best = min(best, ((unsigned long long)v << 32) | (unsigned)m);
    }
    for (int d = 32; d > 0; d >>= 1) best = min(best, (unsigned long long)__shfl_xor((long long)best, d));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int v = 1; v < DP_NW; ++v) best = min(best, red[v]);
        partial[blockIdx.x] = best;
    }
}

// One wavefront follows the records back from the best state (k, m) and stamps the members with the batch number.  The
// records of six consecutive requests are read together, one lane for each way the later of them may have been members
// (63 states): a round trip to memory serves six requests instead of the one to two that tests of (k, m) against a run of
// requests do.  (Ten at a time by sixteen wavefronts is slower: a thousand reads all over the records.)
// load[t]: loads in processing order (LDS).
__device__ void walk_body(const unsigned long long *bits, const int *proc, int r, int kmax, int Mp, const int *load,
                          int32_t nb, int *batch_of, int k, int m)
{
    const int lane = threadIdx.x & 63;
    const size_t per_t = (size_t)(kmax + 1) * (Mp >> 6);
    // lane v >= 1 is a node of a binary tree: depth floor(log2 v), its low bits the choices above (latest first)
    const int depth = 31 - __builtin_clz(lane | 1);
    int bound = r - 1;
    while (k > 0 && bound >= 0) {
        const int ahead = lane < 6 && lane <= bound ? load[bound - lane] : 0;
        const int ids = lane < 6 && lane <= bound ? proc[bound - lane] : 0;
        int kk = k, mm = m;
#pragma unroll
        for (int d = 0; d < 5; ++d) {
            const int l = __builtin_amdgcn_readlane(ahead, d);
            if (d < depth && ((lane >> (depth - 1 - d)) & 1)) {
                kk -= 1;
                mm -= l;
            }
        }
        const int t = bound - depth;
        bool hit = false;
        if (lane > 0 && t >= 0 && kk > 0 && mm >= 0)
            hit = (bits[(size_t)t * per_t + (size_t)kk * (Mp >> 6) + (mm >> 6)] >> (mm & 63)) & 1ull;
        const unsigned long long tree = __builtin_amdgcn_ballot_w64(hit);
        int v = 1;
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            if (k > 0 && bound >= 0) {
                const int in = (int)((tree >> v) & 1ull);
                if (in) {
                    if (lane == d) batch_of[ids] = nb;
                    m -= __builtin_amdgcn_readlane(ahead, d);
                    k -= 1;
                }
                v = 2 * v + in;
                bound -= 1;
            }
        }
    }
}

// Members leave proc[], by_cost[] and left_by_o[] (or NULL; all keep their order); kept = the new count, kmax = the new
// bound on the batch size.
__device__ void compact_body(int *proc, int *by_cost, int *left_by_o, int *tmp, int r, const int *batch_of, const int32_t *s,
                             const int32_t *o, int32_t feas_mode, int32_t M, HelperLds &L, int &kept, int &kmax)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    kept = 0;
    for (int pass = 0; pass < (left_by_o ? 3 : 2); ++pass) {
        int *list = pass == 0 ? proc : pass == 1 ? by_cost : left_by_o;
        int carry = 0;
        for (int tile = 0; tile < r; tile += DP_T) {
            const int i = tile + tid;
            int id = 0, keep = 0;
            if (i < r) {
                id = list[i];
                keep = batch_of[id] < 0;
            }
            int c = keep;
            for (int d = 1; d < 64; d <<= 1) {
                const int u = __shfl_up(c, d);
                if (lane >= d) c += u;
            }
            if (lane == 63) L.scan_c[wave] = c;
            __syncthreads();
            int off = carry, total = carry;
            for (int u = 0; u < DP_NW; ++u) {
                const int x = L.scan_c[u];
                if (u < wave) off += x;
                total += x;
            }
            if (keep) tmp[off + c - 1] = id;
            carry = total;
            __syncthreads();
        }
        kept = carry;
        __threadfence_block();
        __syncthreads();
        for (int i = tid; i < kept; i += DP_T) list[i] = tmp[i];
        __threadfence_block();
        __syncthreads();
    }
    kmax = kept > 0 ? prefix_fit(by_cost, kept, s, o, feas_mode, M, L) : 0;
}

// For the kmax cheapest of the r requests: cost[k] = sum of the k least costs (cost[0] = 0), and kmin (see the top).
// Every thread receives kmin.
__device__ int bounds_body(const int *by_cost, const int *left_by_o, int kmax, const int32_t *s, const int32_t *o, int32_t M,
                           int32_t ga, int32_t gb, int32_t feas_mode, int *cost, HelperLds &L)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __shared__ long long sc[3][DP_NW];
    auto scan3 = [&](long long (&v)[3], long long (&carry)[3]) {  // inclusive sums over the workgroup, behind carry
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            for (int d = 1; d < 64; d <<= 1) {
                const long long u = __shfl_up(v[q], d);
                if (lane >= d) v[q] += u;
            }
            if (lane == 63) sc[q][wave] = v[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            long long off = carry[q];
            for (int u = 0; u < DP_NW; ++u) {
                if (u == wave) v[q] += off;
                off += sc[q][u];
            }
            carry[q] = off;
        }
        __syncthreads();
    };
    // the best prefix in ascending cost that fits by its peaks (it then fits under either constraint)
    long long bS = 0;
    int bk = 0, bm = 0;
    long long carry[3] = {0, 0, 0};
    for (int tile = 0; tile < kmax; tile += DP_T) {
        const int i = tile + tid;
        long long v[3] = {0, 0, 0};  // cost, peak, value
        if (i < kmax) {
            const int id = by_cost[i];
            v[0] = cost_of(s[id], o[id], feas_mode);
            v[1] = (long long)s[id] + o[id];
            v[2] = (long long)ga * s[id] + (long long)gb * o[id];
        }
        scan3(v, carry);
        if (i < kmax) {
            cost[i + 1] = (int)v[0];
            if (v[1] <= (long long)M && dp_better(v[2], i + 1, 0, bS, bk, bm, KVSCHED_TIE_LARGER)) bS = v[2], bk = i + 1;
        }
    }
    if (tid == 0) cost[0] = 0;
    reduce_best(KVSCHED_TIE_LARGER, L, bS, bk, bm);
    // least k whose k smallest values (at least gb o + ga each) could do as well
    if (tid == 0) L.sh[0] = kmax;
    __syncthreads();
    carry[0] = carry[1] = carry[2] = 0;
    for (int tile = 0; tile < kmax; tile += DP_T) {
        const int i = tile + tid;
        long long v[3] = {0, 0, 0};
        if (i < kmax) v[0] = (long long)gb * o[left_by_o[i]] + ga;
        scan3(v, carry);
        if (i < kmax && bk > 0 && dp_cmp_F(v[0], i + 1, bS, bk) <= 0) atomicMin(&L.sh[0], i + 1);
    }
    __syncthreads();
    const int kmin = bk > 0 ? L.sh[0] : 1;
    __syncthreads();
    return kmin;
}

// The plan of a batch over the r requests proc[0 .. r) (DP_G more entries that join nothing).
__device__ void plan_body(const int *proc, int r, int kmin, int kmax, const int32_t *s, const int32_t *o, int32_t M,
                          int32_t ga, int32_t gb, int32_t feas_mode, const int *cost, int4 *req, int2 *range)
{
    for (int t = threadIdx.x; t < r + DP_G; t += DP_T) {
        int4 q = make_int4(M + 1, 0, 0, 0);
        if (t < r) {
            const int id = proc[t], sv = s[id], ov = o[id];
            q = make_int4(feas_mode ? sv : sv + ov, ov, ga * sv + gb * ov, 0);
        }
        req[t] = q;
    }
    for (int k = threadIdx.x; k <= kmax; k += DP_T) {
        const int more = feas_mode ? k : 0;
        range[k] = make_int2(cost[k] - more, M - more - (kmin > k ? cost[kmin - k] : 0));
    }
}

// What the host waits for between batches.
__device__ __forceinline__ void tell_host(int32_t *words, int32_t *host, int32_t seq, int r, int kmax, int kmin, int nb)
{
    host[KVS_H_BATCHES] = nb;
    words[KVS_W_REMAIN] = r;
    words[KVS_W_KMAX] = kmax;
    host[KVS_H_REMAIN] = r;
    host[KVS_H_KMAX] = kmax;
    host[KVS_H_KMIN] = kmin;
    __threadfence_system();
    __hip_atomic_store(&host[KVS_H_SEQ], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The (o, id)-sorted ids ordered by batch number (stable): each batch in nondecreasing o.
__device__ void emit_body(int32_t n, const int *by_o, int *buf0, int *buf1, const int *batch_of, int32_t nb,
                          int32_t *order_out, int32_t *num_batches_out, HelperLds &L)
{
    const int tid = threadIdx.x;
    const int *src = by_o;
    int *dst = buf0, *other = buf1;
    auto key_b = [batch_of](int id) { return batch_of[id]; };
    if (n <= DP_T) {
        rank_sort(by_o, order_out, n, key_b, L);
        if (tid == 0) *num_batches_out = nb;
        return;
    }
    bool first = true;
    for (int shift = 0; shift < bits_of(nb - 1); shift += 8) {
        radix_pass(src, dst, n, shift, key_b, L.radix);
        if (first) { src = dst; dst = other; first = false; }
        else { int *t = (int *)src; src = dst; dst = t; }
    }
    for (int i = tid; i < n; i += DP_T) order_out[i] = src[i];
    if (tid == 0) *num_batches_out = nb;
}

// ---------------------------------------------------------------------------------------------
// Batches decided without a table (sum of peaks, up to CORE_N requests left).
//
// For a price p >= 0 of load and a size k, the k least values of (value + p load) added up, less p M, are a lower bound on the
// value of every set of k requests that fits ("load <= M" relaxed).  With a good set known, of metric F, a size is out of
// the question when its bound exceeds F k^2.  A request is out when for every size left the bound with it forced in does,
// and it is in when the bound without it does.  Bounds come from 16 prices at a time, a wavefront each (one sort gives
// those of all sizes): a coarse grid, a finer one around the best price of the best size, and one over the best prices of the
// sizes that are left.  The good set is the best prefix of any of these orders, bettered by one request more or
// exchanged and by all choices from the CORE_WINDOW requests about the end of a prefix.  The requests that remain undecided are
// tried in all combinations if they are CORE_MAX or fewer.  Of 300 backlogs of 200 chat requests and of others down to 30,
// 8 to 20 % of the batches leave more than 8 undecided, 1 % more than 16, none of 645 more than 18 (without the choices
// about the end: up to 26, and 1 % more than 20).
//
// The batch is the one the tables would give: all sets as good as the best are among those tried, and of those of one
// size and load the tables keep the one whose latest request is the earliest, then whose second latest is, and so on
// (a state's record is the last request that improved it): the least as a binary number, the earliest request its lowest bit.
// Sums are exact; bounds are in double precision, and a request or size is given up only beyond one part in 10^9.  Orders are
// by keys of 24 bits, which tell sums apart that differ by a step: bounds, sizes that fit and requests have that much room.
//
// Bound by the instructions of one workgroup and their chain (a batch of 200 requests left takes 43 us, of 40 or fewer 22:
// three sorts of 0.6 to 1.3 us, 2.5 to 5 for what the prefixes of their orders give, 2 to 3 for better sets, the combinations 1 to 6).
// 200 chat requests, M = 16384: 1.06 ms with tables (126 launches), 0.17 this way, and 0.1 for each batch that needs tables after
// all (one of 200).
constexpr int CORE_N = KVS_EXACT_SEARCH_N;
constexpr int CORE_MAX = 20;
constexpr int CORE_SIZES = 16;
constexpr int CORE_WINDOW = 14;

struct CoreLds {
    int id[CORE_N], value[CORE_N], load[CORE_N];  // the remaining requests in processing order
    unsigned char at[DP_NW][CORE_N];              // by wavefront: the request at a place of its order
    double bound[DP_NW][CORE_N];                  // by wavefront: the bound for size place + 1
    double price[3 * DP_NW];                       // by turn and wavefront
    // by size: the best bound (a double of no sign compares as a whole number), in its last six bits the price it comes from
    unsigned long long best_bound[CORE_N];
    double per_square[CORE_N];
    // of one wavefront's order, with as many places before the first (nothing) and behind the last (never fits)
    long long sum_load[CORE_N], sum_value[CORE_N];
    int2 sorted[64 + CORE_N + 64];  // (load, value)
    unsigned char out[CORE_SIZES][CORE_N], in[CORE_SIZES][CORE_N];  // by size: is the request out of, or in, every set?
    int size[CORE_SIZES], dead[CORE_SIZES];
    unsigned long long best_of[CORE_SIZES];
    int2 undecided[CORE_MAX];  // (load, value)
    int over[CORE_MAX / 2 + 1][CORE_MAX / 2 + 2];  // [b][j]: b over j
    int first[CORE_MAX / 2 + 2];                   // place of the first combination of j members of the lower half
    int2 low[1 << CORE_MAX / 2];                   // (load, value)
    unsigned short low_set[1 << CORE_MAX / 2];
    unsigned long long best_key, total[2];
    int fits, prefix, subset, most[2];
    int sure[3];  // requests in every set: number, value, load
    int wave_count[2][CORE_N / 64];
};

// Places of the threads whose flag is set, in thread order (tid < CORE_N); count receives how many.  (slot: two calls in a row differ.)
__device__ __forceinline__ int place_of(bool flag, CoreLds &C, int slot, int &count)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned long long set = __builtin_amdgcn_ballot_w64(flag && tid < CORE_N);
    if (lane == 0 && wave < CORE_N / 64) C.wave_count[slot][wave] = __popcll(set);
    __syncthreads();
    int before = 0;
    count = 0;
    for (int w = 0; w < CORE_N / 64; ++w) {
        if (w < wave) before += C.wave_count[slot][w];
        count += C.wave_count[slot][w];
    }
    return before + __popcll(set & ((1ull << lane) - 1ull));
}

// Metric and size of a set as a key that orders by the metric (to one part in 10^12).
__device__ __forceinline__ unsigned long long set_key(double value, int k, double per_square)
{
    return ((unsigned long long)__double_as_longlong(value * per_square) & ~4095ull) | (unsigned)k;
}

// What does not change from batch to batch.
__device__ __forceinline__ void core_start(CoreLds &C)
{
    const int tid = threadIdx.x;
    if (tid < CORE_N) C.per_square[tid] = 1.0 / ((double)(tid + 1) * (double)(tid + 1));
    if (tid < 64) {  // Pascal's triangle, a column a lane
        int above = tid == 0;
#pragma unroll 1
        for (int b = 0; b <= CORE_MAX / 2; ++b) {
            if (tid <= CORE_MAX / 2 + 1) C.over[b][tid] = above;
            const int left = __shfl_up(above, 1);
            above += tid == 0 ? 0 : left;
        }
    }
}

// One batch of the r <= CORE_N requests in C.id ..; its members are marked and leave the lists.  False: not decided, nothing has
// changed.
__device__ __forceinline__ bool core_batch(int &r, int32_t M, int32_t gb, int32_t tie_rule, int32_t n, int32_t nb, int *batch_of,
                                           int32_t *batch_end_out, double *F_out, int32_t *words, CoreLds &C)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double margin = 1e-9;
    if (tid < 2) C.total[tid] = 0, C.most[tid] = 0;
    if (tid < 3) C.sure[tid] = 0;
    if (tid == 0) C.best_key = ~0ull, C.subset = INT_MAX;
    if (tid < CORE_SIZES) C.dead[tid] = 0, C.best_of[tid] = ~0ull;
    __syncthreads();
    const int value = tid < r ? C.value[tid] : 0, load = tid < r ? C.load[tid] : 0;
    if (tid < CORE_N) {
        const u64 v = wave_scan_u64((u64)value), w = wave_scan_u64((u64)load);
        const unsigned most_v = ~wave_min_u32(~(unsigned)value), most_w = ~wave_min_u32(~(unsigned)load);
        if (lane == 63) {
            atomicAdd(&C.total[0], v);
            atomicAdd(&C.total[1], w);
            atomicMax(&C.most[0], (int)most_v);
            atomicMax(&C.most[1], (int)most_w);
        }
        C.best_bound[tid] = 0;
    }
    __syncthreads();
    const double scale = (double)C.total[0] / (double)C.total[1];
    const bool wide = ((C.total[0] | C.total[1]) >> 32) != 0;
    double centre = scale, low = 0.0, ratio = 0.0, F = 0.0;
    int sizes = 0, bk = 0;
    if (r <= CORE_MAX / 2) {  // all combinations at once
        sizes = r;
        if (tid < r) C.size[tid] = tid + 1;
    }
#pragma unroll 1
    for (int turn = 0; turn < 3 && sizes != r; ++turn) {
        // the price of this wavefront (turn 0: none, a grid over four orders of magnitude, and load alone)
        double price;
        if (turn == 0) price = wave == 0 ? 0.0 : scale * (double)exp2f(0.7655f * (float)(wave - 10));
        else if (turn == 1) price = centre * (double)exp2f(0.7655f * ((float)wave - 7.5f) / 7.5f);
        else price = low * (double)exp2f((float)ratio * (float)wave / 15.0f);
        const bool by_load = turn == 0 && wave == DP_NW - 1;
        // sorted by their sums in steps of 2^-24 of the greatest
        const double most = by_load ? (double)C.most[1] : (double)C.most[0] + price * (double)C.most[1];
        const double step = most * (1.0 / 16776000.0), per_step = 16777000.0 / most;
        unsigned key[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 64 * e + lane;
            key[e] = ~0u;
            if (i < r) {
                const double c = by_load ? (double)C.load[i] : (double)C.value[i] + price * (double)C.load[i];
                key[e] = ((unsigned)(c * per_step) << 8) | (unsigned)i;
            }
        }
        if (r > 128) wave_sort<4>(key);
        else wave_sort<2>(key);
        if (lane == 0) C.price[turn * DP_NW + wave] = price;
        // Prefixes of the order.  Loads that share a key lie in any order: the sum of the k first is that of the k least but for
        // less than k steps, and with r steps more room no size that fits is lost (less than 1 while r loads are below 2^24).
        const u64 room_sizes = (u64)M + (by_load ? (u64)(step * (double)r) : 0);
        u64 sum_w[4], sum_v[4], cw = 0, cv = 0, best = ~0ull;
        int fits = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (64 * e < r) {
                const int i = 64 * e + lane, who = (int)(key[e] & (CORE_N - 1));
                const unsigned own_w = i < r ? C.load[who] : 0, own_v = i < r ? C.value[who] : 0;
                double v, w;
                if (wide) {
                    sum_w[e] = wave_scan_u64((u64)own_w) + cw;
                    sum_v[e] = wave_scan_u64((u64)own_v) + cv;
                    w = (double)sum_w[e], v = (double)sum_v[e];
                    cw = lane_value_u64(sum_w[e], 63);
                    cv = lane_value_u64(sum_v[e], 63);
                } else {
                    const unsigned w32 = wave_scan_u32(own_w) + (unsigned)cw, v32 = wave_scan_u32(own_v) + (unsigned)cv;
                    w = (double)w32, v = (double)v32;
                    sum_w[e] = w32, sum_v[e] = v32;
                    cw = (unsigned)__builtin_amdgcn_readlane((int)w32, 63);
                    cv = (unsigned)__builtin_amdgcn_readlane((int)v32, 63);
                }
                const bool fit = i < r && sum_w[e] <= (u64)M;
                fits += __popcll(__builtin_amdgcn_ballot_w64(i < r && sum_w[e] <= room_sizes));
                if (i < r) {
                    C.at[wave][i] = (unsigned char)who;
                    const double b = v + price * (w - (double)M) - margin * (v + price * w) - step * (double)(i + 1);
                    C.bound[wave][i] = b;
                    if (b > 0.0 && !by_load)
                        atomicMax(&C.best_bound[i], ((u64)__double_as_longlong(b) & ~63ull) | (unsigned)(turn * DP_NW + wave));
                    if (fit) best = min(best, set_key(v, i + 1, C.per_square[i]));
                }
            }
        }
        best = wave_min_u64(best);
        if (lane == 0) {
            atomicMin(&C.best_key, best);
            if (by_load) C.fits = fits;
        }
        __syncthreads();
        bk = (int)(C.best_key & 4095);
        if (bk < 1 || bk > r) return false;  // cannot happen: a single request fits
        const int from = (int)(C.best_bound[bk - 1] & 63);
        if (turn == 0) {
            centre = C.price[from];
            if (!(centre > 0.0)) centre = scale * (double)exp2f(0.7655f * -10.0f);
            __syncthreads();
            continue;
        }
        // Better sets from the prefixes of one order about the longest that fits.  First of the order whose bound is the best:
        // one request more, or one exchanged (a lane for each of the 64 requests behind, four wavefronts for the 64 before).  Then of
        // one between the sizes' best: any choice from the CORE_WINDOW requests about its end.
        if (wave == (from >= DP_NW && turn == 1 ? from - DP_NW : DP_NW / 2)) {
            C.sorted[lane] = make_int2(-1, -1);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 64 * e + lane;
                if (i < r) {
                    C.sum_load[i] = (long long)sum_w[e];
                    C.sum_value[i] = (long long)sum_v[e];
                    C.sorted[64 + i] = make_int2(C.load[key[e] & (CORE_N - 1)], C.value[key[e] & (CORE_N - 1)]);
                }
            }
            C.sorted[64 + r + lane] = make_int2(INT_MAX, INT_MAX);
            if (lane == 0) C.prefix = fits;
        }
        __syncthreads();
        best = ~0ull;
        if (turn == 1) {
            const int k = C.prefix - 1 + (wave >> 2);
            if (k >= 1 && k <= r) {
                const long long room = (long long)M - C.sum_load[k - 1], sum = C.sum_value[k - 1];
                const int2 more = C.sorted[64 + k + lane];
                if (more.x <= room) best = set_key((double)(sum + more.y), k + 1, C.per_square[k]);  // (k < r here)
                const int need = (int)min((long long)INT_MAX, (long long)more.x - room);
                int dearest = -1;  // value of the dearest request that makes room
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int2 less = C.sorted[k + 16 * (wave & 3) + i];
                    if (less.x >= need) dearest = max(dearest, less.y);
                }
                if (more.x != INT_MAX && dearest >= 0) best = min(best, set_key((double)(sum + more.y - dearest), k, C.per_square[k - 1]));
            }
        } else {
            const int a = max(0, min(C.prefix - CORE_WINDOW / 2, r - CORE_WINDOW)), members = a + __popc(tid);
            double w = a > 0 ? (double)C.sum_load[a - 1] : 0.0, v = a > 0 ? (double)C.sum_value[a - 1] : 0.0;
#pragma unroll
            for (int b = 0; b < 10; ++b) {
                const int2 q = C.sorted[64 + a + CORE_WINDOW - 10 + b];
                if ((tid >> b) & 1) w += (double)q.x, v += (double)q.y;
            }
            double few_w[1 << (CORE_WINDOW - 10)], few_v[1 << (CORE_WINDOW - 10)];
            few_w[0] = w, few_v[0] = v;
#pragma unroll
            for (int g = 0; g < 1 << (CORE_WINDOW - 10); ++g) {
                if (g > 0) {
                    const int2 q = C.sorted[64 + a + __builtin_ctz(g)];
                    few_w[g] = few_w[g & (g - 1)] + (double)q.x;
                    few_v[g] = few_v[g & (g - 1)] + (double)q.y;
                }
                const int k = members + __builtin_popcount(g);
                if (k > 0 && k <= r && few_w[g] <= (double)M) best = min(best, set_key(few_v[g], k, C.per_square[k - 1]));
            }
        }
        best = wave_min_u64(best);
        if (lane == 0) atomicMin(&C.best_key, best);
        __syncthreads();
        best = C.best_key;
        bk = (int)(best & 4095);
        F = __longlong_as_double((long long)(best | 4095)) * (1.0 + margin);
        if (turn == 1) {
            // sizes left, and the range of their prices
            const bool left = tid < r && tid < C.fits && __longlong_as_double((long long)(C.best_bound[tid] & ~63ull)) <= F * (double)(tid + 1) * (double)(tid + 1);
            const int at = place_of(left, C, 0, sizes);
            if (sizes > CORE_SIZES) return false;
            if (left) C.size[at] = tid + 1;
#pragma unroll 1
            for (int i = tid; i < CORE_SIZES * CORE_N / 8; i += DP_T)
                reinterpret_cast<u64 *>(&C.out[0][0])[i] = reinterpret_cast<u64 *>(&C.in[0][0])[i] = 0;
            __syncthreads();
            double lo = C.price[C.best_bound[bk - 1] & 63], hi = lo;
#pragma unroll 1
            for (int a = 0; a < sizes; ++a) {
                const double p = C.price[C.best_bound[C.size[a] - 1] & 63];
                lo = fmin(lo, p);
                hi = fmax(hi, p);
            }
            if (!(hi > 0.0)) hi = centre;
            lo = fmax(lo, hi * 0.125);
            low = lo * 0.93;
            ratio = (double)__log2f((float)(hi * 1.08 / low));
            continue;
        }
        // requests that are in or out, by this wavefront's price
        double c[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (64 * e + lane < r) c[e] = (double)C.value[64 * e + lane] + price * (double)C.load[64 * e + lane];
#pragma unroll 1
        for (int a = 0; a < sizes; ++a) {
            const int k = C.size[a];
            const double limit = F * (double)k * (double)k, b = C.bound[wave][k - 1];
            const int last = C.at[wave][k - 1];
            const double c_last = (double)C.value[last] + price * (double)C.load[last];
            double c_next = 1e300;
            if (k < r) {
                const int next = C.at[wave][k];
                c_next = (double)C.value[next] + price * (double)C.load[next];
            }
            if (lane == 0 && b > limit) C.dead[a] = 1;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = 64 * e + lane;
                if (i < r) {
                    if (b + fmax(0.0, c[e] - c_last - step) * (1.0 - margin) > limit) C.out[a][i] = 1;
                    if (c[e] <= c_last && b + fmax(0.0, c_next - c[e] - step) * (1.0 - margin) > limit) C.in[a][i] = 1;
                }
            }
        }
        __syncthreads();
    }
    // ---- what is decided
    bool out = sizes != r, in = out;
#pragma unroll 1
    for (int a = 0; a < sizes; ++a) {
        if (C.dead[a]) continue;
        if (tid < r) out &= C.out[a][tid] != 0, in &= C.in[a][tid] != 0;
    }
    const bool sure = tid < r && in && !out, open = tid < r && !out && !in;
    if (tid < CORE_N) {
        const int members = __popcll(__builtin_amdgcn_ballot_w64(sure));
        const u64 v = wave_scan_u64(sure ? (u64)value : 0), w = wave_scan_u64(sure ? (u64)load : 0);
        if (lane == 63) {
            atomicAdd(&C.sure[0], members);
            atomicAdd(&C.sure[1], (int)(unsigned)v);
            atomicAdd(&C.sure[2], (int)(unsigned)w);
        }
    }
    int undecided;
    const int bit = place_of(open, C, 1, undecided);
    if (undecided > CORE_MAX) return false;
    if (open) C.undecided[bit] = make_int2(load, value);
    const int hi_bits = min(undecided, CORE_MAX / 2), lo_bits = undecided - hi_bits;
    if (tid <= CORE_MAX / 2 + 1) {
        int first = 0;
#pragma unroll
        for (int j = 0; j <= CORE_MAX / 2; ++j) {
            const int c = C.over[lo_bits][j];
            first += j < tid ? c : 0;
        }
        C.first[tid] = first;
    }
    __syncthreads();
    const int k0 = C.sure[0], v0 = C.sure[1], room = M - C.sure[2];
    if (room < 0) return false;  // cannot happen
    // ---- all combinations of the rest: a thread for each of its ten last requests', the others' from a table by number of
    // members and in ascending order.
    // Loads stop at room + 1 (M < 2^30, or the tables would be refused).
    if (tid < (1 << lo_bits)) {
        int w = 0, rank = 0, j = 0;
        unsigned v = 0;
#pragma unroll 1
        for (int b = 0; b < lo_bits; ++b) {
            if ((tid >> b) & 1) {
                w = min(w + C.undecided[b].x, room + 1);
                v += (unsigned)C.undecided[b].y;
                rank += C.over[b][++j];
            }
        }
        const int at = C.first[j] + rank;
        C.low[at] = make_int2(w, (int)v);
        C.low_set[at] = (unsigned short)tid;
    }
    int hi_load = 0;
    unsigned hi_value = 0;
    const int hi_members = __popc(tid);
#pragma unroll
    for (int b = 0; b < CORE_MAX / 2; ++b) {
        const int2 q = C.undecided[min(lo_bits + b, CORE_MAX - 1)];
        if (b < hi_bits && ((tid >> b) & 1)) {
            hi_load = min(hi_load + q.x, room + 1);
            hi_value += (unsigned)q.y;
        }
    }
    __syncthreads();
    // The best key (value, load) of each size; then, of the best size, the least combination that has it.
    auto combinations = [&](int size, auto &&use) {
        const int low_members = size - k0 - hi_members;
        if (tid < (1 << hi_bits) && low_members >= 0 && low_members <= lo_bits) {
            const int behind = C.first[low_members + 1];
#pragma unroll 2
            for (int x = C.first[low_members]; x < behind; ++x) {
                const int w = hi_load + C.low[x].x;
                if (w <= room) use(x, ((unsigned long long)(hi_value + (unsigned)C.low[x].y) << 32) | (unsigned)w);
            }
        }
    };
#pragma unroll 1
    for (int a = 0; a < sizes; ++a) {
        if (C.dead[a] || 64 * wave >= (1 << hi_bits)) continue;
        unsigned long long best = ~0ull;
        combinations(C.size[a], [&](int, unsigned long long key) { best = min(best, key); });
        best = wave_min_u64(best);
        if (lane == 0) atomicMin(&C.best_of[a], best);
    }
    __syncthreads();
    long long S = 0;
    int k = 0, m = 0;
    unsigned long long least = 0;
#pragma unroll 1
    for (int a = 0; a < sizes; ++a) {
        const unsigned long long key = C.best_of[a];
        if (key == ~0ull) continue;
        const long long total = (long long)v0 + (long long)(key >> 32);
        if (dp_better(total, C.size[a], (int)(unsigned)key, S, k, m, tie_rule)) S = total, k = C.size[a], m = (int)(unsigned)key, least = key;
    }
    if (k < 1) return false;  // cannot happen
    if (F > 0.0 && (double)S * C.per_square[k - 1] > F) return false;  // cannot happen: a set that was met is better
    int own = INT_MAX;
    combinations(k, [&](int x, unsigned long long key) {
        if (key == least && own == INT_MAX) own = (tid << lo_bits) | C.low_set[x];
    });
    if (own != INT_MAX) atomicMin(&C.subset, own);
    __syncthreads();
    // ---- members
    const bool member = sure || (open && ((C.subset >> bit) & 1));
    const int id = tid < r ? C.id[tid] : 0;
    int kept;
    const int to = place_of(tid < r && !member, C, 0, kept);
    if (r - kept != k) return false;  // cannot happen
    if (member) batch_of[id] = nb;
    if (tid == 0) publish_batch(S, k, gb, n - r, nb, batch_end_out, F_out, words);
    if (tid < r && !member) C.id[to] = id, C.value[to] = value, C.load[to] = load;
    r = kept;
    __syncthreads();
    return true;
}

// The batches from number nb on, as far as no table is needed: lists as left by the kernels below (listed: otherwise those
// by cost and by o of what remains are still to be made).  What remains is planned and reported to the host; behind the
// last batch the order is written.
template <bool SEARCH>
__device__ __forceinline__ void go_on(int32_t n, int r, int kmax, bool listed, int32_t nb, const int32_t *s, const int32_t *o, int32_t M,
                                      int32_t ga, int32_t gb, int32_t feas_mode, int32_t tie_rule, bool search, int *proc, int *by_o,
                                      int *by_cost, int *buf0, int *buf1, int *batch_of, int *left_by_o, int *cost, int4 *req,
                                      int2 *range, int32_t *order_out, int32_t *batch_end_out, double *F_out,
                                      int32_t *num_batches_out, int32_t *words, int32_t *host, int32_t seq, HelperLds &L,
                                      CoreLds *core)
{
    const int tid = threadIdx.x, before = r;
    if constexpr (SEARCH) {
        if (search && r > 0 && r <= CORE_N) {
            CoreLds &C = *core;
            if (tid < r) {
                const int id = proc[tid], sv = s[id], ov = o[id];
                C.id[tid] = id;
                C.value[tid] = ga * sv + gb * ov;
                C.load[tid] = sv + ov;
            }
            core_start(C);
            __syncthreads();
            while (r > 0 && core_batch(r, M, gb, tie_rule, n, nb, batch_of, batch_end_out, F_out, words, C)) ++nb;
            __threadfence_block();
            __syncthreads();
        }
    }
    int kmin = 0;
    if (r == 0) {
        kmax = 0;
        emit_body(n, by_o, buf0, buf1, batch_of, nb, order_out, num_batches_out, L);
    } else {
        if (!listed) {  // (of up to CORE_N requests, in which case none had left before this call)
            for (int i = tid; i < before; i += DP_T) {
                buf0[i] = i;
                left_by_o[i] = by_o[i];
            }
            __threadfence_block();
            __syncthreads();
            rank_sort(buf0, by_cost, before, [s, o, feas_mode](int id) { return cost_of(s[id], o[id], feas_mode); }, L);
            __threadfence_block();
            __syncthreads();
        }
        if (!listed || r < before) compact_body(proc, by_cost, left_by_o, buf0, before, batch_of, s, o, feas_mode, M, L, r, kmax);
        kmin = bounds_body(by_cost, left_by_o, kmax, s, o, M, ga, gb, feas_mode, cost, L);
        plan_body(proc, r, kmin, kmax, s, o, M, ga, gb, feas_mode, cost, req, range);
    }
    __syncthreads();
    if (tid == 0) tell_host(words, host, seq, r, kmax, kmin, nb);
}

__host__ __device__ __forceinline__ size_t counted_bytes(int32_t r, int32_t kmax, int32_t M)
{
    const size_t loads = ((size_t)M + 256) & ~(size_t)255;
    return 2 * (size_t)(kmax + 1) * loads * sizeof(int) + (size_t)r * (size_t)(kmax + 1) * (loads / 8) + 6400;
}

// (pad: zeros in all of batch_end_out and F_out first.  SEARCH: with the batches that need no table, under the sum of peaks; the code of
// the search is five times that of the rest, which costs the profile constraint, where there is none, 6 % of a call.)
template <bool SEARCH>
__global__ __launch_bounds__(DP_T) void dp_prepare_kernel(int32_t n, const int32_t *s, const int32_t *o, int32_t M,
                                                          int32_t ga, int32_t gb, int32_t feas_mode, int32_t tie_rule, int32_t pad,
                                                          int *proc, int *by_o, int *by_cost, int *buf0, int *buf1, int *batch_of,
                                                          int *left_by_o, int *cost, int4 *req, int2 *range, size_t most_bytes,
                                                          int32_t *order_out, int32_t *batch_end_out, double *F_out,
                                                          int32_t *words, int32_t *num_batches_out, int32_t *host, int32_t seq)
{
    __shared__ HelperLds L;
    __shared__ char core[SEARCH ? sizeof(CoreLds) : 1] __attribute__((aligned(16)));
    if (pad)
        for (int i = threadIdx.x; i < n; i += DP_T) batch_end_out[i] = 0, F_out[i] = 0.0;
    // Sizes that are refused are refused whether or not a table would have been needed: where no bound on the batch size
    // leads to a refusal, it and the lists it takes are made when a table is needed (5 us of 200 requests).
    const bool listed = !SEARCH || n > CORE_N || counted_bytes(n, n, M) > most_bytes;
    const int kmax = prepare_body(n, s, o, M, feas_mode, proc, by_o, by_cost, buf0, buf1, batch_of, words,
                                  num_batches_out, L, listed);
    if (kmax < 0) {
        if (threadIdx.x == 0) tell_host(words, host, seq, 0, 0, 0, 0);
        return;
    }
    if (listed)
        for (int i = threadIdx.x; i < n; i += DP_T) left_by_o[i] = by_o[i];
    __threadfence_block();
    __syncthreads();
    go_on<SEARCH>(n, n, kmax, listed, 0, s, o, M, ga, gb, feas_mode, tie_rule, !listed || counted_bytes(n, kmax, M) <= most_bytes, proc, by_o,
          by_cost, buf0, buf1, batch_of, left_by_o, cost, req, range, order_out, batch_end_out, F_out, num_batches_out, words, host,
          seq, L, reinterpret_cast<CoreLds *>(core));
}

// The end of a batch: its best state from the rows' (partial[k - kmin]), its members, and how it goes on.
template <bool SEARCH>
__global__ __launch_bounds__(DP_T) void dp_finish_kernel(const unsigned long long *partial, const unsigned long long *bits,
                                                         int *proc, int *by_o, int *by_cost, int *left_by_o, int *buf0, int *buf1, int *batch_of,
                                                         int *cost, int4 *req, int2 *range, int32_t n, int r, int kmin, int kmax, int Mp, const int32_t *s,
                                                         const int32_t *o, int32_t M, int32_t ga, int32_t gb,
                                                         int32_t feas_mode, int32_t tie_rule, int32_t nb, int32_t *order_out,
                                                         int32_t *batch_end_out, double *F_out, int32_t *num_batches_out, int32_t *words,
                                                         int32_t *host, int32_t seq)
{
    __shared__ HelperLds L;
    __shared__ char core[SEARCH ? sizeof(CoreLds) : 1] __attribute__((aligned(16)));
    __shared__ int load[KVSCHED_EXACT_MAX_N];
    long long bS = 0;
    int bk = 0, bm = 0;
    for (int k = kmin + threadIdx.x; k <= kmax; k += DP_T) {
        const unsigned long long v = partial[k - kmin];
        const unsigned S = (unsigned)(v >> 32);
        if (S < DP_NONE && dp_better(S, k, (int)(unsigned)v, bS, bk, bm, tie_rule)) bS = S, bk = k, bm = (int)(unsigned)v;
    }
    for (int t = threadIdx.x; t < r; t += DP_T) load[t] = req[t].x;
    reduce_best(tie_rule, L, bS, bk, bm);
    if (threadIdx.x == 0) publish_batch(bS, bk, gb, n - r, nb, batch_end_out, F_out, words);
    __syncthreads();
    if (threadIdx.x < 64) walk_body(bits, proc, r, kmax, Mp, load, nb, batch_of, bk, bm);
    __threadfence_block();
    __syncthreads();
    int kept, knext;
    compact_body(proc, by_cost, left_by_o, buf0, r, batch_of, s, o, feas_mode, M, L, kept, knext);
    go_on<SEARCH>(n, kept, knext, true, nb + 1, s, o, M, ga, gb, feas_mode, tie_rule, true, proc, by_o, by_cost, buf0, buf1, batch_of, left_by_o, cost, req,
          range, order_out, batch_end_out, F_out, num_batches_out, words, host, seq, L, reinterpret_cast<CoreLds *>(core));
}

// The whole Phase 1 in one workgroup when both tables fit in LDS (the settings Algorithm 2 is meant
// for: about a hundred requests, M of a few hundred to a few thousand): no launch per request and
// no host round trip per batch.  Row length Mp = 2^lg >= M + 1; the records still go to global
// memory.  Same arithmetic and the same order of updates as the kernels above.
//
// Bound by the instructions of one compute unit, whose sixteen wavefronts take 64 states a turn: so two requests are offered at a
// time (four states read, one written, for each state; four requests would read sixteen), a wavefront's row and part of it
// are scalars that step from turn to turn, only parts that hold loads up to M are visited, and a turn's records wait in a lane each
// until the step's end, where one store takes all.  The barrier of a step is for LDS alone.  1620 cycles for two requests of 30 rows
// of 101 loads (2320 with one request a step, every state computing its place); of a batch of 105 requests the walk back takes a
// third as long as all steps, the best state and the lists 9 % each.  200 requests of lengths up to 8, M = 100 1303 -> 1022 us; 100 of
// them 382 -> 307, under the profile 423 -> 375; 60 176 -> 145 and 179 -> 159; 30, M = 60 94 -> 85.
constexpr int DP_SMALL_STATES = 12288;  // (kmax + 1) * Mp at most; two int tables = 96 KB of LDS
constexpr int DP_SMALL_N = 1024;
static_assert(DP_SMALL_STATES / 64 <= 64 * DP_NW, "a lane per turn");

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// A barrier for what is in LDS alone: the records on their way to memory are not waited for.
__device__ __forceinline__ void tables_written() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Lane l (the same in all lanes) of the four becomes a's and b's halves.
__device__ __forceinline__ void keep(unsigned (&to)[4], unsigned long long a, unsigned long long b, int l)
{
    const bool here = (int)(threadIdx.x & 63) == l;
    to[0] = here ? (unsigned)a : to[0];
    to[1] = here ? (unsigned)(a >> 32) : to[1];
    to[2] = here ? (unsigned)b : to[2];
    to[3] = here ? (unsigned)(b >> 32) : to[3];
}

typedef __attribute__((address_space(3))) const unsigned lds_word;

__global__ __launch_bounds__(DP_T) void dp_small_kernel(int32_t n, const int32_t *s, const int32_t *o, int32_t M,
                                                        int32_t ga, int32_t gb, int32_t feas_mode, int32_t tie_rule, int lg, int *proc, int *by_o,
                                                        int *by_cost, int *buf0, int *buf1, int *batch_of,
                                                        unsigned long long *bits, int32_t *order_out,
                                                        int32_t *batch_end_out, double *F_out, int32_t *num_batches_out,
                                                        int32_t *words)
{
    __shared__ HelperLds L;
    __shared__ unsigned tab[2][DP_SMALL_STATES + 1];  // (the last entry says "no set")
    __shared__ int req_o[DP_SMALL_N], req_load[DP_SMALL_N], req_g[DP_SMALL_N];
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int Mp = 1 << lg;
    int kmax = prepare_body(n, s, o, M, feas_mode, proc, by_o, by_cost, buf0, buf1, batch_of, words, num_batches_out, L);
    if (kmax < 0) return;
    int r = n, nb = 0;
    while (r > 0) {
        kmax = uniform(kmax);
        r = uniform(r);
        if (((kmax + 1) << lg) > DP_SMALL_STATES) {  // excluded by the host's choice of this kernel
            if (tid == 0) atomicOr(&words[KVS_W_STATUS], KVSCHED_DEV_BAD_LENGTH);
            break;
        }
        const int states = (kmax + 1) << lg;
        for (int i = tid; i < states; i += DP_T) {
            const unsigned v = i == 0 ? 0 : DP_NONE;
            tab[0][i] = v;
            tab[1][i] = v;
        }
        if (tid < 2) tab[tid][DP_SMALL_STATES] = DP_NONE;
        for (int t = tid; t < r; t += DP_T) {
            const int id = proc[t];
            req_o[t] = o[id];
            req_load[t] = feas_mode ? s[id] : s[id] + o[id];
            req_g[t] = ga * s[id] + gb * o[id];
        }
        __syncthreads();
        const size_t per_t = (size_t)(kmax + 1) << (lg - 6);
        const int parts = uniform((M >> 6) + 1);  // of a row, 64 loads each, that hold states
        const int k_step = uniform(DP_NW / parts), part_step = DP_NW - k_step * parts;
        const int k_first = uniform(1 + wave / parts), part_first = wave - (k_first - 1) * parts;
        // where the records of this wavefront's turn number `lane` lie
        const int turn = wave + DP_NW * lane, mine = ((1 + turn / parts) << (lg - 6)) + turn % parts;
        const unsigned none = (unsigned)(unsigned long long)(lds_word *)&tab[0][DP_SMALL_STATES];
        const int row = 4 << lg;  // (bytes)
        auto steps = [&](auto profile) __attribute__((always_inline)) {
            constexpr bool PROFILE = decltype(profile)::value;
            for (int t = 0; t < r; t += 2) {
                const bool two = t + 1 < r;
                const int l1 = uniform(req_load[t]), l2 = two ? uniform(req_load[t + 1]) : DP_SMALL_STATES;  // (more than any load)
                const int o1 = PROFILE ? uniform(req_o[t]) : 0, o2 = PROFILE && two ? uniform(req_o[t + 1]) : 0;
                const unsigned g1 = (unsigned)uniform(req_g[t]), g2 = two ? (unsigned)uniform(req_g[t + 1]) : 0;
                const int rows = min(t + 2, kmax);
                const unsigned src = (unsigned)(unsigned long long)(lds_word *)&tab[(t >> 1) & 1][lane];
                unsigned *dst = &tab[((t >> 1) + 1) & 1][lane];
                unsigned rec[4] = {0, 0, 0, 0};  // lane j: the records of turn j
                int turns = 0;
                for (int k = k_first, part = part_first; k <= rows; ++turns) {
                    const int first = (k << lg) + 64 * part, m = 64 * part + lane;
                    const unsigned at = src + 4 * (unsigned)first;
                    // what lacks the first request, the second, both: to be read where its load is one, and under the profile where the
                    // memory at the completions leaves room (o <= M < 2^13 and k <= DP_SMALL_STATES / 64: 32 bits hold it)
                    bool in1 = m >= l1, in2 = m >= l2, in12 = m >= (k > 1 ? l1 + l2 : DP_SMALL_STATES);
                    if (PROFILE) {
                        const int most1 = M - o1 * k, most2 = M - o2 * k, most12 = min(M - o1 * (k - 1) + l2, most2);
                        in1 = in1 && m <= most1;
                        in2 = in2 && m <= most2;
                        in12 = in12 && m <= most12;
                    }
                    const unsigned at1 = in1 ? at - (unsigned)(row + 4 * l1) : none, at2 = in2 ? at - (unsigned)(row + 4 * l2) : none;
                    const unsigned at12 = in12 ? at - (unsigned)(2 * row + 4 * (l1 + l2)) : none;
                    const unsigned f = *(lds_word *)(unsigned long long)at, f1 = *(lds_word *)(unsigned long long)at1 + g1;
                    const unsigned f2 = *(lds_word *)(unsigned long long)at2, f12 = *(lds_word *)(unsigned long long)at12 + g1;
                    const unsigned a = min(f, f1), b = min(f2, f12) + g2;
                    dst[first] = min(a, b);
                    keep(rec, __builtin_amdgcn_ballot_w64(f1 < f), __builtin_amdgcn_ballot_w64(b < a), turns);
                    k += k_step;
                    part += part_step;
                    if (part >= parts) {
                        part -= parts;
                        ++k;
                    }
                }
                if (lane < turns) {
                    bits[(size_t)t * per_t + mine] = (unsigned long long)rec[1] << 32 | rec[0];
                    if (two) bits[(size_t)(t + 1) * per_t + mine] = (unsigned long long)rec[3] << 32 | rec[2];
                }
                tables_written();
            }
        };
        // (one kernel for both: with two of them the compiler calls what it has in place in the kernels above, whose calls then take 1 % longer)
        if (feas_mode) steps(std::true_type());
        else steps(std::false_type());
        long long bS;
        int bk, bm;
        argmin_body(tab[((r + 1) >> 1) & 1], kmax, M, lg, tie_rule, L, bS, bk, bm);
        if (tid == 0) publish_batch(bS, bk, gb, n - r, nb, batch_end_out, F_out, words);
        if (bk < 1) break;  // uniform
        __threadfence_block();
        __syncthreads();
        if (tid < 64) walk_body(bits, proc, r, kmax, Mp, req_load, nb, batch_of, bk, bm);
        __threadfence_block();
        __syncthreads();
        int kept, knext;
        compact_body(proc, by_cost, nullptr, buf0, r, batch_of, s, o, feas_mode, M, L, kept, knext);
        if (kept >= r) break;  // cannot happen: a batch has at least one member; never spin
        r = kept;
        kmax = knext;
        ++nb;
    }
    __syncthreads();
    emit_body(n, by_o, buf0, buf1, batch_of, nb, order_out, num_batches_out, L);
}

bool launched() { return hipGetLastError() == hipSuccess; }

}  // namespace

// Lists of ids (and, last, the sums of the least costs) of a construction over n requests.
struct DpLists {
    int *proc, *by_o, *by_cost, *buf0, *buf1, *batch_of, *left_by_o, *cost;
    int4 *req;
    int2 *range;
};

static DpLists dp_lists(void *lists, int32_t n)
{
    const size_t np = ((size_t)n + 64) & ~(size_t)63;
    int *p = (int *)lists;
    return DpLists{p,          p + np,     p + 2 * np, p + 3 * np, p + 4 * np,
                   p + 5 * np, p + 6 * np, p + 7 * np, (int4 *)(p + 8 * np), (int2 *)(p + 12 * np + 64)};
}

static int dp_row(int32_t M) { return (int)(((size_t)M + DP_STEP_M) & ~(size_t)(DP_STEP_M - 1)); }  // >= M + 1

size_t kvs_exact_dp_list_bytes(int32_t n)
{
    const size_t np = ((size_t)n + 64) & ~(size_t)63;
    return np * 14 * sizeof(int) + 1024;
}

size_t kvs_exact_dp_table_bytes(int32_t r, int32_t kmax, int32_t M)
{
    const size_t Mp = (size_t)dp_row(M);
    return DP_FRONT * sizeof(int) + 2 * (size_t)(kmax + 1) * Mp * sizeof(int) + (size_t)r * (size_t)(kmax + 1) * (Mp / 8) +
           sizeof(long long) * (size_t)(kmax + 1) + 256;
}

// What the limit on the tables is compared with: two tables and the records with the loads counted in 256s, and 6400
// bytes.  (Fixed, so that the sizes that are accepted do not move with the kernels' own rows and working memory: the
// allocation may exceed it by the loads that fill a row of DP_STEP_M.)
size_t kvs_exact_dp_counted_bytes(int32_t r, int32_t kmax, int32_t M) { return counted_bytes(r, kmax, M); }

// (most_bytes: what counted bytes are compared with)
int kvs_launch_exact_dp_prepare(int32_t n, const int32_t *s, const int32_t *o, int32_t M, int32_t ga, int32_t gb,
                                int32_t feas_mode, int32_t tie_rule, int pad, size_t most_bytes, void *lists,
                                int32_t *order_out, int32_t *batch_end_out, double *F_out, int32_t *d_words,
                                int32_t *num_batches_out, int32_t *host, int32_t seq, hipStream_t st)
{
    const DpLists l = dp_lists(lists, n);
    hipLaunchKernelGGL(feas_mode == KVSCHED_FEAS_SUM_OF_PEAKS ? dp_prepare_kernel<true> : dp_prepare_kernel<false>, dim3(1), dim3(DP_T), 0, st, n, s, o, M, ga, gb, feas_mode, tie_rule, pad, l.proc, l.by_o,
                       l.by_cost, l.buf0, l.buf1, l.batch_of, l.left_by_o, l.cost, l.req, l.range, most_bytes, order_out, batch_end_out,
                       F_out, d_words, num_batches_out, host, seq);
    return launched() ? KVSCHED_OK : KVSCHED_EHIP;
}

// One batch over the r remaining requests: tables, records, best state, members, compaction.
int kvs_launch_exact_dp_batch(int32_t n, int32_t r, int32_t kmin, int32_t kmax, const int32_t *s, const int32_t *o,
                              int32_t M, int32_t ga, int32_t gb, int32_t feas_mode, int32_t tie_rule, int32_t nb, bool search,
                              void *lists, void *tables, int32_t *order_out, int32_t *batch_end_out, double *F_out,
                              int32_t *num_batches_out, int32_t *d_words, int32_t *host, int32_t seq, hipStream_t st)
{
    const DpLists l = dp_lists(lists, n);
    const int Mp = dp_row(M);
    const size_t table = (size_t)(kmax + 1) * Mp, words = DP_FRONT + 2 * table;
    unsigned *none = (unsigned *)tables;
    unsigned *dp[2] = {none + DP_FRONT, none + DP_FRONT + table};
    unsigned long long *bits = (unsigned long long *)(none + words);
    const size_t per_t = (size_t)(kmax + 1) * (Mp >> 6);
    hipLaunchKernelGGL(dp_init_kernel, dim3((unsigned)((words + DP_STEP_T - 1) / DP_STEP_T)), dim3(DP_STEP_T), 0, st,
                       none, words, table);
    const DpPlan plan{l.req, l.range};
    int at = 0;
    for (int32_t t = 0; t < r; t += DP_G, at ^= 1) {
        const int behind = t + DP_G < r ? t + DP_G : r;  // requests offered when this launch is done
        const int top = behind < kmax ? behind : kmax;   // no set is larger
        // the launch has to leave every row that a set of kmin can still be reached from, after each of its requests
        const int first = kmin - (r - t) + 1 > 1 ? kmin - (r - t) + 1 : 1;
        const dim3 grid((unsigned)(Mp / DP_STEP_M), (unsigned)(top - first + 1));
        if (feas_mode)
            hipLaunchKernelGGL((dp_step_kernel<1>), grid, dim3(DP_STEP_T), 0, st, plan, t, r, M, none, dp[at], dp[at ^ 1],
                               bits, per_t, Mp, first);
        else
            hipLaunchKernelGGL((dp_step_kernel<0>), grid, dim3(DP_STEP_T), 0, st, plan, t, r, M, none, dp[at], dp[at ^ 1],
                               bits, per_t, Mp, first);
    }
    unsigned long long *partial = bits + (size_t)r * per_t;
    hipLaunchKernelGGL(dp_argmin_rows_kernel, dim3((unsigned)(kmax - kmin + 1)), dim3(DP_T), 0, st, dp[at], kmin, Mp,
                       plan, partial);
    hipLaunchKernelGGL(search && feas_mode == KVSCHED_FEAS_SUM_OF_PEAKS ? dp_finish_kernel<true> : dp_finish_kernel<false>, dim3(1), dim3(DP_T), 0, st, partial, bits, l.proc, l.by_o, l.by_cost, l.left_by_o, l.buf0, l.buf1,
                       l.batch_of, l.cost, l.req, l.range, n, r, kmin, kmax, Mp, s, o, M, ga, gb, feas_mode, tie_rule, nb, order_out,
                       batch_end_out, F_out, num_batches_out, d_words, host, seq);
    return launched() ? KVSCHED_OK : KVSCHED_EHIP;
}

// Can the one-workgroup kernel take this problem?  kmax_bound: any bound on the batch size.
// Returns log2 of its row length, or 0.
int kvs_exact_dp_small_lg(int32_t n, int32_t kmax_bound, int32_t M)
{
    if (n > DP_SMALL_N) return 0;
    int lg = 6;
    while (((int64_t)1 << lg) < (int64_t)M + 1) ++lg;
    if (lg > 13) return 0;
    return (((int64_t)kmax_bound + 1) << lg) <= DP_SMALL_STATES ? lg : 0;
}

size_t kvs_exact_dp_small_record_bytes(int32_t n, int32_t kmax_bound, int lg)
{
    return (size_t)n * ((size_t)(kmax_bound + 1) << (lg - 6)) * sizeof(unsigned long long) + 256;
}

int kvs_launch_exact_dp_small(int32_t n, const int32_t *s, const int32_t *o, int32_t M, int32_t ga, int32_t gb,
                              int32_t feas_mode, int32_t tie_rule, int lg, void *lists, void *records, int32_t *order_out,
                              int32_t *batch_end_out, double *F_out, int32_t *num_batches_out, int32_t *d_words,
                              hipStream_t st)
{
    const DpLists l = dp_lists(lists, n);
    hipLaunchKernelGGL(dp_small_kernel, dim3(1), dim3(DP_T), 0, st, n, s, o, M, ga, gb, feas_mode, tie_rule, lg, l.proc, l.by_o,
                       l.by_cost, l.buf0, l.buf1, l.batch_of, (unsigned long long *)records, order_out, batch_end_out, F_out,
                       num_batches_out, d_words);
    return launched() ? KVSCHED_OK : KVSCHED_EHIP;
}
