// Sorted-F order construction: Phase 1 of Algorithm 1 ("Batch Construction") with the batch
// taken among the feasible prefixes of the remaining requests sorted by (s+o, o, id), scored
// by the F-metric of Section 4, F(X) = sum o_i / |X|^2, or by the generalised metric of Section 7
// ("Robustness to prefill weighting"), G(X) = sum (alpha s_i + o_i) / |X|^2 with alpha = ga / gb: the
// effective length ga s_i + gb o_i replaces o_i in the metric's numerator, nowhere else.
//
// Since every batch is a prefix of what remains, the remaining requests stay sorted: one key
// sort serves all batches, and batch b is the segment [a_b, a_b + k*) of the sorted array:
//   1. sort 64-bit keys (s+o, o, id); keys that do not fit in 64 bits (budgets beyond some 2^22 with
//      many requests: the host decides from M and n) are replaced by (s+o, rank in the (o, id) order)
//   2. prefix sums W (of s+o), S (of o) and G (of the effective lengths) over that order
//   3. per batch: the feasible extent K (sum of peaks <= M; or the simultaneous-start memory profile),
//      then the argmin over k <= K of G_k / k^2 compared in exact integers, tie rule applied
//   4. sort (batch, o, id): each batch in nondecreasing o; the metric as one fp64 division
// Up to 1024 requests (128 under the profile constraint) one workgroup does everything in LDS and
// registers; beyond that the sorts and scans are launches over the whole chip and only step 3, a chain
// by nature, is one workgroup's.
#include "device_util.h"
#include "phase1_util.h"
#include "sort_util.h"

#include <type_traits>

namespace {

constexpr int kRun = 2048;          // keys one workgroup sorts (1024 threads, two each)
constexpr int kFan = 8;             // runs merged by one pass
constexpr int kSmallSum = 1024, kSmallProfile = 128;  // requests that one workgroup takes (kvs_sortedF_small_max)
// Requests whose places, and order within a batch, are found by counting the keys before them.  (Sorted runs and counting, us a call: chat requests, budgets of
// 60 tokens a request 13000 94 79, 16384 102 94; of 300, so that one batch holds most of them, 13000 91 89, 14000 92 94, 15000 97 98, 16000 95 101,
// 16384 94 105; mixed ones of 300 13000 96 87, 16384 98 98; lengths up to 4000 and 2000 16384 102 89.)
constexpr int kCountMax = 16384;
constexpr int kSumsHere = 16384;    // requests up to which the prefix sums need no sums ahead
constexpr int kOrderTile = 6144;    // keys held at a time when the places within batches are counted
constexpr int kNextMax = 256;       // profile tests among the first so many requests are made by one wavefront
constexpr int kNextLimit = 2048;    // batches whose extent is below this are found for all places at once
constexpr int kNextWindow = 73728;  // places of which the chain holds what is known in LDS (two bytes each)
constexpr int kSmallBuckets = 2048; // completion-time buckets of the profile test in LDS
constexpr int kLargeBuckets = 4096;

struct SortedArgs {
    int32_t n;
    const int32_t *s, *o;
    int32_t M, ga, gb, tie_rule;
    int32_t *order_out, *batch_end_out;
    double *F_out;
    int32_t *num_batches_out;
    int32_t *words;
    int32_t id_bits, o_bits;  // key fields: (s+o) above o_bits bits of o above id_bits bits of the id
    int32_t packed;           // 0: the keys would not fit, (s+o, rank by (o, id)) instead
    int32_t pad;              // zeros behind the last batch in batch_end_out / F_out
};

// Arrays by sorted position (LDS or scratch), shared by both variants.
struct Sums {
    const u64 *W, *S, *G;  // [n + 1]
    const int *s, *o;      // [n] (profile constraint only)
};

// sign of Sa/ka^2 - Sb/kb^2 in exact integers (Sa, Sb < 2^63; ka, kb < 2^31)
__device__ __forceinline__ int cmp_F(u64 Sa, int ka, u64 Sb, int kb)
{
    const u64 qa = (u64)ka * (u64)ka;
    const u64 qb = (u64)kb * (u64)kb;
    const u64 l_hi = __umul64hi(Sa, qb), l_lo = Sa * qb;
    const u64 r_hi = __umul64hi(Sb, qa), r_lo = Sb * qa;
    if (l_hi != r_hi) return l_hi < r_hi ? -1 : 1;
    if (l_lo != r_lo) return l_lo < r_lo ? -1 : 1;
    return 0;
}

// is prefix (Sa, ka) a better batch than (Sb, kb)?  k == 0 means "none".  SMALL: every S < 2^32 and
// every k < 2^16, so both cross products fit in 64 bits.
template <bool SMALL>
__device__ __forceinline__ bool better(u64 Sa, int ka, u64 Sb, int kb, int tie_rule)
{
    if constexpr (SMALL) {
        const u64 l = (u64)(unsigned)Sa * ((unsigned)kb * (unsigned)kb);
        const u64 r = (u64)(unsigned)Sb * ((unsigned)ka * (unsigned)ka);
        const bool wins = l != r ? l < r : (tie_rule == KVSCHED_TIE_LARGER ? ka > kb : ka < kb);
        return ka != 0 && (kb == 0 || wins);
    } else {
        if (ka == 0) return false;
        if (kb == 0) return true;
        const int c = cmp_F(Sa, ka, Sb, kb);
        if (c != 0) return c < 0;
        return tie_rule == KVSCHED_TIE_LARGER ? ka > kb : ka < kb;
    }
}

// The best (S, k) of the 64 lanes' own, k in every lane (0: no lane has one); S of it in bS.  A float quotient
// (good to a few 1e-7) leaves nearly always one lane; only lanes within 4e-6 of the least are compared exactly.
template <bool SMALL>
__device__ __forceinline__ int wave_best(u64 &bS, int bk, int tie_rule)
{
    const float kf = (float)bk;
    const float f = bk > 0 ? (SMALL ? (float)(unsigned)bS : (float)bS) * __builtin_amdgcn_rcpf(kf * kf) : 3.0e38f;
    const float least = __uint_as_float(wave_min_u32(__float_as_uint(f)));
    u64 near = __builtin_amdgcn_ballot_w64(bk > 0 && f <= least * 1.000004f);
    if (near == 0) return 0;
    int at = __ffsll((long long)near) - 1;
    u64 S = lane_value_u64(bS, at);
    int k = __builtin_amdgcn_readlane(bk, at);
    near &= near - 1;
    while (near != 0) {
        at = __ffsll((long long)near) - 1;
        near &= near - 1;
        const u64 So = lane_value_u64(bS, at);
        const int ko = __builtin_amdgcn_readlane(bk, at);
        if (better<SMALL>(So, ko, S, k, tie_rule)) S = So, k = ko;
    }
    bS = S;
    return k;
}

// One wavefront: size of the batch that starts at place a (0: none).  Feasible are the k <= rem with W_k - W_0 <= M.  First the sizes
// up to 64, where most batches end, then 256 a turn, their sums read together.
template <bool SMALL>
__device__ __forceinline__ int wave_batch(const Sums &c, int a, int rem, u64 M, int tie_rule)
{
    const int lane = threadIdx.x & 63;
    const u64 W0 = c.W[a], G0 = c.G[a];
    const int k1 = min(lane + 1, rem);
    const u64 w1 = c.W[a + k1], g1 = c.G[a + k1];
    const bool ok1 = lane < rem && w1 - W0 <= M;
    u64 bS = ok1 ? g1 - G0 : 0;
    int bk = ok1 ? lane + 1 : 0;
    if (__builtin_amdgcn_ballot_w64(ok1) != ~0ull) return wave_best<SMALL>(bS, bk, tie_rule);
    for (int base = 64; base < rem; base += 256) {
        u64 w[4], g[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = min(base + 64 * q + lane + 1, rem);
            w[q] = c.W[a + k];
            g[q] = c.G[a + k];
        }
        bool ok = false;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = base + 64 * q + lane + 1;
            ok = k <= rem && w[q] - W0 <= M;
            if (ok && better<SMALL>(g[q] - G0, k, bS, bk, tie_rule)) bS = g[q] - G0, bk = k;
        }
        if (__builtin_amdgcn_ballot_w64(ok) != ~0ull) break;  // (feasibility is monotone: the end lies in these 256)
    }
    return wave_best<SMALL>(bS, bk, tie_rule);
}

// One wavefront: the longest feasible prefix at place a under the simultaneous-start profile, if it is shorter than
// kNextMax (or rem is); else -1.  Lane l of row q stands for the completion time o of place a + 64 q + l and sums the
// memory held then, sum over {i: o_i >= o} of (s_i + o) (Section 4), as the requests join one by one; the first that
// takes a sum above M ends the prefix.  (Times of requests that have not joined impose nothing the joined ones do
// not: the memory rises from there to the next completion.)
__device__ __forceinline__ int wave_profile_extent(const Sums &c, int a, int rem, unsigned M)
{
    const int lane = threadIdx.x & 63;
    const u64 P0 = c.W[a] - c.S[a];
    unsigned acc[4];
    int sv[4], ov[4];
    int sure = 0;
    int hi = 0;  // beyond: even the memory at the earliest completion, at least sum (s_i + 1), is too much
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int k = 64 * q + lane + 1;
        const int kk = min(k, rem);
        const bool ok = k <= rem && c.W[a + kk] - c.S[a + kk] - P0 + (u64)k <= (u64)M;
        sv[q] = c.s[a + kk - 1];
        ov[q] = k <= rem ? c.o[a + kk - 1] : 0x7fffffff;
        acc[q] = 0;
        hi += __popcll(__builtin_amdgcn_ballot_w64(ok));
        sure += __popcll(__builtin_amdgcn_ballot_w64(k <= rem && c.W[a + kk] - c.W[a] <= (u64)M));
    }
    // (the first `sure` of them fit: their peaks do)
    auto join = [&](int si, int oi) __attribute__((always_inline)) {
        unsigned most = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            acc[r] += oi >= ov[r] ? (unsigned)si + (unsigned)ov[r] : 0u;
            most = max(most, acc[r]);
        }
        return most;
    };
    int K = -1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int m = min(64, hi - 64 * q), free = min(m, sure - 64 * q);
        int l = 0;
        for (; l < free; ++l) (void)join(__builtin_amdgcn_readlane(sv[q], l), __builtin_amdgcn_readlane(ov[q], l));
        for (; l < m; ++l) {
            const unsigned most = join(__builtin_amdgcn_readlane(sv[q], l), __builtin_amdgcn_readlane(ov[q], l));
            if (__builtin_amdgcn_ballot_w64(most > M) != 0) {
                K = 64 * q + l;
                break;
            }
        }
        if (K >= 0) break;
    }
    if (K >= 0) return K;
    return hi < kNextMax || rem <= kNextMax ? hi : -1;
}

// Largest k in [0, rem] with g(k) <= M, for g increasing in k: coarse probes, then fine ones.  Every thread
// of a workgroup of 1024 receives it.
template <class G>
__device__ __forceinline__ int count_fitting(int rem, G g, u64 M)
{
    int K = 0, span = rem;  // g(K) fits; the answer lies in [K, K + span]
    while (span > 0) {
        const int step = (span + 1023) / 1024;
        const int k = (int)(threadIdx.x + 1) * step;
        const bool ok = k <= span && g(K + k) <= M;
        const int cnt = __syncthreads_count(ok);
        const int top = K + span;
        K += cnt * step;
        span = min(top, K + step - 1) - K;
        __syncthreads();
    }
    return K;
}

// The profile test for a growing prefix by a whole workgroup of 1024: buckets by completion time (o - 1, or the
// rank in the (o, id) order when times are too long for that), base = suffix sums (requests that complete at or after
// the bucket's time, and their prompts) of the prefix accepted so far, delta = those about to join.
template <bool IN_LDS>  // (one instantiation per address space)
struct Profile {
    unsigned *base_c, *base_s, *delta_c, *delta_s;
    int buckets;
    const int *rank_of;   // by position; null: buckets are completion times
    const int *o_of_rank;

    __device__ __forceinline__ unsigned time_of(int b) const { return rank_of ? (unsigned)o_of_rank[b] : (unsigned)b + 1u; }

    __device__ __forceinline__ void clear()
    {
        for (int b = threadIdx.x; b < buckets; b += 1024) base_c[b] = base_s[b] = delta_c[b] = delta_s[b] = 0;
        __syncthreads();
    }

    // Do the places [from, to) fit beside the accepted ones?  If so they are accepted.
    __device__ __forceinline__ bool join(const Sums &c, int from, int to, unsigned M, unsigned *wave_c, unsigned *wave_s)
    {
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
        for (int p = from + tid; p < to; p += 1024) {
            const int b = rank_of ? rank_of[p] : c.o[p] - 1;
            atomicAdd(&delta_c[b], 1u);
            atomicAdd(&delta_s[b], (unsigned)c.s[p]);
        }
        __syncthreads();
        // suffix sums: wavefront 0 takes the latest times, the first lane the latest of all
        const int rows = (buckets + 1023) >> 10;
        const int top = buckets - 1 - 64 * rows * wave - lane;
        unsigned cc = 0, cs = 0;
        for (int j = 0; j < rows; ++j) {
            const int b = top - 64 * j;
            const unsigned vc = wave_scan_u32(b >= 0 ? delta_c[b] : 0u) + cc;
            const unsigned vs = wave_scan_u32(b >= 0 ? delta_s[b] : 0u) + cs;
            if (b >= 0) delta_c[b] = vc, delta_s[b] = vs;
            cc = (unsigned)__builtin_amdgcn_readlane((int)vc, 63);
            cs = (unsigned)__builtin_amdgcn_readlane((int)vs, 63);
        }
        if (lane == 0) wave_c[wave] = cc, wave_s[wave] = cs;
        __syncthreads();
        unsigned off_c = 0, off_s = 0;
        for (int v = 0; v < wave; ++v) off_c += wave_c[v], off_s += wave_s[v];
        int viol = 0;
        for (int j = 0; j < rows; ++j) {
            const int b = top - 64 * j;
            if (b >= 0) {
                const unsigned nc = base_c[b] + delta_c[b] + off_c, ns = base_s[b] + delta_s[b] + off_s;
                viol |= (u64)ns + (u64)nc * time_of(b) > (u64)M;
            }
        }
        const bool fits = __syncthreads_or(viol) == 0;
        for (int j = 0; j < rows; ++j) {
            const int b = top - 64 * j;
            if (b >= 0) {
                if (fits) base_c[b] += delta_c[b] + off_c, base_s[b] += delta_s[b] + off_s;
                delta_c[b] = delta_s[b] = 0;
            }
        }
        __syncthreads();
        return fits;
    }

    // Longest feasible prefix at place a (clear() before; everything is zero again behind it).
    __device__ __forceinline__ int extent(const Sums &c, int a, int rem, unsigned M, unsigned *wave_c, unsigned *wave_s)
    {
        // the sum of peaks bounds the memory from above, sum (s_i + 1) from below
        const u64 W0 = c.W[a], P0 = c.W[a] - c.S[a];
        int lo = count_fitting(rem, [&](int k) { return c.W[a + k] - W0; }, (u64)M);
        int hi = count_fitting(rem, [&](int k) { return c.W[a + k] - c.S[a + k] - P0 + (u64)k; }, (u64)M);
        if (lo < hi) {
            join(c, a, a + lo, M, wave_c, wave_s);
            int step = max(64, lo >> 2);
            bool failed = false;
            while (lo < hi) {
                const int st = failed ? (hi - lo + 1) >> 1 : min(step, hi - lo);
                if (join(c, a + lo, a + lo + st, M, wave_c, wave_s)) {
                    lo += st;
                    step <<= 1;
                } else {
                    hi = lo + st - 1;
                    failed = true;
                }
            }
            clear();
        }
        return lo;
    }
};

// argmin over k = 1..K at place a by a workgroup of 1024; every thread receives k*.
template <bool SMALL>
__device__ int group_argmin(const Sums &c, int a, int K, int tie_rule, u64 *red_S, int *red_k)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const u64 G0 = c.G[a];
    u64 bS = 0;
    int bk = 0;
    // Four reads in flight, where one a turn left the loop to their latency (0.35 us each): 20000 sizes 7.8 -> 5.0 us; 40000 chat
    // requests in 3 / 5 batches 142 -> 137 / 148 -> 144 us a call, under the profile constraint in 3 batches 242 -> 235.
    for (int k0 = tid + 1; k0 <= K; k0 += 4096) {
        u64 g[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) g[q] = c.G[a + min(k0 + 1024 * q, K)];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = k0 + 1024 * q;
            if (k <= K && better<SMALL>(g[q] - G0, k, bS, bk, tie_rule)) bS = g[q] - G0, bk = k;
        }
    }
    bk = wave_best<SMALL>(bS, bk, tie_rule);
    if (lane == 0) red_S[wave] = bS, red_k[wave] = bk;
    __syncthreads();
    bS = red_S[lane & 15];
    bk = lane < 16 ? red_k[lane & 15] : 0;
    bk = wave_best<SMALL>(bS, bk, tie_rule);
    __syncthreads();
    return bk;
}

__device__ __forceinline__ u64 field_mask(int bits) { return (1ull << bits) - 1ull; }

// The batch a place belongs to: the first with ends[b] > place.
__device__ __forceinline__ int batch_of_place(const int *ends, int nb, int place)
{
    int lo = 0, hi = nb - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ends[mid] > place) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

// ------------------------------------------------------------------------------ one workgroup

// Everything in one workgroup: n <= TPB * E requests, element 64 E wave + 64 e + lane of an order in k[e].
// Also the length scan of the call (status word, longest decode).  What bounds it is latency, a chain of short
// steps: 61 requests 22 -> 7 us (one wavefront, no barrier waits for anyone), 200 30 -> 12 us.
template <int TPB, int E, bool PROFILE>
__global__ __launch_bounds__(TPB) void sortedF_small_kernel(SortedArgs p)
{
    constexpr int N = TPB * E, NW = TPB / 64;
    extern __shared__ u64 lds64[];
    // the sort's two buffers and the prefix sums are never alive together
    u64 *W = lds64, *G = W + N + 2, *S = PROFILE ? G + N + 2 : G;
    int *ends = (int *)(lds64 + (PROFILE ? 3 : 2) * (N + 2));
    int *by_o = ends + N;  // id at a rank of the (o, id) order, and the inverse (only when ranks are needed)
    int *rank_of = by_o + N;
    int *s_pos = rank_of + N;  // PROFILE: lengths by sorted position, rank by sorted position
    int *o_pos = s_pos + N, *rank_pos = o_pos + N, *o_of_rank = rank_pos + N;
    unsigned *hist = (unsigned *)(o_of_rank + N);
    __shared__ u64 tot_w[NW], tot_q[NW], red_S[16];
    __shared__ int red_k[16], sh[4];
    __shared__ unsigned wave_c[16], wave_s[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = p.n;
    const int i0 = 64 * E * wave + lane;
    const u64 M = (u64)p.M;

    // ---- lengths, well-formedness, keys
    if (tid == 0) sh[0] = 0, sh[1] = 0, sh[2] = 0;
    __syncthreads();
    int sv[E], ov[E], bad = 0, omax = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = i0 + 64 * e;
        sv[e] = ov[e] = 1;
        if (i < n) sv[e] = p.s[i], ov[e] = p.o[i];
        if (sv[e] < 1 || ov[e] < 1 || (long long)sv[e] + ov[e] > (long long)p.M) bad = 1;
        if (i < n) omax = max(omax, ov[e]);
    }
    omax = wave_max_i32(omax);
    if (lane == 0) atomicMax(&sh[1], omax);
    if (bad) atomicOr(&sh[0], 1);
    __syncthreads();
    bad = sh[0];
    omax = sh[1];
    if (tid == 0) {
        p.words[KVS_W_STATUS] = bad ? KVSCHED_DEV_BAD_LENGTH : 0;
        p.words[KVS_W_STATUS_AT] = KVS_W_STATUS;
        p.words[KVS_W_OMAX] = omax;
        p.words[KVS_W_MINPOS] = 0x7fffffff;
        p.words[KVS_W_MAXPOS] = -1;
        if (bad) *p.num_batches_out = 0;
    }
    if (bad) {  // a request that can never run: no batches
        if (p.pad)
            for (int i = tid; i < n; i += TPB) p.batch_end_out[i] = 0, p.F_out[i] = 0.0;
        return;
    }
    u64 key[E];
    const u64 id_mask = field_mask(p.id_bits);
    const bool ranks = !p.packed || (PROFILE && omax > kSmallBuckets);
    if (ranks) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int i = i0 + 64 * e;
            key[e] = i < n ? ((u64)ov[e] << p.id_bits) | (u64)i : ~0ull;
        }
        block_sort<TPB, E>(key, lds64);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int r = i0 + 64 * e;
            if (r < n) {
                const int id = (int)(key[e] & id_mask);
                by_o[r] = id;
                rank_of[id] = r;
                if (PROFILE) o_of_rank[r] = (int)(key[e] >> p.id_bits);
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = i0 + 64 * e;
        const u64 w = (u64)sv[e] + (u64)ov[e];
        if (i >= n) key[e] = ~0ull;
        else if (p.packed) key[e] = (((w << p.o_bits) | (u64)ov[e]) << p.id_bits) | (u64)i;
        else key[e] = (w << p.id_bits) | (u64)rank_of[i];
    }
    block_sort<TPB, E>(key, lds64);
    __syncthreads();

    // ---- prefix sums over the sorted order
    u64 w[E], q[E], cw = 0, cq = 0;
    int id[E], oid[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = i0 + 64 * e;
        id[e] = oid[e] = 0;
        u64 wv = 0, qv = 0;
        if (i < n) {
            if (p.packed) {
                id[e] = (int)(key[e] & id_mask);
                qv = (key[e] >> p.id_bits) & field_mask(p.o_bits);
                wv = key[e] >> (p.id_bits + p.o_bits);
            } else {
                id[e] = by_o[(int)(key[e] & id_mask)];
                qv = (u64)p.o[id[e]];
                wv = key[e] >> p.id_bits;
            }
            oid[e] = (int)qv;
            if (PROFILE) {
                o_pos[i] = (int)qv;
                s_pos[i] = (int)(wv - qv);
                if (ranks) rank_pos[i] = rank_of[id[e]];
            }
        }
        w[e] = wave_scan_u64(wv) + cw;
        q[e] = wave_scan_u64(qv) + cq;
        cw = lane_value_u64(w[e], 63);
        cq = lane_value_u64(q[e], 63);
    }
    if (lane == 0) tot_w[wave] = cw, tot_q[wave] = cq;
    __syncthreads();
    u64 off_w = 0, off_q = 0, all_w = 0, all_q = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) {
        const u64 xw = tot_w[v], xq = tot_q[v];
        if (v < wave) off_w += xw, off_q += xq;
        all_w += xw;
        all_q += xq;
    }
    const u64 ga = (u64)p.ga, gb = (u64)p.gb;
    const u64 all_g = ga * (all_w - all_q) + gb * all_q;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = i0 + 64 * e;
        if (i < n) {
            const u64 wi = w[e] + off_w, qi = q[e] + off_q;
            W[i + 1] = wi;
            if (PROFILE) S[i + 1] = qi;
            G[i + 1] = ga * (wi - qi) + gb * qi;
        }
    }
    if (tid == 0) W[0] = G[0] = S[0] = 0;
    __syncthreads();

    // ---- batches
    const Sums c{W, S, G, s_pos, o_pos};
    const bool small = all_g < (1ull << 32);
    int nb = 0;
    if constexpr (!PROFILE) {
        // One wavefront, no barriers, 0.4 us a batch.  (The batches of all places at once, by all wavefronts, were 49 us for 256 mixed
        // requests whether in 12 batches or 59; so 10.3 and 24.7.)
        if (wave == 0) {
            for (int a = 0; a < n;) {
                const int k = small ? wave_batch<true>(c, a, n - a, M, p.tie_rule)
                                    : wave_batch<false>(c, a, n - a, M, p.tie_rule);
                if (k < 1) break;  // cannot happen for well-formed input; never spin
                a += k;
                if (lane == 0) ends[nb] = a;
                ++nb;
            }
            if (lane == 0) sh[2] = nb;
        }
        __syncthreads();
        nb = sh[2];
    } else if constexpr (NW == 1) {
        for (int a = 0; a < n;) {  // (n <= 64 < kNextMax: always decided)
            const int K = wave_profile_extent(c, a, n - a, (unsigned)M);
            const int k = small ? wave_batch<true>(c, a, K, ~0ull, p.tie_rule)
                                : wave_batch<false>(c, a, K, ~0ull, p.tie_rule);
            if (k < 1) break;
            a += k;
            if (lane == 0) ends[nb] = a;
            ++nb;
        }
        __syncthreads();
    } else {
        static_assert(TPB == 1024 || !PROFILE || TPB == 64, "the workgroup-wide profile test takes 1024 threads");
        Profile<true> prof{hist, hist + kSmallBuckets, hist + 2 * kSmallBuckets, hist + 3 * kSmallBuckets,
                                 ranks ? n : omax, ranks ? rank_pos : nullptr, o_of_rank};
        prof.clear();
        for (int a = 0; a < n;) {
            if (wave == 0) {
                const int K = wave_profile_extent(c, a, n - a, (unsigned)M);
                int k = -1;
                if (K >= 0)
                    k = small ? wave_batch<true>(c, a, K, ~0ull, p.tie_rule)
                              : wave_batch<false>(c, a, K, ~0ull, p.tie_rule);
                if (lane == 0) sh[3] = k;
            }
            __syncthreads();
            int k = sh[3];
            __syncthreads();
            if (k < 0) {
                const int K = prof.extent(c, a, n - a, (unsigned)M, wave_c, wave_s);
                k = small ? group_argmin<true>(c, a, K, p.tie_rule, red_S, red_k)
                          : group_argmin<false>(c, a, K, p.tie_rule, red_S, red_k);
            }
            if (k < 1) break;
            a += k;
            if (tid == 0) ends[nb] = a;
            ++nb;
        }
        __syncthreads();
    }

    // ---- metric values, and the batches in nondecreasing o
    for (int b = tid; b < (p.pad ? n : nb); b += TPB) {
        if (b < nb) {
            const int lo = b == 0 ? 0 : ends[b - 1], hi = ends[b];
            p.batch_end_out[b] = hi;
            const double k = (double)(hi - lo);
            p.F_out[b] = (double)(G[hi] - G[lo]) / ((double)p.gb * k * k);
        } else {
            p.batch_end_out[b] = 0;
            p.F_out[b] = 0.0;
        }
    }
    if (tid == 0) {
        *p.num_batches_out = nb;
        if (nb == 0 || ends[nb - 1] != n) atomicOr(&p.words[KVS_W_STATUS], KVSCHED_DEV_BAD_LENGTH);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = i0 + 64 * e;
        key[e] = ~0ull;
        if (i < n) {
            const u64 b = (u64)batch_of_place(ends, nb, i);
            key[e] = p.packed ? (((b << p.o_bits) | (u64)oid[e]) << p.id_bits) | (u64)id[e]
                              : (b << p.id_bits) | (u64)rank_of[id[e]];
        }
    }
    __syncthreads();
    block_sort<TPB, E>(key, lds64);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = i0 + 64 * e;
        if (i < n) {
            const int v = (int)(key[e] & id_mask);
            p.order_out[i] = p.packed ? v : by_o[v];
        }
    }
}

// Words of dynamic LDS of the kernel above.
constexpr size_t small_lds_bytes(int N, bool profile)
{
    return (size_t)(profile ? 3 : 2) * 8 * (N + 2) + (size_t)(profile ? 7 : 3) * 4 * N + (profile ? 16 * kSmallBuckets : 0);
}
static_assert(small_lds_bytes(1024, true) + 2048 <= 160 * 1024 && kSmallSum <= 1024 && kSmallProfile <= 1024, "fits the LDS");

// ------------------------------------------------------------------------- many workgroups

// What the launches of a large construction share (arrays in the context's scratch).
struct LargeArrays {
    u64 *key[2];
    u64 *W, *S, *G, *tot;  // tot: two sums per 4096 places (beyond kSumsHere)
    int *s_pos, *o_pos;
    int *by_o, *rank_of, *rank_pos, *o_of_rank;  // (only when the (o, id) order is sorted too)
    unsigned short *next;
    unsigned *hist;
    int *extent;  // by place, where they are found ahead: the longest feasible prefixes under the profile constraint (hist's memory)
};

// Are ranks in the (o, id) order needed?  By keys that do not fit, and by the profile test when the completion times
// are too many for buckets in LDS (the host launches their sort whenever that could be).
__device__ __forceinline__ bool ranks_needed(const SortedArgs &p) { return !p.packed || p.words[KVS_W_OMAX] > kLargeBuckets; }

__device__ __forceinline__ bool faulty(const SortedArgs &p) { return (p.words[KVS_W_STATUS] & KVSCHED_DEV_BAD_LENGTH) != 0; }

enum { KEYS_BY_O, KEYS_BY_SIZE };

__device__ __forceinline__ u64 request_key(const SortedArgs &p, const LargeArrays &m, int what, int i, int s, int o)
{
    if (what == KEYS_BY_O) return ((u64)o << p.id_bits) | (u64)i;
    const u64 w = (u64)s + (u64)o;
    return p.packed ? (((w << p.o_bits) | (u64)o) << p.id_bits) | (u64)i : (w << p.id_bits) | (u64)m.rank_of[i];
}

// What a length scan leaves (one thread): status, longest decode.
__device__ __forceinline__ void lengths_seen(const SortedArgs &p, bool bad, int omax)
{
    p.words[KVS_W_STATUS] = bad ? KVSCHED_DEV_BAD_LENGTH : 0;
    p.words[KVS_W_STATUS_AT] = KVS_W_STATUS;
    p.words[KVS_W_OMAX] = omax;
    p.words[KVS_W_MINPOS] = 0x7fffffff;
    p.words[KVS_W_MAXPOS] = -1;
}

// ------------------------------------------------ up to kCountMax requests: places by counting
//
// A request's place in an order is the number of smaller keys.  Every workgroup holds all keys in LDS and counts them for OWN
// requests, 64 / OWN lanes of each wavefront a request and a 16 OWN / 64-th of the keys each; so the whole chip works, where sorted runs of 2048 keys
// keep five compute units busy and have to be merged.  The first launch of a call is its length scan too, as every workgroup reads all
// lengths.  Bound by vector issue, 2.5 instructions a comparison of 64 pairs, in three
// fifths of the compute units (all up to 16384): 10000 requests 18.4 us where scan, sorted runs and merges took 28 (and two launches, for the order by
// (o, id), that found nothing to do 8), 5000 7.5, 2000 6; the whole construction of 16000 requests 102 -> 95.  (Keys of 32 bits, the
// id told by the place in LDS and two instructions a comparison written out, took 17.6 to 18.6 for 10000.)
template <int OWN>
__global__ __launch_bounds__(1024) void count_places_kernel(SortedArgs p, LargeArrays m, int what, int scan, u64 *out)
{
    extern __shared__ __align__(16) u64 keys[];
    __shared__ int count[OWN], sh_omax;
    constexpr int GROUPS = 1024 / OWN;
    const int tid = threadIdx.x, lane = tid & 63, n = p.n;
    if (!scan && faulty(p)) return;
    if (blockIdx.y == 1) what = KEYS_BY_O;  // (beside the order by size)
    if (tid < OWN) count[tid] = 0;
    if (tid == 0) sh_omax = 0;
    __syncthreads();
    const int padded = (n + 8 * GROUPS - 1) / (8 * GROUPS) * (8 * GROUPS);
    int omax = 0, bad = 0;
    for (int i = tid; i < padded; i += 1024) {
        u64 key = ~0ull;
        if (i < n) {
            const int s = p.s[i], o = p.o[i];
            bad |= s < 1 || o < 1 || (long long)s + o > (long long)p.M;
            omax = max(omax, o);
            key = request_key(p, m, what, i, s, o);
        }
        keys[i] = key;
    }
    omax = wave_max_i32(omax);
    if (lane == 0) atomicMax(&sh_omax, omax);
    bad = __syncthreads_or(bad);
    omax = sh_omax;
    if (scan && blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) lengths_seen(p, bad, omax);
    if (bad || (blockIdx.y == 1 && omax <= kLargeBuckets)) return;  // (no ranks needed)

    const int el = lane & (OWN - 1), i = OWN * blockIdx.x + el;
    const u64 mine = keys[min(i, padded - 1)];
    unsigned c = 0;
    const ulonglong2 *two = (const ulonglong2 *)keys + tid / OWN;
    for (int q = 0; q < padded / 2; q += 4 * GROUPS) {  // (four reads in flight)
        ulonglong2 x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = two[q + r * GROUPS];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            c += x[r].x < mine ? 1u : 0u;
            c += x[r].y < mine ? 1u : 0u;
        }
    }
    atomicAdd(&count[el], (int)c);
    __syncthreads();
    if (tid >= OWN || i >= n) return;
    const int place = count[tid];
    if (what == KEYS_BY_SIZE) {
        out[place] = mine;
    } else {
        const int id = (int)(mine & field_mask(p.id_bits));
        m.by_o[place] = id;
        m.rank_of[id] = place;
        m.o_of_rank[place] = (int)(mine >> p.id_bits);
    }
}

// The order: the requests of a batch, which lie together by size, in nondecreasing (o, id).  (10000 mixed requests, 5500 of them in one
// batch, 22.8 us, sorted runs and merges 26; 5000 12.7.)  A workgroup counts for 64
// places how many of their batch come before each; what lies to the left of the 64 places concerns the first's batch alone, what lies
// to the right the last's.  NARROW: the keys (o, id), or the ranks that stand for them, fit in 32 bits.
template <bool NARROW>
__device__ __forceinline__ void order_of_places(const SortedArgs &p, const LargeArrays &m, const u64 *by_place, int lo_all, int hi_all,
                                                int lo, int hi, u64 own, u64 *tile, int *count)
{
    typedef typename std::conditional<NARROW, unsigned, u64>::type Key;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = p.n, first = 64 * blockIdx.x;
    const u64 low = p.packed ? field_mask(p.o_bits + p.id_bits) : field_mask(p.id_bits);
    Key *const keys = (Key *)tile;
    const Key mine = (Key)(own & low);
    const bool one = __builtin_amdgcn_ballot_w64(lo != lo_all || hi != hi_all) == 0;  // (one batch has all 64 places, mostly)
    unsigned c = 0;
    for (int j0 = lo_all; j0 < hi_all; j0 += kOrderTile) {
        const int held = min(kOrderTile, hi_all - j0), all = (held + 127) & ~127;
        __syncthreads();
        u64 x[kOrderTile / 1024];  // (a trip to memory together)
#pragma unroll
        for (int r = 0; r < kOrderTile / 1024; ++r)
            if (1024 * r < all) x[r] = by_place[j0 + min(1024 * r + tid, held - 1)];
#pragma unroll
        for (int r = 0; r < kOrderTile / 1024; ++r) {
            const int j = 1024 * r + tid;
            if (j < all) keys[j] = j < held ? (Key)(x[r] & low) : ~(Key)0;
        }
        __syncthreads();
        // (sixteen wavefronts, four keys each in turn)
        if (one) {
            for (int j = 4 * wave; j < all; j += 128) {
                Key x[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) x[q] = keys[j + (q & 3) + 16 * (q & 4)];
#pragma unroll
                for (int q = 0; q < 8; ++q) c += x[q] < mine ? 1u : 0u;
            }
        } else {
            for (int j = 4 * wave; j < all; j += 64) {
                const Key x[4] = {keys[j], keys[j + 1], keys[j + 2], keys[j + 3]};
#pragma unroll
                for (int q = 0; q < 4; ++q) c += x[q] < mine && (unsigned)(j0 + j + q - lo) < (unsigned)(hi - lo) ? 1u : 0u;
            }
        }
    }
    atomicAdd(&count[lane], (int)c);
    __syncthreads();
    if (tid >= 64 || first + lane >= n) return;
    const int v = (int)(own & field_mask(p.id_bits));
    p.order_out[lo + count[lane]] = p.packed ? v : m.by_o[v];
}

__global__ __launch_bounds__(1024) void order_batches_kernel(SortedArgs p, LargeArrays m, const u64 *by_place)
{
    __shared__ __align__(16) u64 tile[kOrderTile];
    __shared__ int count[64], ends[64];
    const int tid = threadIdx.x, lane = tid & 63, n = p.n, first = 64 * blockIdx.x;
    const int i = min(first + lane, n - 1), last = min(first + 63, n - 1);
    const int nb = *p.num_batches_out;
    const u64 own = by_place[i];
    const int end = p.batch_end_out[lane];  // (n > 64)
    if (faulty(p) || nb < 1) return;
    if (tid < 64) count[tid] = 0;
    int lo, hi, lo_all, hi_all;
    if (nb <= 64) {  // (each end in a lane, read together with the rest: 5000 requests 10.8 -> 9.9 us, 1100 5.8 -> 5.2)
        const u64 there = ~0ull >> (64 - nb);
        int b = __popcll(__builtin_amdgcn_ballot_w64(end <= first) & there);
        lo = lo_all = b > 0 ? __builtin_amdgcn_readlane(end, max(b - 1, 0)) : 0;
        hi = hi_all = __builtin_amdgcn_readlane(end, b);
        while (hi_all <= last && b + 1 < nb) {
            const int next = __builtin_amdgcn_readlane(end, ++b);
            if (hi_all <= i) lo = hi_all, hi = next;
            hi_all = next;
        }
        __syncthreads();
    } else {
        // the batch of the first place, by counting the ends before it, and the next 64 ends
        int before = 0;
        for (int b0 = 0; b0 < nb; b0 += 1024) before += __syncthreads_count(b0 + tid < nb && p.batch_end_out[min(b0 + tid, nb - 1)] <= first);
        if (tid < 64) ends[tid] = p.batch_end_out[min(before + tid, nb - 1)];
        __syncthreads();
        lo = lo_all = before > 0 ? p.batch_end_out[before - 1] : 0;
        hi = hi_all = ends[0];
        for (int b = 0; b < 63 && ends[b] <= last; ++b) {  // (the same in all lanes; at most 64 batches touch 64 places)
            if (ends[b] <= i) lo = ends[b], hi = ends[b + 1];
            hi_all = ends[b + 1];
        }
    }
    const int bits = p.packed ? 32 - __builtin_clz(max(p.words[KVS_W_OMAX], 1)) + p.id_bits : p.id_bits;
    if (bits < 32) order_of_places<true>(p, m, by_place, lo_all, hi_all, lo, hi, own, tile, count);
    else order_of_places<false>(p, m, by_place, lo_all, hi_all, lo, hi, own, tile, count);
}

// ------------------------------------------------ beyond: sorted runs and merges

// Keys of kRun consecutive requests, sorted.  scan: the launch is the call's length scan as well (the workgroup that is done last takes
// what the others have seen).  The second row of workgroups, if there is one, sorts by (o, id).
template <int WHAT>
__global__ __launch_bounds__(1024) void sort_runs_kernel(SortedArgs p, LargeArrays m, int scan, u64 *out, u64 *out_by_o)
{
    __shared__ u64 buf[2 * kRun];
    __shared__ int sh_omax;
    if (!scan && faulty(p)) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool beside = blockIdx.y == 1;
    if (threadIdx.x == 0) sh_omax = 0;
    __syncthreads();
    u64 key[2];
    int omax = 0, bad = 0;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int i = kRun * blockIdx.x + 128 * wave + 64 * e + lane;
        key[e] = ~0ull;
        if (i < p.n) {
            const int s = p.s[i], o = p.o[i];
            bad |= s < 1 || o < 1 || (long long)s + o > (long long)p.M;
            omax = max(omax, o);
            key[e] = request_key(p, m, beside ? KEYS_BY_O : WHAT, i, s, o);
        }
    }
    if (scan && !beside) {
        omax = wave_max_i32(omax);
        if (lane == 0) atomicMax(&sh_omax, omax);
        bad = __syncthreads_or(bad);
        if (threadIdx.x == 0) {
            atomicMax(&p.words[KVS_W_SCAN_OMAX], sh_omax);
            atomicOr(&p.words[KVS_W_SCAN_FLAGS], bad ? KVSCHED_DEV_BAD_LENGTH : 0);
            device_writes_done();
            if (atomicAdd(&p.words[KVS_W_SCAN_DONE], 1) == (int)gridDim.x - 1) {
                omax = atomicExch(&p.words[KVS_W_SCAN_OMAX], 0);
                lengths_seen(p, atomicExch(&p.words[KVS_W_SCAN_FLAGS], 0) != 0, omax);
                atomicExch(&p.words[KVS_W_SCAN_DONE], 0);
            }
        }
    }
    block_sort<1024, 2>(key, buf);
    u64 *const to = beside ? out_by_o : out;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int i = kRun * blockIdx.x + 128 * wave + 64 * e + lane;
        if (i < p.n) to[i] = key[e];
    }
}

// Keys (batch, o, id) of kRun consecutive places, sorted.
__global__ __launch_bounds__(1024) void sort_batch_runs_kernel(SortedArgs p, const u64 *by_place, u64 *out)
{
    __shared__ u64 buf[2 * kRun];
    if (faulty(p)) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nb = *p.num_batches_out;
    u64 key[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int i = kRun * blockIdx.x + 128 * wave + 64 * e + lane;
        key[e] = ~0ull;
        if (i < p.n) {
            const u64 old = by_place[i];
            const u64 b = (u64)batch_of_place(p.batch_end_out, nb, i);
            const int low = p.packed ? p.o_bits + p.id_bits : p.id_bits;
            key[e] = (b << low) | (old & field_mask(low));
        }
    }
    block_sort<1024, 2>(key, buf);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int i = kRun * blockIdx.x + 128 * wave + 64 * e + lane;
        if (i < p.n) out[i] = key[e];
    }
}

// One pass of merging sorted runs of `run` keys, kFan at a time: the keys are distinct, so a key's place is its place
// in its own run plus the number of smaller keys in the others, found by binary searches that advance together.
// The last pass may emit what the key stands for: MERGE_IDS the request ids (the order), MERGE_RANKS the (o, id)
// order and its inverse.  The second row of workgroups, if there is one, merges the runs by (o, id) (its last pass emits ranks).
enum { MERGE_KEYS, MERGE_IDS, MERGE_RANKS };
template <int EMIT>
__global__ __launch_bounds__(256) void merge_runs_kernel(SortedArgs p, LargeArrays m, const u64 *in, u64 *out, int run, int of_ranks,
                                                         const u64 *in_by_o, u64 *out_by_o)
{
    const bool beside = blockIdx.y == 1;
    if (faulty(p) || ((of_ranks || beside) && !ranks_needed(p))) return;
    if (beside) in = in_by_o, out = out_by_o;
    const int g = blockIdx.x * 256 + threadIdx.x, n = p.n;
    if (g >= n) return;
    const u64 key = in[g];
    const int r = g / run, first = r / kFan * kFan;
    int below[kFan - 1], start[kFan - 1], len[kFan - 1];
#pragma unroll
    for (int q = 0; q < kFan - 1; ++q) {
        const int rr = first + q + (first + q >= r ? 1 : 0);
        const long long st = (long long)rr * run;
        start[q] = (int)min(st, (long long)n);
        len[q] = (int)min((long long)run, (long long)n - start[q]);
        below[q] = 0;
    }
    for (int step = run; step > 0; step >>= 1) {
#pragma unroll
        for (int q = 0; q < kFan - 1; ++q) {
            const int at = below[q] + step - 1;
            if (at < len[q] && in[start[q] + at] < key) below[q] += step;
        }
    }
    int place = first * run + (g - r * run);
#pragma unroll
    for (int q = 0; q < kFan - 1; ++q) place += below[q];
    const int v = (int)(key & field_mask(p.id_bits));
    const bool last = (long long)run * kFan >= n;
    if (EMIT == MERGE_RANKS || (beside && last)) {
        m.by_o[place] = v;
        m.rank_of[v] = place;
        m.o_of_rank[place] = (int)(key >> p.id_bits);
    } else if (EMIT == MERGE_IDS && !beside) {
        p.order_out[place] = p.packed ? v : m.by_o[v];
    } else {
        out[place] = key;
    }
}

// s + o and o of a sorted key.
__device__ __forceinline__ void key_lengths(const SortedArgs &p, const LargeArrays &m, u64 key, u64 &w, u64 &o)
{
    w = p.packed ? key >> (p.id_bits + p.o_bits) : key >> p.id_bits;
    o = p.packed ? (key >> p.id_bits) & field_mask(p.o_bits) : (u64)m.o_of_rank[(int)(key & field_mask(p.id_bits))];
}

// The sums of s + o and o over each 4096 places.
__global__ __launch_bounds__(1024) void place_sums_kernel(SortedArgs p, LargeArrays m, const u64 *sorted)
{
    if (faulty(p)) return;
    __shared__ u64 tw[16], tq[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    u64 aw = 0, aq = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = 4096 * blockIdx.x + 1024 * e + threadIdx.x;
        u64 w = 0, o = 0;
        if (i < p.n) key_lengths(p, m, sorted[i], w, o);
        aw += w;
        aq += o;
    }
    aw = lane_value_u64(wave_scan_u64(aw), 63);
    aq = lane_value_u64(wave_scan_u64(aq), 63);
    if (lane == 0) tw[wave] = aw, tq[wave] = aq;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int v = 1; v < 16; ++v) aw += tw[v], aq += tq[v];
        m.tot[2 * blockIdx.x] = aw;
        m.tot[2 * blockIdx.x + 1] = aq;
    }
}

// Lengths by sorted place and their prefix sums, 4096 places a workgroup.  What lies before its own comes from the sums that a launch
// ahead has left (summed), or is added up here: up to kSumsHere requests that costs less than the launch (4.7 us; 100000 requests 19 us
// against 8 and 5).
__global__ __launch_bounds__(1024) void prefix_sums_kernel(SortedArgs p, LargeArrays m, const u64 *sorted, int ranks, int summed)
{
    if (faulty(p)) return;
    ranks = ranks && ranks_needed(p);
    __shared__ u64 tw[16], tq[16], bw[16], bq[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const u64 id_mask = field_mask(p.id_bits);
    u64 key[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = 4096 * blockIdx.x + 256 * wave + 64 * e + lane;
        key[e] = sorted[min(i, p.n - 1)];
    }
    u64 fw = 0, fq = 0;  // everything before this block
    if (summed) {
        for (int b = threadIdx.x; b < (int)blockIdx.x; b += 1024) fw += m.tot[2 * b], fq += m.tot[2 * b + 1];
    } else {
        for (int i0 = threadIdx.x; i0 < 4096 * (int)blockIdx.x; i0 += 4096) {
            u64 k[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) k[e] = sorted[i0 + 1024 * e];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                u64 w, o;
                key_lengths(p, m, k[e], w, o);
                fw += w;
                fq += o;
            }
        }
    }
    fw = lane_value_u64(wave_scan_u64(fw), 63);
    fq = lane_value_u64(wave_scan_u64(fq), 63);
    if (lane == 0) bw[wave] = fw, bq[wave] = fq;
    u64 w[4], q[4], cw = 0, cq = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = 4096 * blockIdx.x + 256 * wave + 64 * e + lane;
        u64 wi = 0, o = 0;
        if (i < p.n) {
            key_lengths(p, m, key[e], wi, o);
            m.s_pos[i] = (int)(wi - o);
            m.o_pos[i] = (int)o;
            if (ranks) m.rank_pos[i] = p.packed ? m.rank_of[(int)(key[e] & id_mask)] : (int)(key[e] & id_mask);
        }
        w[e] = wave_scan_u64(wi) + cw;
        q[e] = wave_scan_u64(o) + cq;
        cw = lane_value_u64(w[e], 63);
        cq = lane_value_u64(q[e], 63);
    }
    if (lane == 0) tw[wave] = cw, tq[wave] = cq;
    __syncthreads();
    u64 ow = 0, oq = 0;
    for (int v = 0; v < 16; ++v) {
        ow += bw[v] + (v < wave ? tw[v] : 0);
        oq += bq[v] + (v < wave ? tq[v] : 0);
    }
    const u64 ga = (u64)p.ga, gb = (u64)p.gb;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = 4096 * blockIdx.x + 256 * wave + 64 * e + lane;
        if (i < p.n) {
            const u64 wi = w[e] + ow, qi = q[e] + oq;
            m.W[i + 1] = wi;
            m.S[i + 1] = qi;
            m.G[i + 1] = ga * (wi - qi) + gb * qi;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) m.W[0] = m.S[0] = m.G[0] = 0;
}

__device__ __forceinline__ bool small_numbers(const SortedArgs &p, const Sums &c) { return p.n < 65536 && c.G[p.n] < (1ull << 32); }

// Under the profile constraint: are the extents of all places found ahead (profile_extents_kernel), or each where the chain
// needs it?  The former costs what one extent costs, 15 to 45 us, and then a microsecond or two for each of the 1 (up to 1536 requests) to
// 26 (40000) places that a wavefront takes; the chain takes some 20 us for each batch, if the extents are beyond kNextMax, and the
// launch before it some time for each place if they are below.  Completion times up to 2048, the chain and ahead: 5000 mixed
// requests in 6 batches 170 and 75 us, in 73 213 and 80, in 240 175 and 91; 1000 chat requests in 3 73 and 56, 10000 143 and 130; 400
// mixed ones in 5 64 and 41.  The other side: extents of 16 requests and fewer, 300 chat requests in 23 batches 32 and 39, 2000 in 37 47
// and 53; those beyond some 10000 on average, which every wavefront reads through, 40000 chat requests in 3 batches 219 and 240; and
// constructions of up to kNextMax requests, none of whose extents is beyond what one wavefront tests (no launch is made for them): 129
// chat requests in 3 / 6 / 25 batches 32 / 28 / 29 and 41 / 39 / 32, 256 in 3 / 6 / 29 40 / 33 / 30 and 45 / 42 / 34.  Beyond 2048 an
// extent costs twice and more and half as many wavefronts find them: 400 bimodal requests in 12 batches 36 and 56, 10000 in 42
// 145 and 193, 2000 in 11 91 and 127.
constexpr u64 kAheadMost = 10000;

__device__ __forceinline__ bool extents_ahead(const SortedArgs &p, const LargeArrays &m)
{
    if (p.n <= kNextMax) return false;
    const int omax = p.words[KVS_W_OMAX];
    const u64 all = m.W[p.n], M = (u64)p.M, some = (u64)p.n * M;  // (some / all requests an extent, on average)
    if (omax <= kLargeBuckets / 2) return all >= M && some >= 16 * all && some <= kAheadMost * all;
    return omax <= kLargeBuckets && all >= 6 * M && some >= kNextMax * all;
}

// The longest feasible prefix at every place under the simultaneous-start profile, where extents_ahead.  A
// wavefront takes `per` consecutive places: it keeps the memory held at each completion time, sum over {i: o_i >= time} of (s_i +
// time) (Section 4), for the prefix of the present place, finds the first place's extent by adding
// many requests at a time (a histogram of their completion times in LDS, summed from the end), and then goes on place by place: one request
// leaves, those behind the end join as long as they fit (a prefix without its first request stays feasible, so
// the end never moves back).  What bounds it is latency, the first extent's chain of some five joins of 3 us and the wavefront
// whose end moves most; the loops over times are kept rolled and everything in LDS, because the code is run once: with the times in
// registers and the loops unrolled, 19 KB of code, 10000 requests took 120 us instead of 66.  One request costs a pass over the times up
// to its own, which adds it and finds whether it fits (if not, a second pass takes it away again; with a pass to look and one to
// add, and every time compared with the request's, the whole call took 135 us instead of 120, 40000 bimodal requests in 11 batches 1690
// instead of 1360).

// The largest k in [0, rem] with g(k) <= M, for g increasing in k, by one wavefront.
template <class G>
__device__ __forceinline__ int wave_count_fitting(int rem, G g, u64 M)
{
    int K = 0, span = rem;
    while (span > 0) {
        const int step = (span + 63) / 64, k = (int)((threadIdx.x & 63) + 1) * step;
        const int cnt = __popcll(__builtin_amdgcn_ballot_w64(k <= span && g(K + min(k, span)) <= M));
        const int top = K + span;
        K += cnt * step;
        span = min(top, K + step - 1) - K;
    }
    return K;
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Words of LDS that completion times up to 64 `rows` take.
constexpr int extent_words(int rows) { return 64 * rows + 2 * 64 * (rows + 2); }

// Two wavefronts a workgroup, each with half of its LDS, where completion times are up to 2048; beyond, the first one has all of it.
__global__ __launch_bounds__(128) void profile_extents_kernel(SortedArgs p, LargeArrays m)
{
    constexpr int kRows = kLargeBuckets / 64;
    __shared__ __align__(16) unsigned lds[2 * extent_words(kRows / 2)];
    static_assert(2 * extent_words(kRows / 2) >= extent_words(kRows), "");
    const int omax = p.words[KVS_W_OMAX];
    if (faulty(p) || !extents_ahead(p, m)) return;
    const bool pairs = omax <= kLargeBuckets / 2;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (wave == 1 && !pairs) return;
    unsigned *const held = lds + wave * extent_words(kRows / 2);           // at time b + 1
    u64 *const slot = (u64 *)(held + 64 * (pairs ? kRows / 2 : kRows));    // (number, sum of s) of the requests that join, by their time
    const int waves = pairs ? 2 * (int)gridDim.x : (int)gridDim.x, mine_no = pairs ? 2 * (int)blockIdx.x + wave : (int)blockIdx.x;
    // Fewer requests are added one by one (10000 mixed requests in 17 batches 120 -> 115 us with 8 instead of 16; of completion times beyond
    // 2048, a join of which costs twice as much, 40000 bimodal ones in 11 1340 -> 1760).
    const int join_min = pairs ? 8 : 16;
    const int lane = threadIdx.x & 63, n = p.n, per = (n + waves - 1) / waves, a0 = mine_no * per, a1 = min(a0 + per, n);
    if (a0 >= a1) return;
    const unsigned M = (unsigned)p.M;
    // Times four to a lane, 256 a turn; while those of a join are summed lane l has the times rows l + 1 .. rows l + rows (rows a
    // power of two; two slots between the lanes' keep their 16-byte accesses off each other's banks).
    const int lg = max(2, 32 - __builtin_clz(((omax + 63) >> 6) - 1 | 1)), rows = 1 << lg;
    auto place = [&](int b) __attribute__((always_inline)) { return b + 2 * (b >> lg); };
    u32x4 *const mine = (u32x4 *)held + lane;
    for (int r = 0; r < rows / 4; ++r) mine[64 * r] = (u32x4)0u;

    // the most that any time holds when the places [from, to) join; they do if that is at most M (fewer than 2^18 of them: 32
    // bits hold the sums)
    auto join = [&](int from, int to) __attribute__((always_inline)) -> unsigned {
        u32x4 *own = (u32x4 *)(slot + (rows + 2) * lane);
        for (int g = 0; g < rows / 2; ++g) own[g] = (u32x4)0u;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int i0 = from; i0 < to; i0 += 512) {  // (512 requests a trip to memory)
            int ob[8], sb[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int i = min(i0 + 64 * q + lane, to - 1);
                ob[q] = m.o_pos[i];
                sb[q] = m.s_pos[i];
            }
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (i0 + 64 * q + lane < to) atomicAdd(&slot[place(ob[q] - 1)], (1ull << 32) | (unsigned)sb[q]);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        unsigned sums = 0, numbers = 0;
#pragma unroll 4
        for (int g = 0; g < rows / 2; ++g) {
            const u32x4 q = own[g];
            sums += q.x + q.z;
            numbers += q.y + q.w;
        }
        const unsigned us = wave_scan_u32(sums), un = wave_scan_u32(numbers);
        sums = (unsigned)__builtin_amdgcn_readlane((int)us, 63) - us;  // behind the lane's times
        numbers = (unsigned)__builtin_amdgcn_readlane((int)un, 63) - un;
#pragma unroll 4
        for (int g = rows / 2 - 1; g >= 0; --g) {
            u32x4 q = own[g];
            const unsigned time = (unsigned)(rows * lane + 2 * g + 1);
            sums += q.z;
            numbers += q.w;
            q.z = sums + __umul24(numbers, time + 1);
            sums += q.x;
            numbers += q.y;
            q.x = sums + __umul24(numbers, time);
            own[g] = q;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        auto more = [&](int r) __attribute__((always_inline)) {
            const u32x4 *at = (const u32x4 *)(slot + place(256 * r + 4 * lane));
            const u32x4 x = at[0], y = at[1];
            return (u32x4){x.x, x.z, y.x, y.z};
        };
        u32x4 most = (u32x4)0u;
#pragma unroll 4
        for (int r = 0; r < rows / 4; ++r) most = __builtin_elementwise_max(most, mine[64 * r] + more(r));
        const unsigned all = ~wave_min_u32(~max(max(most.x, most.y), max(most.z, most.w)));
        if (all <= M) {
#pragma unroll 4
            for (int r = 0; r < rows / 4; ++r) mine[64 * r] += more(r);
        }
        return all;
    };
    // One request more (sign 1), and the most that any time it touches holds then, or one less (sign -1).  Turns that lie in its times
    // as a whole need no choice by the time.
    auto change = [&](int s, int o, auto sign) __attribute__((always_inline)) -> unsigned {
        constexpr unsigned kSign = (unsigned)decltype(sign)::value;
        u32x4 most = (u32x4)0u;
        unsigned v = kSign * (unsigned)(s + 4 * lane + 1);
        const int whole = o >> 8;
#pragma unroll 4
        for (int r = 0; r < whole; ++r) {
            const u32x4 x = mine[64 * r] + (u32x4){v, v + kSign, v + 2 * kSign, v + 3 * kSign};
            mine[64 * r] = x;
            most = __builtin_elementwise_max(most, x);
            v += 256 * kSign;
        }
        if ((o & 255) != 0) {
            const int left = (o & 255) - 4 * lane;
            const u32x4 x = mine[64 * whole] +
                            (u32x4){left > 0 ? v : 0u, left > 1 ? v + kSign : 0u, left > 2 ? v + 2 * kSign : 0u, left > 3 ? v + 3 * kSign : 0u};
            mine[64 * whole] = x;
            most = __builtin_elementwise_max(most, x);
        }
        return ~wave_min_u32(~max(max(most.x, most.y), max(most.z, most.w)));
    };
    const std::integral_constant<int, 1> joins;
    const std::integral_constant<int, -1> leaves;

    // the sum of peaks bounds the memory of the first place's prefixes from above, sum (s_i + 1) that of every place's from below
    const u64 W0 = m.W[a0];
    int a = a0, e = a0;
    int step = wave_count_fitting(n - a, [&](int k) { return m.W[a + k] - W0; }, (u64)M);  // requests to try next
    int base = -64, sv = 1, ov = 1;  // lengths of the places base .. base + 63
    int first = -64, sa = 1, oa = 1;  // ... and of those that leave
    int over = 0;  // by how much the request behind the end is too much, at least
    for (;;) {
        bool failed = false;
        while (e < n && over <= 0) {
            if (step >= join_min) {
                step = min(step, min(1 << 18, n - e));
                const u64 Pa = m.W[a] - m.S[a];
                unsigned most = ~0u;
                if (m.W[e + step] - m.S[e + step] - Pa + (u64)(e + step - a) <= (u64)M) most = join(e, e + step);
                if (most <= M) {
                    e += step;
                    // as many more, in proportion, as the fullest time has room for
                    const int room = (int)((float)(e - a) * (float)(M - most) / (float)most);
                    step = failed ? min(room, step >> 1) : room;
                } else {
                    failed = true;
                    step >>= 1;
                }
                continue;
            }
            if (e >= base + 64) {
                base = e;
                const int i = min(base + lane, n - 1);
                sv = m.s_pos[i];
                ov = m.o_pos[i];
            }
            const int s = __builtin_amdgcn_readlane(sv, e - base), o = __builtin_amdgcn_readlane(ov, e - base);
            over = (int)(change(s, o, joins) - M);
            if (over > 0) {
                change(s, o, leaves);
            } else {
                ++e;
                if (!failed && ++step == 4) step = 2 * join_min;  // (a few in a row: many may follow)
            }
        }
        step = 0;
        if (lane == 0) m.extent[a] = e - a;
        if (a + 1 >= a1) break;
        if (a >= first + 64) {
            first = a;
            const int i = min(first + lane, n - 1);
            sa = m.s_pos[i];
            oa = m.o_pos[i];
        }
        const int s = __builtin_amdgcn_readlane(sa, a - first), o = __builtin_amdgcn_readlane(oa, a - first);
        change(s, o, leaves);
        over -= s + o;  // (no time loses more)
        ++a;
    }
}

// The batch every place would start, one wavefront each; 0 where that is left to the chain: extents of kNextLimit requests
// or more (a place costs up to kNextLimit / 256 turns, all of them together less than the 3 us that the chain takes for a batch of
// that many; such a place is recognised by one sum), and of kNextMax where the profile test is made here.  With 256 for both, 100000 bimodal
// requests in 197 batches of 510 were 554 us of chain.  (100000 chat requests in 16 batches, all but two beyond the limit: 261 -> 267.)
// The zeros behind the last batch are written here, ahead of the batches, by the whole chip (by the chain's one workgroup 100000 requests
// took 227 us a call instead of 213, 40000 146 instead of 141, 10000 66 instead of 65).
template <bool PROFILE>
__global__ __launch_bounds__(256) void next_batch_kernel(SortedArgs p, LargeArrays m)
{
    if (p.pad && threadIdx.x < 4) {
        const int b = blockIdx.x * 4 + (int)threadIdx.x;
        if (b < p.n) p.batch_end_out[b] = 0, p.F_out[b] = 0.0;
    }
    if (faulty(p)) return;
    const int a = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (a >= p.n) return;
    const Sums c{m.W, m.S, m.G, m.s_pos, m.o_pos};
    const bool small = small_numbers(p, c);
    int rem = p.n - a;
    u64 M = (u64)p.M;
    int k = 0;
    const bool ahead = PROFILE && extents_ahead(p, m);
    const int limit = PROFILE && !ahead ? kNextMax : kNextLimit;
    // (a sum of peaks that holds so many requests or more is feasible: nothing to decide here)
    if (rem >= limit && c.W[a + limit] - c.W[a] <= M) rem = -1;
    if constexpr (PROFILE) {
        if (rem > 0) rem = ahead ? m.extent[a] : wave_profile_extent(c, a, rem, (unsigned)M);
        if (rem >= limit) rem = -1;
        M = ~0ull;
    }
    if (rem > 0) k = small ? wave_batch<true>(c, a, rem, M, p.tie_rule) : wave_batch<false>(c, a, rem, M, p.tie_rule);
    if ((threadIdx.x & 63) == 0) m.next[a] = (unsigned short)(k > 0 && k < limit ? k : 0);
}

// The chain of batches by one workgroup: the small ones are read off next[], of which LDS holds the part the chain is in,
// the others found by all threads.
template <bool PROFILE>
__global__ __launch_bounds__(1024) void batch_chain_kernel(SortedArgs p, LargeArrays m, int window)
{
    extern __shared__ u64 lds64[];
    __shared__ u64 red_S[16];
    __shared__ int red_k[16], sh[2];
    __shared__ unsigned wave_c[16], wave_s[16];
    const int tid = threadIdx.x, n = p.n;
    if (faulty(p)) {
        if (tid == 0) *p.num_batches_out = 0;
        return;
    }
    const Sums c{m.W, m.S, m.G, m.s_pos, m.o_pos};
    const bool small = small_numbers(p, c);
    const u64 M = (u64)p.M;
    const bool ahead = PROFILE && extents_ahead(p, m), tests = PROFILE && !ahead;  // profile tests are made here
    unsigned *hist_lds = (unsigned *)lds64;
    unsigned short *next_in = (unsigned short *)((char *)lds64 + (PROFILE ? 16 * kLargeBuckets : 0));
    int first = 0;  // next_in holds the places [first, first + window), once there is use for them (80 KB take one workgroup 8 us)
    bool loaded = tests;
    auto load_window = [&](int from) __attribute__((always_inline)) {  // eight places at a time (next[] is as long as that takes)
        first = from & ~7;
        for (int i = tid; i < (min(window, n - first) + 7) / 8; i += 1024) ((uint4 *)next_in)[i] = ((const uint4 *)(m.next + first))[i];
    };
    if (loaded) load_window(0);
    const bool by_rank = p.words[KVS_W_OMAX] > kLargeBuckets;  // (then the ranks are there)
    const int *rank_pos = by_rank ? m.rank_pos : nullptr;
    const int buckets = by_rank ? n : p.words[KVS_W_OMAX];
    if (tests) {
        for (int i = tid; i < 4 * kLargeBuckets; i += 1024) hist_lds[i] = 0;
        if (buckets > kLargeBuckets) {
            for (int i = tid; i < 4 * n; i += 1024) m.hist[i] = 0;
        }
    }
    __syncthreads();
    int a = 0, nb = 0;
    while (a < n) {
        if (loaded && a >= first + window) {
            load_window(a);
            __syncthreads();
        }
        if (loaded && tid < 64) {  // follow the chain as far as it is known
            // (by scalars, which the compiler cannot tell by itself: with a branch by the lane in each step the loop's time hung on where in the
            // instruction cache it lay, e.g. 4000 requests in 1691 batches under the profile constraint 225 or 243 us a call; 207 so)
            int at = __builtin_amdgcn_readfirstlane(a), b = __builtin_amdgcn_readfirstlane(nb);
            const int known_to = __builtin_amdgcn_readfirstlane(min(n, first + window));
            while (at < known_to) {
                const int k = __builtin_amdgcn_readfirstlane((int)next_in[at - first]);
                if (k < 1) break;
                at += k;
                if (tid == 0) p.batch_end_out[b] = at;
                ++b;
            }
            if (tid == 0) sh[0] = at, sh[1] = b;
        }
        if (loaded) {
            __syncthreads();
            a = sh[0];
            nb = sh[1];
            if (a >= n) break;
            if (a >= first + window) continue;
        }
        int K;
        if constexpr (!PROFILE) {
            const u64 W0 = c.W[a];
            K = count_fitting(n - a, [&](int k) { return c.W[a + k] - W0; }, M);
        } else if (ahead) {
            K = m.extent[a];
        } else if (buckets <= kLargeBuckets) {
            Profile<true> prof{hist_lds, hist_lds + kLargeBuckets, hist_lds + 2 * kLargeBuckets, hist_lds + 3 * kLargeBuckets,
                               buckets, rank_pos, m.o_of_rank};
            K = prof.extent(c, a, n - a, (unsigned)M, wave_c, wave_s);
        } else {
            Profile<false> prof{m.hist, m.hist + n, m.hist + 2 * (size_t)n, m.hist + 3 * (size_t)n, buckets, rank_pos, m.o_of_rank};
            K = prof.extent(c, a, n - a, (unsigned)M, wave_c, wave_s);
        }
        if (!loaded && K < kNextLimit) {  // from here on batches may be known
            load_window(a);
            loaded = true;
            __syncthreads();
            continue;
        }
        int k;  // (likely, so that the other form's code lies behind the loop: 100000 bimodal requests in 197 batches 241 us without)
        if (__builtin_expect(small, 1)) k = group_argmin<true>(c, a, K, p.tie_rule, red_S, red_k);
        else k = group_argmin<false>(c, a, K, p.tie_rule, red_S, red_k);
        if (k < 1) {  // cannot happen for well-formed input; never spin
            if (tid == 0) atomicOr(&p.words[KVS_W_STATUS], KVSCHED_DEV_BAD_LENGTH);
            break;
        }
        a += k;
        if (tid == 0) p.batch_end_out[nb] = a;
        ++nb;
    }
    __threadfence_block();
    __syncthreads();
    if (tid == 0) *p.num_batches_out = nb;
    for (int b = tid; b < nb; b += 1024) {
        const int lo = b == 0 ? 0 : p.batch_end_out[b - 1], hi = p.batch_end_out[b];
        const double k = (double)(hi - lo);
        p.F_out[b] = (double)(m.G[hi] - m.G[lo]) / ((double)p.gb * k * k);
    }
}

int ok() { return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP; }

template <int TPB, int E, bool PROFILE>
int launch_small(const SortedArgs &p, hipStream_t st)
{
    constexpr size_t bytes = small_lds_bytes(TPB * E, PROFILE);
    if constexpr (bytes > 64 * 1024) {
        static const hipError_t granted = hipFuncSetAttribute((const void *)sortedF_small_kernel<TPB, E, PROFILE>,
                                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (granted != hipSuccess) return KVSCHED_EHIP;
    }
    hipLaunchKernelGGL((sortedF_small_kernel<TPB, E, PROFILE>), dim3(1), dim3(TPB), bytes, st, p);
    return ok();
}

// Merge sorted runs of kRun keys of m.key[0] (through m.key[1] and back) to the end; returns where the keys are
// (EMIT other than MERGE_KEYS: the last pass emits instead and the result is void).  by_o: two arrays with the runs by (o, id) in
// the first, merged beside them, or null.
template <int EMIT>
const u64 *launch_merges(const SortedArgs &p, const LargeArrays &m, u64 *const *by_o, hipStream_t st)
{
    const dim3 grid((unsigned)((p.n + 255) / 256), by_o ? 2u : 1u), block(256);
    int at = 0;
    for (long long run = kRun; run < p.n; run *= kFan) {
        const bool last = run * kFan >= p.n;
        const u64 *const from = by_o ? by_o[at] : nullptr;
        u64 *const to = by_o ? by_o[at ^ 1] : nullptr;
        if (last) hipLaunchKernelGGL((merge_runs_kernel<EMIT>), grid, block, 0, st, p, m, m.key[at], m.key[at ^ 1], (int)run, EMIT == MERGE_RANKS, from, to);
        else hipLaunchKernelGGL((merge_runs_kernel<MERGE_KEYS>), grid, block, 0, st, p, m, m.key[at], m.key[at ^ 1], (int)run, EMIT == MERGE_RANKS, from, to);
        at ^= 1;
    }
    return m.key[at];
}

template <int OWN>
int launch_count(const SortedArgs &p, const LargeArrays &m, int what, bool beside, bool scan, u64 *out, hipStream_t st)
{
    static const hipError_t granted = hipFuncSetAttribute((const void *)count_places_kernel<OWN>,
                                                          hipFuncAttributeMaxDynamicSharedMemorySize, 8 * kCountMax);
    if (granted != hipSuccess) return KVSCHED_EHIP;
    constexpr int turn = 8 * 1024 / OWN;
    static_assert(kCountMax % turn == 0 && 8 * kCountMax + 1024 <= 160 * 1024, "fits the LDS");
    const int padded = (p.n + turn - 1) / turn * turn;
    hipLaunchKernelGGL(count_places_kernel<OWN>, dim3((unsigned)((p.n + OWN - 1) / OWN), beside ? 2u : 1u), dim3(1024), 8 * padded, st, p, m,
                       what, scan ? 1 : 0, out);
    return ok();
}

// The sorted keys by size (and the ranks in the (o, id) order where they may be needed); returns where they are.
int launch_places(const SortedArgs &p, LargeArrays &m, bool ranks, const u64 **sorted, hipStream_t st)
{
    const bool beside = ranks && p.packed;  // (otherwise the keys by size hold ranks)
    if (p.n <= kCountMax) {
        // 32 requests a workgroup up to as many workgroups as compute units
        auto count = [&](int what, bool both, bool scan) {
            return p.n <= 32 * 256 ? launch_count<32>(p, m, what, both, scan, m.key[0], st)
                                   : launch_count<64>(p, m, what, both, scan, m.key[0], st);
        };
        int rc = KVSCHED_OK;
        if (ranks && !beside) rc = count(KEYS_BY_O, false, true);
        if (rc == KVSCHED_OK) rc = count(KEYS_BY_SIZE, beside, !ranks || beside);
        *sorted = m.key[0];
        return rc;
    }
    const dim3 runs((unsigned)((p.n + kRun - 1) / kRun)), both(runs.x, 2);
    u64 *const by_o[2] = {m.W, m.S};  // (not in use yet)
    if (ranks && !beside) {
        hipLaunchKernelGGL((sort_runs_kernel<KEYS_BY_O>), runs, dim3(1024), 0, st, p, m, 1, m.key[0], (u64 *)nullptr);
        (void)launch_merges<MERGE_RANKS>(p, m, nullptr, st);
    }
    hipLaunchKernelGGL((sort_runs_kernel<KEYS_BY_SIZE>), beside ? both : runs, dim3(1024), 0, st, p, m, !ranks || beside ? 1 : 0, m.key[0], by_o[0]);
    *sorted = launch_merges<MERGE_KEYS>(p, m, beside ? by_o : nullptr, st);
    return ok();
}

template <bool PROFILE>
int launch_chain(const SortedArgs &p, const LargeArrays &m, hipStream_t st)
{
    constexpr int most = 2 * kNextWindow;
    static_assert(most + 4096 <= 160 * 1024 && kNextWindow % 8 == 0, "fits the LDS");
    static const hipError_t granted = hipFuncSetAttribute((const void *)batch_chain_kernel<PROFILE>,
                                                          hipFuncAttributeMaxDynamicSharedMemorySize, most);
    if (granted != hipSuccess) return KVSCHED_EHIP;
    const int window = PROFILE ? kNextWindow - 8 * kLargeBuckets : kNextWindow;
    const int bytes = (PROFILE ? 16 * kLargeBuckets : 0) + 2 * (p.n < window ? (p.n + 7) & ~7 : window);
    hipLaunchKernelGGL((batch_chain_kernel<PROFILE>), dim3(1), dim3(1024), bytes, st, p, m, window);
    return ok();
}

int bits_for(long long v)  // bits that hold 0..v
{
    int b = 1;
    while (b < 62 && (v >> b) != 0) ++b;
    return b;
}

size_t padded(int32_t n) { return ((size_t)n + 64) & ~(size_t)63; }

}  // namespace

// Largest construction done by one workgroup.  Its sorts and the chain grow with the requests and batches, most of the chip's launches
// do not.  Mixed requests in 6 / 20 / 40 batches, one workgroup and the chip: 700 17 / 22 / 30 us against 26 for all; 1025 (two keys a
// thread) 30 / 38 / 87 before the chain was one wavefront's, 27 / 27 / 29 by the chip; 2000 31 / 34 / 40 and 32 / 30 / 31; 4000 55 / 59 /
// 63 and 43 / 38 / 37.  The other way, chat requests in 4 batches: 1100 28.3 and 29.2, 2000 30.3 and 32.2.  Under the profile constraint,
// where one workgroup finds one extent after the other and the chip those of all places: 129 chat requests in 3 / 6 / 25 batches 28 / 30 /
// 48 and 32 / 28 / 29, 200 in 3 / 4 / 14 34 / 34 / 43 and 37 / 33 / 29, 256 mixed ones in 8 / 16 / 67 41 / 49 / 100 and 37 / 37 / 40.  100
// chat requests in 2 / 4 / 17 batches 23.5 / 25 / 38 and 27 / 24 / 24, 65 in 3 / 6 / 13 22 / 25 / 32 and 23 / 22 / 23: from some 4 batches
// on the line could be as low as 64.
int32_t kvs_sortedF_small_max(int32_t feas_mode) { return feas_mode == KVSCHED_FEAS_PROFILE ? kSmallProfile : kSmallSum; }

size_t kvs_sortedF_scratch_bytes(int32_t n)
{
    if (n <= kvs_sortedF_small_max(KVSCHED_FEAS_PROFILE)) return 256;
    const size_t np = padded(n);
    // two key arrays and three sums; block sums; six arrays of ints, four of profile buckets; two bytes each
    return np * 5 * sizeof(u64) + (2 * sizeof(u64)) * (np / 4096 + 1) + np * 10 * sizeof(int) + 2 * np + 1024;
}

// (The first launch scans the lengths as well: status word and longest decode.)
int kvs_launch_sortedF(int32_t n, const int32_t *s, const int32_t *o, int32_t M, int32_t ga, int32_t gb,
                       int32_t tie_rule, int32_t feas_mode, int32_t pad, int32_t *order_out, int32_t *batch_end_out,
                       double *F_out, int32_t *num_batches_out, void *scratch, int32_t *d_words, hipStream_t st)
{
    SortedArgs p;
    p.n = n;
    p.s = s;
    p.o = o;
    p.M = M;
    p.ga = ga;
    p.gb = gb;
    p.tie_rule = tie_rule;
    p.order_out = order_out;
    p.batch_end_out = batch_end_out;
    p.F_out = F_out;
    p.num_batches_out = num_batches_out;
    p.words = d_words;
    p.id_bits = bits_for(n - 1);
    p.o_bits = bits_for(M);
    // the keys (s+o, o, id) and (batch, o, id) in 64 bits, and not all ones (that stands for "no key")
    p.packed = 2 * p.o_bits + p.id_bits <= 63 && p.o_bits + 2 * p.id_bits <= 63;
    p.pad = pad;
    const bool profile = feas_mode == KVSCHED_FEAS_PROFILE;
    // One workgroup: as few wavefronts as hold the keys one each (a barrier costs by the wavefront).
    if (n <= kvs_sortedF_small_max(feas_mode)) {
        if (profile) {
            if (n <= 64) return launch_small<64, 1, true>(p, st);
            return launch_small<1024, 1, true>(p, st);
        }
        if (n <= 64) return launch_small<64, 1, false>(p, st);
        if (n <= 256) return launch_small<256, 1, false>(p, st);
        return launch_small<1024, 1, false>(p, st);
    }
    const size_t np = padded(n);
    LargeArrays m;
    u64 *q = (u64 *)scratch;
    m.key[0] = q;
    m.key[1] = q + np;
    m.W = q + 2 * np;
    m.S = q + 3 * np;
    m.G = q + 4 * np;
    m.tot = q + 5 * np;
    int *i = (int *)(m.tot + 2 * (np / 4096 + 1));
    m.s_pos = i;
    m.o_pos = i + np;
    m.by_o = i + 2 * np;
    m.rank_of = i + 3 * np;
    m.rank_pos = i + 4 * np;
    m.o_of_rank = i + 5 * np;
    m.hist = (unsigned *)(i + 6 * np);
    m.extent = (int *)m.hist;
    m.next = (unsigned short *)(i + 10 * np);
    // Ranks in the (o, id) order are needed by keys that do not fit and, under the profile constraint, when completion
    // times may be too many for buckets in LDS.
    const bool ranks = !p.packed || (profile && M > kLargeBuckets);
    const u64 *sorted = nullptr;
    int rc = launch_places(p, m, ranks, &sorted, st);
    if (rc != KVSCHED_OK) return rc;
    if (sorted != m.key[1]) {  // (the batches' keys are written beside them)
        m.key[0] = m.key[1];
        m.key[1] = (u64 *)sorted;
    }
    const dim3 sums((unsigned)((n + 4095) / 4096));
    if (n > kSumsHere) hipLaunchKernelGGL(place_sums_kernel, sums, dim3(1024), 0, st, p, m, sorted);
    hipLaunchKernelGGL(prefix_sums_kernel, sums, dim3(1024), 0, st, p, m, sorted, ranks ? 1 : 0, n > kSumsHere ? 1 : 0);
    const dim3 waves((unsigned)((n + 3) / 4));
    // (as many workgroups as the LDS of 256 compute units holds)
    if (profile && n > kNextMax) hipLaunchKernelGGL(profile_extents_kernel, dim3((unsigned)(n < 3 * 256 ? n : 3 * 256)), dim3(128), 0, st, p, m);
    if (profile) hipLaunchKernelGGL((next_batch_kernel<true>), waves, dim3(256), 0, st, p, m);
    else hipLaunchKernelGGL((next_batch_kernel<false>), waves, dim3(256), 0, st, p, m);
    rc = profile ? launch_chain<true>(p, m, st) : launch_chain<false>(p, m, st);
    if (rc != KVSCHED_OK) return rc;
    if (n <= kCountMax) {
        hipLaunchKernelGGL(order_batches_kernel, dim3((unsigned)((n + 63) / 64)), dim3(1024), 0, st, p, m, sorted);
    } else {
        hipLaunchKernelGGL(sort_batch_runs_kernel, dim3((unsigned)((n + kRun - 1) / kRun)), dim3(1024), 0, st, p, sorted, m.key[0]);
        (void)launch_merges<MERGE_IDS>(p, m, nullptr, st);
    }
    return ok();
}
