// Phase 2 under predicted decode lengths (Section 5, "Handling Prediction Uncertainty via Adaptive
// Output Length Refinement"; appendix algorithm "Sorted-F + A_min"), many candidate orders at once,
// one 64-lane wavefront per candidate.
//
// The scheduler does not know o_i.  It holds a running estimate e_i (started from the caller's
// est0: lower bounds for A_min, upper bounds for the conservative A_max) and runs the admission
// of Algorithm 1's Phase 2 on the memory the running requests are PROJECTED to hold; round t:
//   1. a running request that has produced a = t - p tokens leaves if a = o_i, else needs one
//      more: e_i <- max(e_i, a + 1);
//   2. waiting requests are started in the order's sequence while the projection stays <= M;
//   3. while the projection exceeds M, the running request of least (e_i, i) is stopped; it keeps
//      e_i, loses its progress and waits again at its own place of the order.
//
// State of a candidate (one wavefront per workgroup):
//   * the projected memory of the requests that are still inside their estimate: in vector registers up to 4096 rounds
//     (Rows), as a ring in LDS beyond (Ring);
//   * the requests that have outrun their estimate are not in there: each of them reserves
//     exactly the next round, s_j + (t + 1 - p_j), so two scalars (their count and the sum of
//     s_j - p_j) give their share of round t + 1, and a round costs nothing per such request;
//   * per position of the order only what changes and must outlive a stop: one bit "waits" (every
//     position from `frontier` on waits and none of them was ever started, so the bits are looked
//     at only after a request was stopped).  The estimate a stopped request keeps is needed twice
//     per stop (written when it is stopped, read when it is looked at again), so it lives in
//     global memory, 16 bits per position and candidate, written and read by the same wavefront;
//     a position that was never started takes its estimate from est0;
//   * the RUNNING requests as a compact unordered list of entries in LDS, ten bytes each: position | id << 16,
//     o | estimate << 16 and, in an array of its own, the low 16 bits of the round at which the entry next
//     matters: it reaches its estimate or its true length, start + min(estimate, o), or start + o
//     once it has outrun its estimate.  The start round follows from that (a running request
//     started at most o <= 16384 rounds ago, so 16 bits and the current round give the round
//     itself), s from the length table when an entry is handled.  Entries that finish leave holes, which the others of
//     their tile of 64 and the list's last entries fill.
// Lengths and ids of the waiting positions are not kept at all: admission walks the order from the
// front, so the 64 positions around the first waiting one sit in registers (one position per lane,
// fetched from the order row and the length tables when the walk leaves the window).
// What bounds the call is the number of candidates in flight times the chain of dependent instructions each is (2000 mixed
// requests: 380 k vector and 475 k scalar instructions; four candidates share a SIMD, whose scalar unit is 65 % busy, and wait for
// memory, LDS and branches a third of the time).  Hence no branch of the loop over rounds depends on the lane with Rows (see
// lane_mask.h; the passes over a Ring are loops from the lane's round on), tiles of the list are read two at a time, and what scalars would
// add up entry by entry is added up a lane each: 613 k and 759 k instructions before; 4096 / 256 / 16 candidates 7.58 / 6.42 / 5.10 ->
// 4.75 / 3.79 / 2.98 ms, 1024 of 2000 chat requests 7.94 -> 4.81; with a Ring (decodes four times as long) 2048 / 512 / 16 of 2000 mixed
// requests 65.7 / 22.3 / 21.3 -> 50.2 / 16.8 / 16.0, 1024 of 500 chat requests 5.7 -> 4.7.  And the
// list decides how many candidates fit a compute unit: a first launch runs every candidate with a list of at
// most `cap` entries (launch_variant); a candidate whose list overflows gives up and is run again by a second launch
// whose list holds all n positions.
// A blocked request is not re-examined round by round: the search over the projection gives the earliest
// start its reservations allow, and that bound holds until memory is released (an eviction, or a
// request that finishes before its estimate), whoever outruns an estimate meanwhile.
#include "kvsched_internal.h"
#include "lane_mask.h"

#include <limits.h>

namespace {

constexpr int PW = 64;
constexpr int EST_OVERRUN = 0;  // estimate field of a request that has outrun it: e = t - p + 1

struct PredParams {
    const int32_t *orders;  // [C][n]
    int32_t C, n;
    const int32_t *s, *o;
    const int32_t *est0;  // [E][n]
    int32_t E;
    int32_t M;
    int32_t H;            // power of two >= every estimate and every o
    int32_t cap;          // entries of the running list (even)
    int32_t second;       // 0: every candidate, overflow sets retry[c]; 1: only candidates with retry[c] != 0
    int32_t *retry;       // [C]
    unsigned short *est_stopped;  // [C][n]: estimate kept by a stopped request, by position
    int32_t step_back;    // candidates that run at a time, if they give way near their ends (0: they do not)
    int32_t round_limit;  // a run that lasts longer is reported, not continued
    int64_t *tel_out;         // [C]
    int32_t *completion_out;  // [C][n] by request id, or NULL
    int32_t *evictions_out;   // [C] or NULL
    int32_t *d_words;
};

__device__ __forceinline__ int p_uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ void p_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Minimum over the 64 lanes by lane exchanges inside the vector unit (four steps within the rows of
// 16 lanes, two row broadcasts; lane 63 ends up with the result).
__device__ __forceinline__ int p_wave_min(int v)
{
    // (lanes that receive nothing compare with the largest number, which lets the exchange be part of the comparison)
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0xB1, 0xf, 0xf, false));   // quad_perm [1,0,3,2]
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x4E, 0xf, 0xf, false));   // quad_perm [2,3,0,1]
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x141, 0xf, 0xf, false));  // row_half_mirror
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x140, 0xf, 0xf, false));  // row_mirror
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x142, 0xa, 0xf, false));  // row_bcast:15 into rows 1 and 3
    v = min(v, __builtin_amdgcn_update_dpp(INT_MAX, v, 0x143, 0xc, 0xf, false));  // row_bcast:31 into rows 2 and 3
    return __builtin_amdgcn_readlane(v, 63);
}

// Sum over the 64 lanes (modulo 2^32).
__device__ __forceinline__ int p_wave_sum(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return __builtin_amdgcn_readlane(v, 63);
}

// The projected memory in vector registers (H <= 4096): row r of lane l is round b + 64 r + l, with b
// kept at 64 floor((t + 1) / 64), so that round t + 1 lies in row 0 and every loop over rounds names its registers at
// compile time; when t passes a multiple of 64 the rows move down by one.  Rounds at or before t keep stale values.
// With a ring and entries of 14 bytes in LDS eight candidates fit a compute unit (two wavefronts per SIMD, some nine
// cycles an instruction); 10 KB a candidate without the ring let sixteen in.  4096 candidates of n = 2000, M = 131072:
// 16.1 -> 9.4 ms.
//
// The rows live in physical vector registers (KVP_PB upward) that only the assembly statements
// below touch: a C++ array of this size under this kernel's control flow becomes copies of the whole file at every way
// out of a loop over rows.  The compiler's own registers have to stay below the block, which the build checks on the
// emitted assembly (as for the timeline kernel).  Every statement waits out what the compiler may have issued just before
// (an SGPR written by a vector instruction needs two instructions, as a lane select four, before it is used) and keeps two
// instructions between a compare and the use of VCC.  A pass over rows ends when the rounds left run out.
#define KVP_PB "60"
#define KVP_CLOB_9 "v60", "v61", "v62", "v63", "v64", "v65", "v66", "v67", "v68"
#define KVP_CLOB_17 KVP_CLOB_9, "v69", "v70", "v71", "v72", "v73", "v74", "v75", "v76"
#define KVP_CLOB_33 KVP_CLOB_17, "v77", "v78", "v79", "v80", "v81", "v82", "v83", "v84", "v85", "v86", "v87", "v88", "v89", "v90",  \
    "v91", "v92"
#define KVP_CLOB_65 KVP_CLOB_33, "v93", "v94", "v95", "v96", "v97", "v98", "v99", "v100", "v101", "v102", "v103", "v104", "v105",  \
    "v106", "v107", "v108", "v109", "v110", "v111", "v112", "v113", "v114", "v115", "v116", "v117",  \
    "v118", "v119", "v120", "v121", "v122", "v123", "v124"

#define KVP_FOR_NR(STMT)                                                                 \
    do {                                                                                 \
        static_assert(NR == 9 || NR == 17 || NR == 33 || NR == 65, "register files");    \
        if constexpr (NR == 9) {                                                         \
            STMT(KVP_CLOB_9);                                                            \
        } else if constexpr (NR == 17) {                                                 \
            STMT(KVP_CLOB_17);                                                           \
        } else if constexpr (NR == 33) {                                                 \
            STMT(KVP_CLOB_33);                                                           \
        } else {                                                                         \
            STMT(KVP_CLOB_65);                                                           \
        }                                                                                \
    } while (0)

template <int NR>
__device__ __forceinline__ void rows_clear()
{
#define KVP_STMT(CLOB)                                    \
    asm volatile(".set kvs_r, 0\n"                        \
                 ".rept %c[nr]\n"                         \
                 "  v_mov_b32 v[" KVP_PB "+kvs_r], 0\n"   \
                 "  .set kvs_r, kvs_r+1\n"                \
                 ".endr\n"                                \
                 :                                        \
                 : [nr] "n"(NR)                           \
                 : CLOB)
    KVP_FOR_NR(KVP_STMT);
#undef KVP_STMT
}

// every row takes the next one's place; an empty one enters
template <int NR>
__device__ __forceinline__ void rows_down()
{
#define KVP_STMT(CLOB)                                                          \
    asm volatile(".set kvs_r, 0\n"                                              \
                 ".rept %c[nr]-1\n"                                             \
                 "  v_mov_b32 v[" KVP_PB "+kvs_r], v[" KVP_PB "+kvs_r+1]\n"     \
                 "  .set kvs_r, kvs_r+1\n"                                      \
                 ".endr\n"                                                      \
                 "v_mov_b32 v[" KVP_PB "+%c[nr]-1], 0\n"                        \
                 :                                                              \
                 : [nr] "n"(NR)                                                 \
                 : CLOB)
    KVP_FOR_NR(KVP_STMT);
#undef KVP_STMT
}

// Rows += first + j for the rounds with 0 <= j < count (j: the lane's in row 0); left >= 0: the last of those rounds as
// row and lane.  Returns the most any row visited holds afterwards.
template <int NR>
__device__ __forceinline__ int rows_add(int left, int j, int count, int first)
{
    int most, y;
#define KVP_STMT(CLOB)                                                              \
    asm volatile("s_nop 4\n"                                                        \
                 "v_mov_b32 %[most], 0\n"                                           \
                 ".set kvs_r, 0\n"                                                  \
                 ".rept %c[nr]\n"                                                   \
                 "  v_cmp_gt_u32 vcc, %[count], %[j]\n"                             \
                 "  v_add_u32 %[y], %[first], %[j]\n"                               \
                 "  v_add_u32 %[j], 64, %[j]\n"                                     \
                 "  v_cndmask_b32 %[y], 0, %[y], vcc\n"                             \
                 "  v_add_u32 v[" KVP_PB "+kvs_r], %[y], v[" KVP_PB "+kvs_r]\n"     \
                 "  v_max_i32 %[most], %[most], v[" KVP_PB "+kvs_r]\n"              \
                 "  s_sub_u32 %[left], %[left], 64\n"                               \
                 "  s_cbranch_scc1 9f\n"                                            \
                 "  .set kvs_r, kvs_r+1\n"                                          \
                 ".endr\n"                                                          \
                 "9:\n"                                                             \
                 : [most] "=&v"(most), [y] "=&v"(y), [j] "+v"(j), [left] "+s"(left) \
                 : [count] "s"(count), [first] "s"(first), [nr] "n"(NR)             \
                 : "vcc", "scc", CLOB)
    KVP_FOR_NR(KVP_STMT);
#undef KVP_STMT
    return most;
}

// ... and the same taken off again.
template <int NR>
__device__ __forceinline__ void rows_take(int left, int j, int count, int first)
{
    int y;
#define KVP_STMT(CLOB)                                                              \
    asm volatile("s_nop 4\n"                                                        \
                 ".set kvs_r, 0\n"                                                  \
                 ".rept %c[nr]\n"                                                   \
                 "  v_cmp_gt_u32 vcc, %[count], %[j]\n"                             \
                 "  v_add_u32 %[y], %[first], %[j]\n"                               \
                 "  v_add_u32 %[j], 64, %[j]\n"                                     \
                 "  v_cndmask_b32 %[y], 0, %[y], vcc\n"                             \
                 "  v_sub_u32 v[" KVP_PB "+kvs_r], v[" KVP_PB "+kvs_r], %[y]\n"     \
                 "  s_sub_u32 %[left], %[left], 64\n"                               \
                 "  s_cbranch_scc1 9f\n"                                            \
                 "  .set kvs_r, kvs_r+1\n"                                          \
                 ".endr\n"                                                          \
                 "9:\n"                                                             \
                 : [y] "=&v"(y), [j] "+v"(j), [left] "+s"(left)                     \
                 : [count] "s"(count), [first] "s"(first), [nr] "n"(NR)             \
                 : "vcc", "scc", CLOB)
    KVP_FOR_NR(KVP_STMT);
#undef KVP_STMT
}

// Per lane: the largest min(tq, row + bias + tq) over its rounds tq with 0 <= k <= span (k, tq: the lane's in row 0).
template <int NR>
__device__ __forceinline__ int rows_bound(int left, int k, int span, int tq, int bias)
{
    int acc, y, none;
#define KVP_STMT(CLOB)                                                                       \
    asm volatile("s_nop 4\n"                                                                 \
                 "v_mov_b32 %[none], 0x80000001\n"                                           \
                 "v_mov_b32 %[acc], %[none]\n"                                               \
                 ".set kvs_r, 0\n"                                                           \
                 ".rept %c[nr]\n"                                                            \
                 "  v_cmp_ge_u32 vcc, %[span], %[k]\n"                                       \
                 "  v_add_u32 %[y], %[bias], %[tq]\n"                                        \
                 "  v_add_u32 %[y], %[y], v[" KVP_PB "+kvs_r]\n"                             \
                 "  v_min_i32 %[y], %[tq], %[y]\n"                                           \
                 "  v_cndmask_b32 %[y], %[none], %[y], vcc\n"                                \
                 "  v_max_i32 %[acc], %[acc], %[y]\n"                                        \
                 "  v_add_u32 %[k], 64, %[k]\n"                                              \
                 "  v_add_u32 %[tq], 64, %[tq]\n"                                            \
                 "  s_sub_u32 %[left], %[left], 64\n"                                        \
                 "  s_cbranch_scc1 9f\n"                                                     \
                 "  .set kvs_r, kvs_r+1\n"                                                   \
                 ".endr\n"                                                                   \
                 "9:\n"                                                                      \
                 : [acc] "=&v"(acc), [y] "=&v"(y), [none] "=&v"(none), [k] "+v"(k), [tq] "+v"(tq), [left] "+s"(left) \
                 : [span] "s"(span), [bias] "s"(bias), [nr] "n"(NR)                          \
                 : "vcc", "scc", CLOB)
    KVP_FOR_NR(KVP_STMT);
#undef KVP_STMT
    return acc;
}

// Lane `at` of row 0.
template <int NR>
__device__ __forceinline__ int row0_lane(int at)
{
    int v;
#define KVP_STMT(CLOB)                                        \
    asm volatile("s_nop 4\n"                                  \
                 "v_readlane_b32 %[v], v[" KVP_PB "], %[at]\n" \
                 : [v] "=s"(v)                                \
                 : [at] "s"(at)                               \
                 : CLOB)
    KVP_FOR_NR(KVP_STMT);
#undef KVP_STMT
    return v;
}

// The first row, of those that `left` (the last round as row and lane) lets in, in which a round's total, what the row holds and `held` together,
// exceeds M, or is at most `fit` and the row is none before the lane's `from`: its rounds as a mask (0: no such row) and 64 times its number.
// In row 0 only the lanes of `lanes` count.  held grows by `step` from row to row.  (Ten instructions a row; with a computed jump to
// each row some forty: 4096 candidates of 2000 mixed requests 4760 -> 4690 us, 95 of 2383 4280 -> 4210.)
template <int NR>
__device__ __forceinline__ unsigned long long rows_event(int left, int held, int step, int M, int fit, int from, unsigned long long lanes, int &at)
{
    unsigned long long out, in, on;
    int x;
    at = 0;
#define KVP_STMT(CLOB)                                                                  \
    asm volatile("s_nop 4\n"                                                            \
                 ".set kvs_r, 0\n"                                                      \
                 ".rept %c[nr]\n"                                                       \
                 "  v_add_u32 %[x], %[held], v[" KVP_PB "+kvs_r]\n"                     \
                 "  v_cmp_ge_u32 %[on], kvs_r, %[from]\n"                               \
                 "  v_cmp_lt_u32 %[out], %[M], %[x]\n"                                  \
                 "  v_cmp_ge_u32 %[in], %[fit], %[x]\n"                                 \
                 "  v_add_u32 %[held], %[step], %[held]\n"                              \
                 "  s_and_b64 %[in], %[in], %[on]\n"                                    \
                 "  s_or_b64 %[out], %[out], %[in]\n"                                   \
                 "  .if kvs_r == 0\n"                                                   \
                 "    s_and_b64 %[out], %[out], %[lanes]\n"                             \
                 "  .endif\n"                                                           \
                 "  s_cbranch_scc1 9f\n"                                                \
                 "  s_sub_u32 %[left], %[left], 64\n"                                   \
                 "  s_cbranch_scc1 9f\n"                                                \
                 "  s_add_u32 %[at], %[at], 64\n"                                       \
                 "  .set kvs_r, kvs_r+1\n"                                              \
                 ".endr\n"                                                              \
                 "9:\n"                                                                 \
                 : [out] "=&s"(out), [in] "=&s"(in), [on] "=&s"(on), [x] "=&v"(x), [held] "+v"(held), [left] "+s"(left), [at] "+s"(at) \
                 : [step] "s"(step), [M] "s"(M), [fit] "s"(fit), [from] "v"(from), [lanes] "s"(lanes), [nr] "n"(NR) \
                 : "scc", CLOB)
    KVP_FOR_NR(KVP_STMT);
#undef KVP_STMT
    return out;
}

// The two forms of the projected memory.  Rounds past t only; every lane touches the same rounds in add() and take() at
// one t.
template <int NR>
struct Rows {
    static constexpr int H = 64 * (NR - 1);  // longest estimate and decode length
    int lane, b;

    static __device__ __forceinline__ int lds_words(int) { return 0; }
    __device__ __forceinline__ Rows(int *, int, int lane_) : lane(lane_), b(0) { rows_clear<NR>(); }
    __device__ __forceinline__ int longest() const { return H; }
    // the present round goes on from t to `to`: rows move down while row 0 ends before round to + 1
    __device__ __forceinline__ void advance(int, int to)
    {
        const int nb = p_uni((to + 1) & ~63);
        if (nb - b >= 64 * NR) {
            rows_clear<NR>();
            b = nb;
        }
        for (; b < nb; b += 64) rows_down<NR>();
    }
    // s + j into the rounds t + j, j = 1 .. count; does one of them hold more than M now?  (No reservation exceeds M, so a
    // round above M afterwards is one of these.)
    __device__ __forceinline__ bool add(int t, int s, int count, int M)
    {
        const int most = rows_add<NR>(p_uni(t + count - b), b + lane - t - 1, p_uni(count), p_uni(s + 1));
        return __builtin_amdgcn_ballot_w64(most > M) != 0;
    }
    // s + (tq - ps) off the rounds tq = t + 1 .. last
    __device__ __forceinline__ void take(int t, int s, int ps, int last)
    {
        rows_take<NR>(p_uni(last - b), b + lane - t - 1, p_uni(last - t), p_uni(s + t + 1 - ps));
    }
    // reserved for round t + 1
    __device__ __forceinline__ int next_round(int t) const { return row0_lane<NR>(p_uni((t + 1) & 63)); }
    // per lane: the largest min(tq, reserved + bias + tq) over its rounds tq = lo .. hi
    __device__ __forceinline__ int bound(int lo, int hi, int bias) const
    {
        return rows_bound<NR>(p_uni(hi - b), b + lane - lo, p_uni(hi - lo), b + lane, p_uni(bias));
    }
    // The first round tr, t < tr < last (else last), in which what is reserved for the next one and cnt requests that hold sp + cnt (tr + 1)
    // there exceed M, or, from round `from` on, leave `first` of it.
    __device__ __forceinline__ int next_event(int t, int last, unsigned sp, int cnt, int M, unsigned first, int from) const
    {
        const unsigned round = (unsigned)(b + lane);  // (of row 0: tr + 1)
        const unsigned wait = (__builtin_elementwise_sub_sat((unsigned)from + 1u, round) + 63u) >> 6;  // rows before `from`
        const int s = t + 2 - b;  // 1 .. 64
        int at;
        const unsigned long long m = rows_event<NR>(p_uni(last - b), (int)(sp + (unsigned)cnt * round), p_uni(64 * cnt), p_uni(M), p_uni(M - (int)first),
                                                    (int)wait, scalar_mask(s < 64 ? ~0ull << s : 0ull), at);
        return m != 0 ? min(b - 1 + at + (int)__builtin_ctzll(m), last) : last;
    }
};

// A ring of H slots in LDS for longer estimates; one launch, 10 bytes an entry as above (with s in the list, 14 bytes, the
// same time for few candidates and fewer of them side by side: 2048 candidates of n = 2000 with decodes up to 8192
// 65 ms, 52 without, as the loop over rounds was then; 512 of them 21.1 and 21.5).  The slots of rounds at or before t are empty and stand for the rounds H later.
struct Ring {
    int lane, mask;
    int *slot;

    static __device__ __forceinline__ int lds_words(int H) { return H; }
    __device__ __forceinline__ Ring(int *lds, int H, int lane_) : lane(lane_), mask(H - 1), slot(lds)
    {
        for (int i = lane; i < H; i += PW) slot[i] = 0;
        p_sync();
    }
    __device__ __forceinline__ int longest() const { return mask + 1; }
    __device__ __forceinline__ void advance(int t, int to)
    {
        const int span = min(to - t, mask + 1);
        if (span == 1) {  // (most rounds; the loop took 2 % of such a run)
            if (lane == 0) slot[(t + 1) & mask] = 0;
        } else {
            for (int i = lane; i < span; i += PW) slot[(t + 1 + i) & mask] = 0;
        }
        p_sync();
    }
    // (two tiles of 64 rounds a turn, their reads in flight together; a slot behind the window is read and left alone)
    __device__ __forceinline__ bool add(int t, int s, int count, int M)
    {
        bool over = false;
        for (int j = lane + 1; j <= count; j += 2 * PW) {
            const int i0 = (t + j) & mask, i1 = (t + j + PW) & mask;
            const int r0 = slot[i0] + s + j, r1 = slot[i1] + s + j + PW;
            const bool in1 = j + PW <= count;
            over |= r0 > M;
            over |= in1 && r1 > M;
            slot[i0] = r0;
            if (in1) slot[i1] = r1;
        }
        return __builtin_amdgcn_ballot_w64(over) != 0;
    }
    __device__ __forceinline__ void take(int t, int s, int ps, int last)
    {
        for (int tq = t + 1 + lane; tq <= last; tq += PW) slot[tq & mask] -= s + (tq - ps);
        p_sync();
    }
    __device__ __forceinline__ int next_round(int t) const { return p_uni(slot[(t + 1) & mask]); }
    __device__ __forceinline__ int bound(int lo, int hi, int bias) const
    {
        int acc = INT_MIN + 1;
        for (int tq = lo + lane; tq <= hi; tq += PW) acc = max(acc, min(tq, slot[tq & mask] + bias + tq));
        return acc;
    }
    __device__ __forceinline__ int next_event(int t, int last, unsigned sp, int cnt, int M, unsigned first, int from) const
    {
        int tr = t + 1 + lane;
        unsigned held = sp + (unsigned)cnt * (unsigned)(tr + 1);
        for (int r0 = t + 1; r0 < last; r0 += PW) {
            const unsigned left = (unsigned)(M - slot[(tr + 1) & mask]);
            const unsigned long long out = __builtin_amdgcn_ballot_w64(held > left);
            const unsigned long long fits = __builtin_amdgcn_ballot_w64(held + first <= left) & __builtin_amdgcn_ballot_w64(tr >= from);
            const unsigned long long m = (out | fits) & __builtin_amdgcn_ballot_w64(tr < last);
            if (m != 0) return r0 + (int)__builtin_ctzll(m);
            tr += PW;
            held += (unsigned)PW * (unsigned)cnt;
        }
        return last;
    }
};

// A running request: position | id << 16 and o | estimate << 16.
struct Entry {
    int pi, oe;
};

// An entry and the round it is due, by the lanes of `mask`.
__device__ __forceinline__ void put_entry(unsigned long long mask, const Entry *e, const unsigned short *d, int pi, int oe, int due)
{
    unsigned long long all;
    const unsigned long long v = (unsigned long long)(unsigned)pi | ((unsigned long long)(unsigned)oe << 32);
    asm volatile("s_and_saveexec_b64 %[all], %[mask]\n"
                 "ds_write_b64 %[e], %[v]\n"
                 "ds_write_b16 %[d], %[due]\n"
                 "s_mov_b64 exec, %[all]\n"
                 : [all] "=&s"(all)
                 : [mask] "s"(mask), [e] "v"(lds_at(e)), [v] "v"(v), [d] "v"(lds_at(d)), [due] "v"(due)
                 : "memory", "scc");
}

template <class Projection>
__device__ __forceinline__ void run_candidate(const PredParams &p, int *lds)
{
    const int lane = threadIdx.x;
    const int cand = blockIdx.x;
    if (p.second && p.retry[cand] == 0) return;
    const int n = p.n, M = p.M, cap = p.cap;
    const int stw = (n + 31) >> 5;
    unsigned *WAIT = (unsigned *)(lds + Projection::lds_words(p.H));  // bit k & 31 of word k >> 5: position k waits (below the frontier)
    Entry *LE = (Entry *)(WAIT + ((stw + 1) & ~1));  // the running list
    unsigned short *LDUE = (unsigned short *)(LE + cap);
    unsigned short *est_stopped = p.est_stopped + (size_t)cand * (size_t)n;

    const int32_t *row = p.orders + (size_t)cand * (size_t)n;
    const int32_t *est0 = p.est0 + (p.E > 1 ? (size_t)cand * (size_t)n : 0);
    int32_t *crow = p.completion_out ? p.completion_out + (size_t)cand * (size_t)n : nullptr;

    for (int i = lane; i < stw; i += PW) WAIT[i] = 0;  // nobody was stopped yet
    int bad = 0;
    for (int k = lane; k < n; k += PW) {
        const int id = min(max(row[k], 0), n - 1);
        const int sv = p.s[id], ov = p.o[id], ev = est0[id];
        if (sv < 1 || ov < 1 || ev < 1 || ov > p.H || ev > p.H || (long long)sv + ov > (long long)M ||
            (long long)sv + ev > (long long)M)
            bad = 1;
    }
    if (__builtin_amdgcn_ballot_w64(bad) != 0) {  // cannot be scheduled: report, do not loop forever
        if (lane == 0) {
            p.tel_out[cand] = -1;
            if (p.evictions_out) p.evictions_out[cand] = 0;
            atomicOr(&p.d_words[KVS_W_STATUS], KVSCHED_DEV_BAD_LENGTH);
        }
        return;
    }
    p_sync();

    Projection proj(lds, p.H, lane);

    // the 64 positions [w_base, w_base + 64) of the order: lane l holds id, s, o of position w_base + l
    int w_base = -PW, w_id = 0, w_s = 1, w_o = 1, w_e = 1;
    int x_base = -PW, x_id = 0, x_s = 1, x_o = 1, x_e = 1;  // ... and the 64 behind them, fetched ahead of need
    int frontier = 0;  // every position from here on waits and was never started
    int c_pos = -1, c_s = 0, c_o = 0, c_id = 0, c_e = 0;  // the request stopped last: position, lengths, id, estimate kept

    int t = 0;
    int head = 0;      // no waiting position lies before it
    int hpos = -1, hs = 0, he = 0, ho = 0, hid = 0;  // the waiting position the admission is stuck at, if any
    int ring_start = 0;  // ... and a round before which the reservations rule out its start
    int nact = 0;      // entries of the list
    int done = 0;
    int ov_cnt = 0;    // requests past their estimate ...
    unsigned ov_sp = 0;  // ... and the sum of s_j - p_j over them, modulo 2^32 (what they hold together is at most M < 2^30)
    int next_due = INT_MAX;  // earliest round at which a running request reaches its estimate or its end
    int evictions = 0;
    int visited = 0;
    long long tel = 0;  // per lane: completion rounds of the entries it has seen end
    bool over_limit = false, overflow = false;

    const int first_last = p.C - p.step_back;  // no other takes the place of the candidates from here on
    while (done < n) {
        if (t >= p.round_limit) { over_limit = true; break; }
        // A candidate that visits many rounds for each request it finishes (a random order: twice as many as the Sorted-F
        // order's neighbours) runs longest, and the call lasts as long as it does: it goes first on its SIMD.  The others go
        // first while they have a quarter of their requests before them, then while they have an eighth: of equal ones a SIMD
        // serves the oldest, and the last third of the time would see fewer than four.  4096 candidates of 2000 mixed requests
        // without any priority / without the two lines / with them: 5.82 / 5.17 / 4.73 ms, of 1000 3.15 / 2.85 / 2.62, of 300
        // chat requests 1.66 / 1.64 / 1.64.
        // Those whose place another candidate takes (all but as many as run at a time) step back in their last eighth only: 6000
        // of 1000 requests 4.92 / 4.76 / 4.53 ms, 8192 / 16384 of 2000 10.9 / 10.3 / 9.4 and 19.6 / 19.0 / 19.0.  Which calls
        // have these lines: may_step_back.
        if ((++visited & 63) == 0) {
            if (2 * visited > 3 * done) __builtin_amdgcn_s_setprio(3);
            else if (p.step_back == 0) __builtin_amdgcn_s_setprio(0);
            else if (cand < first_last ? 8 * done < 7 * n : 4 * done < 3 * n) __builtin_amdgcn_s_setprio(2);
            else if (8 * done < 7 * n) __builtin_amdgcn_s_setprio(1);
            else __builtin_amdgcn_s_setprio(0);
        }
        // nothing waits, nobody outruns an estimate: nothing can happen before the next due round
        if (__builtin_expect(head >= n, 0)) {
            asm volatile("");  // (three branches, of which the first is hardly ever taken, and not one on all three)
            if (ov_cnt == 0 && next_due > t) {
                proj.advance(t, next_due);
                t = next_due;
            }
        }

        // ---- 1. running requests that reach their estimate or their end at this round: the tiles of the list from the last
        //         to the first (an entry that fills a hole has then been looked at), the due entries of a tile side by side.
        if (t >= next_due) {
            unsigned wait_min = 0x7fffffffu;  // per lane: rounds from t + 1 until its entries matter again
            unsigned sp_sum = 0;              // per lane: what its entries change ov_sp by
            // the due entries `due` of the tile at a0; e and wait (rounds from t + 1 until it is due) of the lane's entry
            auto handle = [&](int a0, unsigned long long in, unsigned long long due, const Entry e, int wait) __attribute__((always_inline)) {
                // due now: it started min(estimate, o) rounds ago, o rounds ago if it had outrun its estimate
                const int id = (int)((unsigned)e.pi >> 16);
                const int sv = p.s[__builtin_amdgcn_inverse_ballot_w64(due) ? id : 0];
                const unsigned ol = e.oe & 0xffff, el = (unsigned)e.oe >> 16;
                static_assert(EST_OVERRUN == 0, "an estimate of 0 less 1 is the largest");
                const int ran = (int)min(el - 1u, ol - 1u) + 1;
                const unsigned long long ends = __builtin_amdgcn_ballot_w64(el - 1u >= ol - 1u) & due;
                // goes on past its estimate: from now on it reserves the next round only
                const unsigned long long goes = due & ~ends;
                const bool on = __builtin_amdgcn_inverse_ballot_w64(goes);
                const int more = (int)ol - ran;  // (of one that goes on)
                wait_min = on ? min(wait_min, (unsigned)(more - 1)) : wait_min;
                const unsigned sp = (unsigned)(sv - t + ran);  // (a running request started at most 16384 rounds ago, s < 2^30)
                ov_cnt += __popcll(goes);
                if (ends == 0) {
                    put_entry(goes, LE + a0 + lane, LDUE + a0 + lane, e.pi, (int)ol, t + more);
                    sp_sum += on ? sp : 0u;
                    return;
                }
                const unsigned long long leaves = ends & __builtin_amdgcn_ballot_w64(el == EST_OVERRUN);
                const int k = __popcll(ends);
                tel += __builtin_amdgcn_inverse_ballot_w64(ends) ? t : 0;
                done += k;
                ov_cnt -= __popcll(leaves);
                if (crow) put_global(ends, crow + id, t);
                // the entries that stay move together within the tile, the list's last ones behind them
                const unsigned long long stay = in & ~ends;
                const int to = a0 + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(stay >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)stay, 0));
                put_entry(stay, LE + to, LDUE + to, e.pi, on ? (int)ol : e.oe, on ? t + more : wait + t + 1);
                const int tail = min(k, nact - (a0 + PW));
                if (tail > 0) {
                    const int from = min(nact - tail + lane, nact - 1), hole = a0 + PW - k + lane;
                    const Entry f = LE[from];
                    put_entry(~0ull >> (PW - tail), LE + hole, LDUE + hole, f.pi, f.oe, LDUE[from]);
                }
                nact -= k;
                // over-estimated: rounds t+1 .. p + e were reserved for it
                for (unsigned long long m = ends & __builtin_amdgcn_ballot_w64(el > ol); m != 0; m &= m - 1) {
                    const int l = __builtin_ctzll(m);
                    const int ps_l = t - __builtin_amdgcn_readlane((int)ol, l);
                    proj.take(t, __builtin_amdgcn_readlane(sv, l), ps_l, ps_l + __builtin_amdgcn_readlane((int)el, l));
                    ring_start = 0;  // memory released: the blocked request may fit earlier
                }
                sp_sum += on ? sp : 0u;
                sp_sum -= __builtin_amdgcn_inverse_ballot_w64(leaves) ? sp : 0u;
            };
            // two tiles a turn, all their reads in flight together (a tile takes longer to read than to look at)
            unsigned long long in1 = ~0ull >> (63 - ((nact - 1) & 63));  // the lanes of the tile that hold an entry
            for (int a1 = (nact - 1) & ~(PW - 1); a1 >= 0; a1 -= 2 * PW, in1 = ~0ull) {
                const int i1 = min(a1 + lane, nact - 1), i0 = max(a1 - PW, 0) + lane;
                const unsigned short d1 = LDUE[i1], d0 = LDUE[min(i0, nact - 1)];
                Entry e1 = LE[i1], e0 = LE[min(i0, nact - 1)];
                asm volatile("" : "+v"(e1.pi), "+v"(e1.oe), "+v"(e0.pi), "+v"(e0.oe));  // (read now, needed or not)
                const int w1 = (int)(short)(unsigned short)(d1 - (unsigned short)(t + 1));  // due - t - 1 (at most 16383)
                const int w0 = (int)(short)(unsigned short)(d0 - (unsigned short)(t + 1));
                wait_min = min(wait_min, min((unsigned)w1, (unsigned)w0));  // (-1, due now: the largest)
                const unsigned long long due1 = __builtin_amdgcn_ballot_w64(w1 < 0) & in1;
                const unsigned long long due0 = __builtin_amdgcn_ballot_w64(w0 < 0) & (a1 > 0 ? ~0ull : 0ull);
                if (due1 != 0) handle(a1, in1, due1, e1, w1);
                if (due0 != 0) handle(a1 - PW, ~0ull, due0, e0, w0);
            }
            const int w = p_wave_min((int)wait_min);
            next_due = w == INT_MAX ? INT_MAX : t + 1 + w;
            ov_sp += (unsigned)p_wave_sum((int)sp_sum);
        }

        // ---- 2. admission in the order's sequence
        int room = 0;  // of round t + 1 (while some are past their estimate: without them the reservations alone decide)
        if (ov_cnt > 0) room = M - proj.next_round(t) - (int)(ov_sp + (unsigned)ov_cnt * (unsigned)(t + 1));
        int t_skip = t + 1;  // the next round at which anything can happen
        while (head < n) {
            if (hpos < 0) {  // first waiting position at or after head; kept while it stays blocked
                hpos = head;
                if (head < frontier) {  // among the stopped ones: 32 positions a lane, 2048 a turn
                    hpos = frontier;  // none: the first position never started
                    for (int w0 = head >> 5; w0 < stw; w0 += PW) {
                        const int wi = w0 + lane;
                        unsigned wait = WAIT[min(wi, stw - 1)];
                        wait = wi < stw ? wait : 0u;
                        wait &= wi == (head >> 5) ? ~0u << (head & 31) : ~0u;  // not before head
                        const unsigned long long any = __builtin_amdgcn_ballot_w64(wait != 0);
                        if (any != 0) {
                            const int l = __builtin_ctzll(any);
                            hpos = (w0 + l) * 32 + __builtin_ctz((unsigned)__builtin_amdgcn_readlane((int)wait, l));
                            break;
                        }
                    }
                }
                head = hpos;
                if (hpos >= n) {
                    hpos = -1;
                    break;
                }
                if (hpos == c_pos) {
                    // the request stopped last: what admission needs of it was at hand when it was stopped
                    hs = c_s, ho = c_o, hid = c_id, he = c_e;
                } else if (hpos < frontier) {
                    // an older stopped one: fetched alone (two dependent loads), the window stays at the frontier
                    hid = p_uni(min(max(row[hpos], 0), n - 1));
                    hs = p_uni(p.s[hid]);
                    ho = p_uni(p.o[hid]);
                    he = p_uni((int)est_stopped[hpos]);  // a stopped request kept its estimate
                } else {
                    if ((unsigned)(hpos - w_base) >= (unsigned)PW) {  // the 64 positions around it
                        const int base = hpos & ~(PW - 1);
                        if (base == x_base) {  // fetched ahead
                            w_id = x_id, w_s = x_s, w_o = x_o, w_e = x_e;
                        } else {
                            w_id = min(max(row[min(base + lane, n - 1)], 0), n - 1);
                            w_s = p.s[w_id];
                            w_o = p.o[w_id];
                            w_e = est0[w_id];
                        }
                        w_base = base;
                        x_base = base + PW;  // the loads for the next 64 are issued now and waited for when used
                        x_id = min(max(row[min(x_base + lane, n - 1)], 0), n - 1);
                        x_s = p.s[x_id];
                        x_o = p.o[x_id];
                        x_e = est0[x_id];
                    }
                    hs = __builtin_amdgcn_readlane(w_s, hpos - w_base);
                    ho = __builtin_amdgcn_readlane(w_o, hpos - w_base);
                    hid = __builtin_amdgcn_readlane(w_id, hpos - w_base);
                    he = __builtin_amdgcn_readlane(w_e, hpos - w_base);  // one that never ran starts from est0
                }
                ring_start = 0;
            }
            if (t < ring_start) {  // the reservations rule this round out (nothing was released since that was found)
                if (ov_cnt == 0) t_skip = min(ring_start, next_due);
                break;
            }
            // The requests past their estimate hold round t + 1 as well; that test is one slot, so it
            // goes first (when it fails no request starts this round, whatever the reservations say).
            if (ov_cnt > 0 && hs >= room) break;
            if (nact == cap) { overflow = true; break; }  // (first launch only: the second one's list holds every position)
            // A start at t against the reservations, the request's own entered in the same pass and
            // taken back if some round cannot hold them (rare: the verdict is known for a blocked request).
            if (proj.add(t, hs, he, M)) {
                proj.take(t, hs, t, t + he);
                // Blocked by them.  They change only by admissions (none while this request is blocked)
                // and releases, so they are searched once for the earliest start they allow: round tq
                // rules out the starts t' < tq with t' < R(tq) + s + tq - M; rounds further ahead than the longest
                // estimate hold nothing.  Each turn moves the start to the largest bound seen and looks only at the
                // rounds that entered the window (t', t' + e] since.
                int start = t, lo = t + 1;
                const int bias = hs - M;
                for (;;) {
                    const int hi = min(start + he, t + proj.longest());
                    const int bound = -p_wave_min(-proj.bound(lo, hi, bias));
                    if (bound <= start) break;  // fits at `start`
                    start = bound;
                    lo = hi + 1;
                    if (start >= next_due) break;  // the running set changes first
                }
                ring_start = start;  // (> t)
                if (ov_cnt == 0) t_skip = min(start, next_due);  // nothing happens before
                break;
            }
            ring_start = t;  // a start is allowed now
            room -= hs + 1;
            if (hpos < frontier) {  // a stopped one starts again
                const unsigned *w = WAIT + (hpos >> 5);
                put_b32(1, w, *w & ~(1u << (hpos & 31)));
            }
            const int until = t + min(he, ho);
            put_entry(1, LE + nact, LDUE + nact, hpos | (hid << 16), ho | (he << 16), until);
            frontier = max(frontier, hpos + 1);
            ++nact;
            next_due = min(next_due, until);
            head = hpos + 1;
            hpos = -1;
        }
        if (overflow) break;

        // ---- 3. eviction while round t + 1 is projected above M (only that round can be: the reservations
        //         held a feasible projection and only the overrunners' are new)
        if (ov_cnt > 0) {
            while (room < 0) {
                int best = INT_MAX, best_at = -1;  // (current estimate, id) of the running requests, least first, and its place
                for (int a0 = 0; a0 < nact; a0 += 2 * PW) {  // two tiles a turn, as above
                    int at[2];
                    Entry e[2];
                    unsigned short due[2];
                    for (int h = 0; h < 2; ++h) {
                        at[h] = min(a0 + h * PW + lane, nact - 1);
                        e[h] = LE[at[h]];
                        due[h] = LDUE[at[h]];
                    }
                    for (int h = 0; h < 2; ++h) {
                        const int ev = (int)((unsigned)e[h].oe >> 16);
                        // past its estimate: it has run o - (due - t) rounds and needs one more
                        const int out = (e[h].oe & 0xffff) - (int)(unsigned short)(due[h] - (unsigned short)t) + 1;
                        const int key = ((ev == EST_OVERRUN ? out : ev) << 16) | (int)((unsigned)e[h].pi >> 16);
                        best_at = key < best ? at[h] : best_at;
                        best = min(best, key);
                    }
                }
                const int least = p_wave_min(best);
                if (least == INT_MAX) break;  // cannot happen: an empty system holds nothing
                // ids of a permutation are distinct: one entry holds it
                const unsigned long long holder = __builtin_amdgcn_ballot_w64(best == least);
                const int slot = __builtin_amdgcn_readlane(best_at, __builtin_ctzll(holder));
                if (slot < 0) break;
                const int sv = p_uni(p.s[least & 0xffff]);
                const Entry er = LE[slot];
                const int pi_r = p_uni(er.pi), oe_r = p_uni(er.oe), due16 = p_uni(LDUE[slot]);
                const int vpos = pi_r & 0xffff;
                const int ev = (int)((unsigned)oe_r >> 16), ov = oe_r & 0xffff;
                const int due = t + (int)(unsigned short)((unsigned short)due16 - (unsigned short)t);
                const int ps = due - (ev == EST_OVERRUN ? ov : min(ev, ov));
                room += sv + t + 1 - ps;
                if (ev == EST_OVERRUN) {
                    --ov_cnt;
                    ov_sp -= (unsigned)(sv - ps);
                } else {
                    proj.take(t, sv, ps, ps + ev);
                    ring_start = 0;  // memory released
                }
                c_pos = vpos, c_s = sv, c_o = ov, c_id = (int)((unsigned)pi_r >> 16);
                c_e = ev == EST_OVERRUN ? t - ps + 1 : ev;  // what it is known to need
                est_stopped[vpos] = (unsigned short)c_e;
                const unsigned *w = WAIT + (vpos >> 5);
                put_b32(1, w, *w | 1u << (vpos & 31));  // waits again
                --nact;
                const Entry last = LE[nact];
                put_entry(1, LE + slot, LDUE + slot, last.pi, last.oe, LDUE[nact]);
                if (vpos < head) { head = vpos; hpos = -1; }
                ++evictions;
            }
        }
        // While requests outrun their estimates the projection of round t' + 1 grows by their count
        // every round; until the next due round nothing else changes.  Round t' needs work only if
        // that projection passes M (eviction) or, from the round on that the reservations allow the blocked
        // request to start at, leaves room for its first token (both necessary for its admission):
        // find the first such round.  (They hold at most M < 2^30 now and 65535 * 16384 more at the next due round.)
        if (ov_cnt > 0 && (hpos >= 0 || head >= n) && next_due > t + 1) {
            const unsigned first = hpos >= 0 ? hs + 1 : 1;
            const int from = hpos >= 0 ? ring_start : INT_MAX;  // (nothing waits: only the overflow matters)
            t_skip = proj.next_event(t, next_due, ov_sp, ov_cnt, M, first, from);
        }
        const int to = max(t_skip, t + 1);  // rounds t + 1 .. to - 1 change nothing
        proj.advance(t, to);
        t = to;
    }

    // the lanes' completion rounds, 21 bits at a time (64 lanes of 2^21 - 1 stay below 2^31)
    long long total = 0;
    for (int bit = 42; bit >= 0; bit -= 21) total = (total << 21) + p_wave_sum((int)((unsigned long long)tel >> bit) & 0x1fffff);
    if (lane == 0) {
        if (overflow) {
            p.retry[cand] = 1;  // the second launch runs this candidate with a list of n entries
        } else {
            if (over_limit) {
                p.tel_out[cand] = -1;
                atomicOr(&p.d_words[KVS_W_STATUS], KVSCHED_DEV_ROUND_LIMIT);
            } else {
                p.tel_out[cand] = total;
            }
            if (p.evictions_out) p.evictions_out[cand] = evictions;
        }
    }
}

template <int NR>
__global__ __launch_bounds__(PW) void predicted_reg_kernel(PredParams p)
{
    extern __shared__ int lds[];
    run_candidate<Rows<NR>>(p, lds);
}

__global__ __launch_bounds__(PW) void predicted_ring_kernel(PredParams p)
{
    extern __shared__ int lds[];
    run_candidate<Ring>(p, lds);
}

__global__ void clear_retry_kernel(int32_t *retry, int32_t C)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < C) retry[i] = 0;
}

// Largest estimate; the length scan before it has cleared the word.
__global__ __launch_bounds__(1024) void scan_estimates_kernel(const int32_t *est, size_t count, int32_t *words)
{
    __shared__ int sh[16];
    int mx = 0;
    const size_t stride = (size_t)gridDim.x * 1024;
#pragma unroll 8
    for (size_t i = (size_t)blockIdx.x * 1024 + threadIdx.x; i < count; i += stride) mx = max(mx, est[i]);
    mx = -p_wave_min(-mx);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) mx = max(mx, sh[w]);
        atomicMax(&words[KVS_W_ESTMAX], mx);
    }
}

}  // namespace

int kvs_launch_scan_estimates(const int32_t *est, size_t count, int32_t *d_words, hipStream_t st)
{
    // 16 estimates a thread, at most two workgroups per compute unit: 4096 rows of 2000 2175 -> 12 us (one workgroup before)
    const size_t groups = (count + 16383) / 16384;
    hipLaunchKernelGGL(scan_estimates_kernel, dim3((unsigned)(groups < 512 ? groups : 512)), dim3(1024), 0, st, est, count, d_words);
    return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}

// LDS of one candidate whose running list has `cap` entries of `entry` bytes; ring: slots of a projection in LDS.
static size_t lds_bytes(int32_t n, int32_t ring, int32_t cap, int32_t entry = 10)
{
    return sizeof(int) * ((size_t)ring + (((size_t)n + 31) >> 5)) + (size_t)entry * (size_t)cap;
}

// ... as launched: the entries lie at a multiple of eight bytes.
static size_t lds_taken(int32_t n, int32_t ring, int32_t cap) { return lds_bytes((n + 63) & ~63, ring, cap); }

// For C candidates of `bytes` of LDS each: how many run at a time on 256 compute units if they step back near their ends, or 0.
// Sixteen per unit is the most that counts: with short lists a few more fit, but with the kernel of the time 6000 / 7000 candidates of
// 400 chat requests took 3.92 / 4.30 ms with 4096, 4.00 / 4.35 with the 5120 that run.  The second launch has whole lists; which of its candidates
// run is not known here, and it goes by the case that all do (as if others took the places of all of them: up to 1 % slower).
// Not where the last ones are a quarter or fewer, one for each SIMD: they start when the first end, and equal progress
// ends all the others at once and late.  1000 mixed requests, 4200 / 5000 / 9000 candidates with the lines 4.18 / 4.33 / 6.73 ms,
// without 3.95 / 4.15 / 6.37; 6000 the other way, 4.53 and 4.76.
static int32_t may_step_back(int32_t C, size_t bytes)
{
    const int32_t by_lds = (int32_t)((160 * 1024) / ((bytes + 1023) & ~(size_t)1023));
    const int32_t at_a_time = 256 * (by_lds < 16 ? by_lds : 16), last = C % at_a_time;
    return C > at_a_time && last > 0 && 4 * last <= at_a_time ? 0 : at_a_time;
}

// The longest list of the first launch is the one with which sixteen candidates share a compute unit's 160 KB (LDS is
// handed out in whole KB); worth it when that is at least 128 entries and fewer than all.
static int launch_rows(const void *kernel, PredParams p, hipStream_t st)
{
    const int32_t cap_all = (p.n + 1) & ~1;
    const size_t bytes_all = lds_taken(p.n, 0, cap_all), fixed = lds_taken(p.n, 0, 0), budget = 10 * 1024;
    const int32_t cap_first = fixed < budget ? (int32_t)((budget - fixed) / 10) & ~1 : 0;
    // beyond 64 KB of dynamic LDS the kernel's limit has to be raised first
    if (bytes_all > 64 * 1024 &&
        hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes_all) != hipSuccess)
        return KVSCHED_EHIP;
    auto launch = [&](int32_t cap, int32_t second) {
        p.cap = cap;
        p.second = second;
        p.step_back = may_step_back(p.C, lds_taken(p.n, 0, cap));
        void *args[] = {&p};
        return hipLaunchKernel(kernel, dim3((unsigned)p.C), dim3(PW), args, lds_taken(p.n, 0, cap), st) == hipSuccess;
    };
    if (cap_first >= 128 && cap_first < cap_all && p.retry) {
        hipLaunchKernelGGL(clear_retry_kernel, dim3((unsigned)((p.C + 255) / 256)), dim3(256), 0, st, p.retry, p.C);
        if (!launch(cap_first, 0) || !launch(cap_all, 1)) return KVSCHED_EHIP;
    } else if (!launch(cap_all, 0)) {
        return KVSCHED_EHIP;
    }
    return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}

// One launch with the whole list (a ring is 32 KB or more: a short list lets no further candidate in).  Its candidates have a
// SIMD each and do not step back: 512 of 2000 requests 22.2 -> 21.7 ms without, 1024 of 800 with the largest ring 57.6 -> 56.2.
static int launch_ring(const void *kernel, PredParams p, hipStream_t st)
{
    p.cap = (p.n + 1) & ~1;
    p.second = 0;
    p.step_back = 0;
    const size_t bytes = lds_taken(p.n, p.H, p.cap);
    if (bytes > 64 * 1024 &&
        hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess)
        return KVSCHED_EHIP;
    void *args[] = {&p};
    return hipLaunchKernel(kernel, dim3((unsigned)p.C), dim3(PW), args, bytes, st) == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}

// What the documented limit is compared with: a ring, a bit and 14 bytes per position.  (More than either form takes: the
// sizes that are accepted do not move with them.)
size_t kvs_predicted_lds_bytes(int32_t n, int32_t H) { return lds_bytes(n, H, (n + 1) & ~1, 14); }

int kvs_launch_predicted(const int32_t *orders, int32_t C, int32_t n, const int32_t *s, const int32_t *o,
                         const int32_t *est0, int32_t E, int32_t M, int32_t H, int32_t round_limit, int64_t *tel_out,
                         int32_t *completion_out, int32_t *evictions_out, int32_t *retry, uint16_t *est_stopped,
                         int32_t *d_words, hipStream_t st)
{
    if (kvs_predicted_lds_bytes(n, H) > KVS_PREDICTED_MAX_LDS || n > 65535) return KVSCHED_ERANGE;
    PredParams p;
    p.orders = orders;
    p.C = C;
    p.n = n;
    p.s = s;
    p.o = o;
    p.est0 = est0;
    p.E = E;
    p.M = M;
    p.H = H;
    p.retry = retry;
    p.est_stopped = est_stopped;
    p.round_limit = round_limit;
    p.tel_out = tel_out;
    p.completion_out = completion_out;
    p.evictions_out = evictions_out;
    p.d_words = d_words;
    // The projection in registers while its rows leave room for four wavefronts per SIMD (125 registers in the largest
    // file), hence sixteen candidates per compute unit with every file; else in LDS.  65 rows, 4096 candidates of 2000 mixed
    // requests with decodes up to 4096, eight / twelve / sixteen per unit: 21.0 / 19.3 / 12.3 ms, of 1000: 6.7 / 6.7 / 6.7.
    if (H <= 512) return launch_rows((const void *)predicted_reg_kernel<9>, p, st);
    if (H <= 1024) return launch_rows((const void *)predicted_reg_kernel<17>, p, st);
    if (H <= 2048) return launch_rows((const void *)predicted_reg_kernel<33>, p, st);
    if (H <= 4096) return launch_rows((const void *)predicted_reg_kernel<65>, p, st);
    return launch_ring((const void *)predicted_ring_kernel, p, st);
}
