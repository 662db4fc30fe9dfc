// Internal declarations shared by the translation units of libkvsched.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/kvsched.h"

// Device-side scratch words owned by a context (int32 each).
enum {
    KVS_W_STATUS = 0,  // OR of KVSCHED_DEV_* bits for the call in flight
    KVS_W_OMAX = 1,    // largest decode length found by the length scan
    KVS_W_MINPOS = 2,  // smallest position any move touches (best_neighbor)
    KVS_W_REMAIN = 3,  // exact DP: requests not yet in a batch
    KVS_W_KMAX = 4,    // exact DP: bound on the size of the next batch
    KVS_W_ESTMAX = 7,  // largest initial estimate (kvsched_simulate_predicted)
    KVS_W_MAXPOS = 8,  // largest position any move touches (best_neighbor), -1: none
    KVS_W_STATUS_AT = 9,     // which word holds the status of the last call: KVS_W_STATUS (or 0), or one of the following two,
    KVS_W_STATUS_TURN = 10,  // which calls without a length scan use in turn, each clearing the other (SimParams::scan_here)
    KVS_W_COUNT = 16,  // (what kvsched_device_status and the waits of kvsched_exact_dp read back)
    // Behind them, working words of kernels that split one pass over several workgroups: what they have gathered so
    // far and how many are done.  The workgroup that is done last takes the results and leaves the neutral values.
    KVS_W_SCAN_OMAX = 16,
    KVS_W_SCAN_FLAGS = 17,
    KVS_W_SCAN_MINPOS = 18,  // INT_MAX between calls
    KVS_W_SCAN_MAXPOS = 19,  // -1 between calls
    KVS_W_SCAN_DONE = 20,
    KVS_W_AGREE = 21,  // workgroups of rows_agree_kernel that are done << 16 | rows that agree
    KVS_W_ARGMIN_DONE = 24,
    KVS_W_ARGMIN_PART = 32,  // two int64 per workgroup
    KVS_ARGMIN_GROUPS = 64,
    KVS_W_ALLOCATED = KVS_W_ARGMIN_PART + 4 * KVS_ARGMIN_GROUPS
};

// What the length scan leaves in pinned host memory for a call that waits for it.
// ... and what the exact DP leaves there between batches.
enum {
    KVS_H_OMAX = 0,  // (it and the number are one word of 64 bits; its sign bit: the decode lengths are few, see KVS_H_FEW)
    KVS_H_SEQ = 1,   // number of the launch that has written the others
    KVS_H_MINPOS = 2,
    KVS_H_MAXPOS = 3,
    KVS_H_REMAIN = 4,
    KVS_H_KMAX = 5,
    KVS_H_KMIN = 6,
    KVS_H_BATCHES = 7,
    KVS_H_FEW = 8,  // 1: the last backlog looked over had few decode lengths (few_lengths); nobody waits for it, so it may be an earlier call's
    KVS_H_AGREE = 9,  // of KVS_AGREE_ROWS rows of the call, those that agree with row 0 over their leading positions
    KVS_H_COUNT = 16
};

struct kvsched_ctx {
    int device;
    int32_t o_max_bound;   // 0 = scan o[] on every call
    int32_t *d_words;      // [KVS_W_ALLOCATED] device
    int32_t *h_words;      // [KVS_W_COUNT] pinned host mirror
    int32_t *h_scan;       // [KVS_H_COUNT] pinned host memory the length scan writes to
    int32_t scan_seq;      // number of the last scan that was asked to
    void *d_scratch;       // grows on demand
    size_t scratch_bytes;
    void *static_scratch;  // this device's address of the library's fixed working array (never freed)
    void *d_tables;        // exact DP: tables and records, grows on demand
    size_t tables_bytes;
    int32_t o_file;        // longest decode of the register file the last kvsched_simulate needed (0: unknown, or none): what a
                           // small call starts with before its own is known
    int pad_outputs;       // Phase-1 calls write zeros behind the last batch
    int32_t status_turn;   // which of the two words at KVS_W_STATUS_TURN the last launch without a length scan ahead used
    int timing;            // record events around the timeline kernel
    int timed;             // a pair of events has been recorded
    int32_t resume_rows;   // rows of the last kvsched_simulate call if it resumed rows from snapshots, else 0
    int32_t resume_first;  // ... and how many of them (in sorted order) ran from the start
    size_t rejoin_offset;  // ... and where in the scratch buffer the blocks at which rows stopped early are (0: nowhere)
    size_t neighbor_stop_offset;  // the same for the moves of the last kvsched_best_neighbor / kvsched_horizon_step call
    int32_t neighbor_moves;       // ... and how many moves that call had
    int32_t resume_min_rows;  // kvsched_simulate resumes rows from row 0's snapshots from this many rows on
    int32_t resume_wait_polls;  // ... in one launch, a row waiting at most so many polls for its snapshot; 0: in two launches
    hipEvent_t ev0, ev1;
    // kvsched_horizon_step: the chosen order's saved states and start rounds as far as the last step placed it, with
    // what they were computed from (copies of the order and of the lengths, compared on the device before use)
    void *d_horizon;
    size_t horizon_bytes;
    int32_t hz_kept;             // 0: nothing kept
    int32_t hz_n, hz_o_bound;    // ... for these
    int64_t hz_M;
    int32_t hz_completion;       // what kvsched_horizon_completion has: 0 nothing, 1 start rounds, 2 completion rounds by id
};

// How a candidate's order is presented to the timeline kernel.
struct OrderSource {
    const int32_t *orders;  // [C][n] explicit rows, or NULL
    const int32_t *base;    // [n] base order when moves are applied on the fly
    const int32_t *moves;   // [K][3]; candidate K (one past the last move) is the base itself
};

// Positions up to which the launch scans the lengths itself (SimParams::scan_here).  A launch ahead takes 2 us with a bound on the decodes, 3
// to 4 without, at any size; here every wavefront reads all lengths.  2048 chat orders, scan ahead and here, without a bound 40 13.2
// and 11.8 us, 256 58.7 and 54.8, 512 96.1 and 92.3, 768 137.9 and 137.6, 1024 167.4 and 167.2; with one 11.7 and 9.4, 54.1 and 51.8, 91.4 and 89.4,
// 130.3 and 128.3, 160.2 and 158.3; one order of 256 49.0 and 46.9.  No size measured loses: up to 512 the line leaves 2 to 6 %, beyond it
// nothing to 1 %.
constexpr int KVS_SCANNED_HERE = 256;
constexpr int KVS_CHECKED_ROW = 1024;  // (a bit each has room in the LDS of the smallest file, and a word per lane of 32)

struct SimParams {
    OrderSource src;
    int32_t C;  // number of timelines to run
    int32_t n;
    const int32_t *s;
    const int32_t *o;
    int32_t M;
    int64_t *tel_out;         // [C]
    int32_t *completion_out;  // [C][n] or NULL
    int32_t completion_by_position;  // 1: row entry k = completion of position k (a later pass permutes)
    int32_t *d_words;
    int32_t o_bound;          // lengths above this are reported, not simulated
    // Register kernel, explicit rows of up to KVS_CHECKED_ROW positions placed in full: rows that are no permutations are reported
    int32_t check_rows = 0;
    // Register kernel, explicit rows that are not resumed: the launch leaves everything as it is when *gate > o_bound
    const int32_t *gate = nullptr;
    // Plain launches of the register kernel, and orders placed a lane each: the launch looks the lengths over itself, every wavefront
    // for the longest decode (above scan_limit: everything is left as it is) and the first one for what a scan ahead of it would
    // have left: longest and flags (scan_bound: the caller's bound or 0) in d_words and, with seq, in host.  Nothing has cleared a
    // status word just before it, so there are two in turn: the launch reports in status_word and clears the other.
    int32_t scan_here = 0;
    int32_t scan_limit = 0;
    int32_t scan_bound = 0;
    int32_t status_word = KVS_W_STATUS;  // (with or without a scan: where rows that are no permutations are reported)
    int32_t *host = nullptr;
    int32_t seq = 0;
    int32_t *few_out = nullptr;  // pinned: whether the decode lengths are few, by a launch that looks them over
    int32_t few_known = 0;       // ... and what it held before
    // Rows of more than 64 positions: the event kernel sets todo[c] = 0 for the rows it has placed and 1 for those it has not, and
    // the register kernel's plain launch behind it (which has it set too) places those.
    int32_t *todo = nullptr;
    // Register kernel only: simulate positions [k_begin, k_end) (k_end == 0: up to n), starting
    // from / leaving behind a saved timeline state of KVS_STATE_HEAD_WORDS + 64 NR int32 words:
    // {b64, t, 62 unused, the 64 lanes' partial sums of completion rounds as int64, then the
    // NR x 64 profile registers}.  t = -1 marks a state nothing may resume from.
    int32_t k_begin = 0;
    int32_t k_end = 0;
    const int32_t *state_in = nullptr;
    int32_t *state_out = nullptr;
    // Register kernel, explicit rows only: resuming rows from snapshots of row 0.  When cand_list is
    // set, wave w of the launch runs candidate cand_list[w].  Snapshot j (j >= 1) is the timeline
    // state of row 0 after 64 j positions, at snapshots + (j - 1) * snap_stride.  The wave that runs
    // candidate snap_cand (row 0) writes snapshots 1..snap_blocks (word 1 of a snapshot, the round t, is set to -1 by
    // the host beforehand: a snapshot that is never taken poisons whoever resumes from it); a
    // candidate c with resume_block[c] = b > 0 starts from snapshot b at position 64 b.
    // With snap_flags (the progress word in KVS_PROGRESS_WORDS words, zero at launch) both happen in ONE launch: the wave of
    // candidate snap_cand stores there the number of snapshots it has published so far (or ~that number
    // when it stops early), a candidate with b > 0 waits until the word reaches b, as long as the word
    // keeps moving, then takes the latest snapshot that is there and writes the block it really started
    // from back to resume_block[c].
    const int32_t *cand_list = nullptr;
    int32_t *resume_block = nullptr;
    int32_t *snapshots = nullptr;
    int32_t snap_stride = 0;
    int32_t snap_blocks = 0;
    int32_t *snap_flags = nullptr;
    int32_t snap_wait_polls = 0;  // polls (about 3 us each) a candidate waits for its snapshot at most
    int32_t snap_cand = 0;        // the candidate whose wave writes the snapshots (row 0; the base order among moves)
    // Explicit rows resumed from row 0 may also stop early: a row that differs from row 0 at positions
    // diff_first[c] .. diff_last[c] only, and whose timeline is row 0's again behind them, stops at the
    // 64-position boundary b behind diff_last[c] (b <= rejoin_blocks, the boundaries row 0 saves a state at) and
    // writes b to rejoin_block[c] (INT_MAX: placed everything itself; 0: placed nothing); its tel_out is then
    // relative to row 0's and its completion rounds from position 64 b on are row 0's.  The test needs row 0's
    // start rounds by position, which the wave of row 0 stores in start0.
    // With moves the stretch is the move's own (positions min(i, j) .. max(i, j)) and diff_first / diff_last stay
    // unset; the candidate whose timeline the others rejoin is snap_cand, the base order.
    const int32_t *diff_first = nullptr;
    const int32_t *diff_last = nullptr;
    int32_t *rejoin_block = nullptr;
    int32_t *start0 = nullptr;  // (a launch of one timeline that takes no snapshots stores its start rounds here too)
    int32_t rejoin_blocks = 0;
    // Candidates with skip[c] != INT_MAX are not run at all: they are known to stop at block skip[c] (the
    // encoding of rejoin_block; in practice 0, nothing to place); their tel_out is set to 0.
    const int32_t *skip = nullptr;
    // The wave that writes the snapshots may itself start from one left by an earlier launch, number *snap_start (the
    // progress word then starts there too), and stop at the first 64-position boundary at which the round has passed
    // *t_limit; *placed_out = positions placed.
    const int32_t *snap_start = nullptr;
    const int32_t *t_limit = nullptr;
    int32_t *placed_out = nullptr;
};
constexpr int KVS_STATE_HEAD_WORDS = 192;
// the progress word of the snapshot hand-over: this many copies, this far apart (SimParams::snap_flags)
constexpr int KVS_PROGRESS_COPIES = 64;
constexpr int KVS_PROGRESS_STRIDE_WORDS = 16;
constexpr int KVS_PROGRESS_WORDS = KVS_PROGRESS_COPIES * KVS_PROGRESS_STRIDE_WORDS;
constexpr size_t KVS_STATE_MAX_WORDS = KVS_STATE_HEAD_WORDS + 225 * 64;

// simulate.hip
// (moves: the positions they touch are scanned along; host: pinned words that receive the results and then seq)
int kvs_launch_scan_lengths(const int32_t *s, const int32_t *o, int32_t n, int32_t M, int32_t o_bound,
                            int32_t *d_words, hipStream_t st, const int32_t *moves = nullptr, int32_t K = 0,
                            int32_t *host = nullptr, int32_t seq = 0, int32_t *few_out = nullptr);
int kvs_launch_simulate(const SimParams &p, int32_t ring_slots, hipStream_t st);
// timeline_reg.hip (decode lengths up to KVS_REG_MAX_O)
constexpr int32_t KVS_REG_MAX_O = 14336;  // 224 rows of 64 rounds, and one more row for the window's offset
int kvs_launch_simulate_reg(const SimParams &p, hipStream_t st);

// shortrows.hip: orders of up to 32 requests, a lane each
bool kvs_short_rows(int32_t rows, int32_t n);
int kvs_launch_short_rows(const SimParams &p, int32_t o_limit, hipStream_t st);

// eventrows.hip: a lane per completion round
constexpr int KVS_FEW_LENGTHS = 4;
constexpr int32_t KVS_EVENTS_MAX_N = 400000;  // (a bit per request beside what a chunk takes, within 64 KB of LDS)
int kvs_launch_event_rows(const SimParams &p, hipStream_t st);
int32_t kvs_reg_state_words(int32_t o_bound);  // words of one snapshot for this decode bound
int32_t kvs_reg_file_bound(int32_t o_bound);   // the longest decode its register file takes
int32_t kvs_reg_wavefronts(int32_t o_bound);   // timelines of this decode bound that the chip holds at once

// (o_limit: the launch does nothing when the length scan before it found a longer decode; todo: nor for rows with todo[c] = 0)
int kvs_launch_check_orders(const int32_t *orders, int32_t C, int32_t n, int64_t *tel_out, int32_t *d_words,
                            hipStream_t st, int32_t o_limit = INT32_MAX, const int32_t *todo = nullptr);
int kvs_launch_argmin(const int64_t *tel, int32_t K, int64_t *result_out, int32_t *d_words, hipStream_t st);
// The end of a local-search step: latencies of timelines that stopped early completed from the base order's (rejoin or
// NULL), malformed moves marked, latencies copied to tel_out (or NULL), best move, its latency and the base order's.
int kvs_launch_neighbor_finish(const int64_t *tel, const int32_t *rejoin, const int32_t *moves, int32_t K, int32_t n,
                               int64_t *tel_out, int64_t *result_out, int32_t *d_words, hipStream_t st);

// exactdp.hip
size_t kvs_exact_dp_list_bytes(int32_t n);
size_t kvs_exact_dp_table_bytes(int32_t r, int32_t kmax, int32_t M);
size_t kvs_exact_dp_counted_bytes(int32_t r, int32_t kmax, int32_t M);
// (host, seq: pinned words that receive the batches found, the requests left and the bounds kmin..kmax on the next batch's size, then seq;
// ga, gb: the metric's numerator sums ga s_i + gb o_i -- 0, 1: the F-metric; else G with alpha = ga / gb)
constexpr int32_t KVS_EXACT_SEARCH_N = 256;
// Of up to KVS_EXACT_SEARCH_N requests the batches that need no table are found on the way (search: also behind this one); behind the last one the order is written.
int kvs_launch_exact_dp_prepare(int32_t n, const int32_t *s, const int32_t *o, int32_t M, int32_t ga, int32_t gb,
                                int32_t feas_mode, int32_t tie_rule, int pad, size_t most_bytes, void *lists,
                                int32_t *order_out, int32_t *batch_end_out, double *F_out, int32_t *d_words,
                                int32_t *num_batches_out, int32_t *host, int32_t seq, hipStream_t st);
int kvs_launch_exact_dp_batch(int32_t n, int32_t r, int32_t kmin, int32_t kmax, const int32_t *s, const int32_t *o,
                              int32_t M, int32_t ga, int32_t gb, int32_t feas_mode, int32_t tie_rule, int32_t nb, bool search,
                              void *lists, void *tables, int32_t *order_out, int32_t *batch_end_out, double *F_out,
                              int32_t *num_batches_out, int32_t *d_words, int32_t *host, int32_t seq, hipStream_t st);
int kvs_exact_dp_small_lg(int32_t n, int32_t kmax_bound, int32_t M);
size_t kvs_exact_dp_small_record_bytes(int32_t n, int32_t kmax_bound, int lg);
int kvs_launch_exact_dp_small(int32_t n, const int32_t *s, const int32_t *o, int32_t M, int32_t ga, int32_t gb,
                              int32_t feas_mode,
                              int32_t tie_rule, int lg, void *lists, void *records, int32_t *order_out,
                              int32_t *batch_end_out, double *F_out, int32_t *num_batches_out, int32_t *d_words,
                              hipStream_t st);
// localswap.hip
size_t kvs_local_swap_scratch_bytes(int32_t n);
int kvs_launch_local_swap(int32_t n, const int32_t *s, const int32_t *o, int32_t M, int32_t ga, int32_t gb, int32_t pad,
                          int32_t *order_out,
                          int32_t *batch_end_out, double *F_out, int32_t *swaps_out, int32_t *num_batches_out,
                          void *scratch, int32_t *d_words, hipStream_t st);

// sortedf.hip (up to kvs_sortedF_small_max requests the launch replaces the length scan; pad: zeros behind the last batch)
int32_t kvs_sortedF_small_max(int32_t feas_mode);
size_t kvs_sortedF_scratch_bytes(int32_t n);
int kvs_launch_sortedF(int32_t n, const int32_t *s, const int32_t *o, int32_t M, int32_t ga, int32_t gb,
                       int32_t tie_rule, int32_t feas_mode, int32_t pad,
                       int32_t *order_out, int32_t *batch_end_out, double *F_out, int32_t *num_batches_out,
                       void *scratch, int32_t *d_words, hipStream_t st);

// permute.hip: rows of completion rounds from position order to request-id order, in place; rows
// that are no permutation get tel = -1 and KVSCHED_DEV_BAD_ORDER (what kvs_launch_check_orders does)
constexpr int32_t KVS_PERMUTE_MAX_N = 15872;  // one row and its bitmap must fit in 64 KB of LDS
// resume_block / row0 (or NULL): row c placed only the positions from 64 resume_block[c] on; the
// completion rounds before them are row0[k], row 0's in position order
int kvs_launch_permute_rows(const int32_t *orders, int32_t C, int32_t n, int32_t *completion, int64_t *tel_out,
                            int32_t *d_words, const int32_t *resume_block, const int32_t *row0,
                            const int32_t *rejoin_block, hipStream_t st, int32_t o_limit = INT32_MAX, const int32_t *todo = nullptr);

// horizon.hip.  What the context keeps between horizon steps (one device buffer).
enum {
    KVS_HZ_AVAIL = 0,   // blocks of 64 positions of the order whose saved states are valid
    KVS_HZ_BAD = 1,     // working words of the comparison with the copies
    KVS_HZ_DONE = 2,
    KVS_HZ_FIRST = 3,   // block the chosen order's timeline starts from
    KVS_HZ_LIMIT = 4,   // round behind which it need not go on
    KVS_HZ_PLACED = 5,  // positions it has placed
    KVS_HZ_ZERO = 6,
    KVS_HZ_WORDS = 64
};
struct HorizonKept {
    int32_t *ctrl;      // [KVS_HZ_WORDS]
    int32_t *progress;  // [KVS_PROGRESS_WORDS]
    int32_t *order, *s, *o;   // copies
    int32_t *start;           // start rounds of the order by position (ctrl[KVS_HZ_PLACED] of them)
    int32_t *completion;      // by request id, where the saved states are not used
    int32_t *snapshots;
};
// Before the candidates: is what the context keeps (kept != 0: something) still true of the caller's arrays?  Copies
// brought up to date, KVS_HZ_AVAIL and the progress words set; blocks[m] = what move m shares with the order (entry K: 0).
int kvs_launch_horizon_begin(const HorizonKept &h, int32_t kept, const int32_t *order, const int32_t *s, const int32_t *o,
                             int32_t n, const int32_t *moves, int32_t K, int32_t *blocks, hipStream_t st);
// After them: the best move applied to the order in place, and how far the new order's timeline has to go (everything
// if `full`): it starts from block first_block.
int kvs_launch_horizon_choose(const HorizonKept &h, int32_t *order, int32_t n, const int32_t *moves, const int64_t *result,
                              const int32_t *d_words, int32_t stride, int64_t completed_in, int32_t complete_every,
                              int32_t full, hipStream_t st);
// After the new order's timeline: commit point; completion rounds by request id if wanted.
int kvs_launch_horizon_advance(const HorizonKept &h, const int32_t *order, int32_t n, int32_t blocks, int64_t completed_in,
                               int32_t complete_every, int32_t *completion_out, int64_t *result_out, hipStream_t st);
// The same from completion rounds by request id (result: all six of the step's numbers; nothing is committed of an order that is faulty).
int kvs_launch_horizon_advance_by_id(const int32_t *order, const int32_t *completion, const int32_t *o, int32_t n,
                                     int64_t completed_in, int32_t complete_every, int64_t *result, hipStream_t st);
int kvs_launch_apply_best_move(const int32_t *order, int32_t n, const int32_t *moves, const int64_t *result,
                               int32_t *order_out, hipStream_t st);
int kvs_launch_horizon_completion(const HorizonKept &h, const int32_t *order, const int32_t *o, int32_t n,
                                  int32_t *completion_out, hipStream_t st);

// online.hip
int kvs_launch_online(int32_t B, const int32_t *streams, int32_t N, const int32_t *a, const int32_t *s,
                      const int32_t *o, int32_t M, int32_t backlog_cap, int32_t ring_slots, int32_t *completion_out,
                      int32_t out_len, int64_t *stats_out, int32_t *order_scratch, int32_t *d_words, hipStream_t st);

// predicted.hip
constexpr size_t KVS_PREDICTED_MAX_LDS = 160 * 1024;  // LDS of one workgroup on gfx950
int kvs_launch_scan_estimates(const int32_t *est, size_t count, int32_t *d_words, hipStream_t st);
size_t kvs_predicted_lds_bytes(int32_t n, int32_t H);
int kvs_launch_predicted(const int32_t *orders, int32_t C, int32_t n, const int32_t *s, const int32_t *o,
                         const int32_t *est0, int32_t E, int32_t M, int32_t H, int32_t round_limit, int64_t *tel_out,
                         int32_t *completion_out, int32_t *evictions_out, int32_t *retry /*[C] scratch*/,
                         uint16_t *est_stopped /*[C][n] scratch*/, int32_t *d_words, hipStream_t st);

// prefix.hip
int kvs_launch_check_prefix(const int32_t *orders, int32_t C, int32_t n, int32_t cp, int64_t *tel_out,
                            int32_t *d_words, hipStream_t st);
int kvs_launch_broadcast_prefix(const int32_t *prefix, int32_t cp, int32_t C, int32_t n, int32_t *completion,
                                hipStream_t st);
// rows resumed from snapshots of row 0 (see SimParams)
constexpr int32_t KVS_AGREE_ROWS = 16;
// How many of KVS_AGREE_ROWS rows spread over the call agree with row 0 on their first `first` positions, to host[KVS_H_AGREE], and then the
// number `seq`, beside it what a length scan has left there: the longest decode, and that the lengths are few.  C >= 2.
int kvs_launch_rows_agree(const int32_t *orders, int32_t C, int32_t n, int32_t first, int32_t *d_words, int32_t *host, int32_t longest,
                          int32_t seq, hipStream_t st);
int kvs_launch_shared_blocks(const int32_t *orders, int32_t C, int32_t n, int32_t *blocks, int32_t *diff_first,
                             int32_t *diff_last, hipStream_t st);
// tel[c] += tel[base] for the candidates that stopped early (rejoin[c] != INT_MAX), c != base
int kvs_launch_rejoin_finish(const int32_t *rejoin, int32_t C, int32_t base, int64_t *tel, hipStream_t st);
int kvs_launch_stop_positions(const int32_t *rejoin, int32_t C, int32_t n, int32_t *stop_pos_out, hipStream_t st);
// Moves behind a common prefix of `first` positions whose timeline is the base order's: the move only reorders
// requests that the base order starts in one round (start rounds of positions first .. first + count - 1 in
// window_start, that of position first - 1 in word 1 of the prefix's state).  rejoin[m] = 0 for those (and for
// moves that change nothing), INT_MAX for the others and for the base order itself (entry K).
int kvs_launch_mark_noop_moves(const int32_t *moves, int32_t K, int32_t n, int32_t first, int32_t count,
                               const int32_t *window_start, const int32_t *prefix_state, int32_t *rejoin,
                               hipStream_t st);
// flags / nflags: words to clear on the way (the snapshot flags of the launch that follows), or NULL
int kvs_launch_sort_by_blocks(const int32_t *blocks, int32_t C, int32_t first_row, int32_t *tmp, int32_t *sorted,
                              int32_t *flags, int32_t nflags, hipStream_t st);
int kvs_launch_move_blocks(const int32_t *moves, int32_t K, int32_t n, int32_t *blocks, hipStream_t st);
int kvs_launch_copy_row0_prefix(const int32_t *orders, int32_t C, int32_t n, const int32_t *sorted, int32_t first,
                                const int32_t *blocks, int32_t by_position, int32_t *completion, hipStream_t st);
int kvs_launch_mark_snapshots_unusable(int32_t *snapshots, int32_t count, int32_t stride, hipStream_t st);
int kvs_launch_resume_plan(const int32_t *sorted, int32_t C, int32_t first, const int32_t *blocks,
                           int32_t *resume_pos_out, hipStream_t st);
