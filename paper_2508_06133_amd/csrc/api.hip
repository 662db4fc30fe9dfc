// C ABI of libkvsched: argument checks, context and scratch management, kernel sequencing.
// All arithmetic of the method runs in the kernels of simulate.hip and sortedf.hip.
#include "kvsched_internal.h"

#include <mutex>
#include <new>

// Working memory of kvsched_best_neighbor_static: a fixed array in the library's device image, so
// that the call needs no allocation.  Every GPU the library is used on holds its own copy at its
// own address; host code never uses the array's name as an address but asks the runtime for it,
// once per device (static_scratch_of_current_device), and passes that pointer on.
constexpr size_t KVS_STATIC_SCRATCH_BYTES = (size_t)KVSCHED_STATIC_SCRATCH_MIB << 20;
static __device__ __align__(256) unsigned char scratch[KVS_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_static_mu;
void *g_static_scratch[kMaxDevices];  // device address of `scratch` on each GPU, once resolved

// Address of this library's `scratch` array on the device that is current (call after hipSetDevice).
int static_scratch_of_current_device(int device, void **out)
{
    *out = nullptr;
    if (device < 0 || device >= kMaxDevices) return KVSCHED_ERANGE;
    std::lock_guard<std::mutex> guard(g_static_mu);
    if (!g_static_scratch[device]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return KVSCHED_EHIP;
        g_static_scratch[device] = p;
    }
    *out = g_static_scratch[device];
    return KVSCHED_OK;
}

constexpr int64_t kMaxM = (int64_t)1 << 30;
constexpr int32_t WAVE_POSITIONS = 64;  // positions of an order a wavefront fetches at a time
constexpr size_t kMaxExactTableBytes = (size_t)16 << 30;  // tables + records of the exact DP

int ensure_scratch(kvsched_ctx *ctx, size_t bytes)
{
    ctx->resume_rows = 0;  // whoever asks for scratch overwrites the last resume plan
    ctx->rejoin_offset = 0;
    ctx->neighbor_stop_offset = 0;
    if (bytes <= ctx->scratch_bytes) return KVSCHED_OK;
    if (ctx->d_scratch) {
        // kernels of earlier calls may still be reading the old buffer
        if (hipDeviceSynchronize() != hipSuccess) return KVSCHED_EHIP;
        (void)hipFree(ctx->d_scratch);
        ctx->d_scratch = nullptr;
        ctx->scratch_bytes = 0;
    }
    size_t cap = (bytes + ((size_t)1 << 20)) & ~(((size_t)1 << 20) - 1);
    if (hipMalloc(&ctx->d_scratch, cap) != hipSuccess) return KVSCHED_ENOMEM;
    ctx->scratch_bytes = cap;
    return KVSCHED_OK;
}

int ensure_tables(kvsched_ctx *ctx, size_t bytes)
{
    if (bytes <= ctx->tables_bytes) return KVSCHED_OK;
    if (ctx->d_tables) {
        if (hipDeviceSynchronize() != hipSuccess) return KVSCHED_EHIP;
        (void)hipFree(ctx->d_tables);
        ctx->d_tables = nullptr;
        ctx->tables_bytes = 0;
    }
    size_t cap = (bytes + ((size_t)1 << 20)) & ~(((size_t)1 << 20) - 1);
    if (hipMalloc(&ctx->d_tables, cap) != hipSuccess) return KVSCHED_ENOMEM;
    ctx->tables_bytes = cap;
    return KVSCHED_OK;
}

// Read the context's device words back (one stream synchronisation).
int read_words(kvsched_ctx *ctx, hipStream_t st)
{
    if (hipMemcpyAsync(ctx->h_words, ctx->d_words, sizeof(int32_t) * KVS_W_COUNT, hipMemcpyDeviceToHost, st) !=
        hipSuccess)
        return KVSCHED_EHIP;
    return hipStreamSynchronize(st) == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}

// The timeline kernel, bracketed by the context's events when timing is on.
// events: by the event kernel (o_bound <= KVS_REG_MAX_O), and what it leaves, if it may leave any, by the register kernel.
int run_timelines(kvsched_ctx *ctx, const SimParams &p, int32_t H, hipStream_t st, bool short_rows = false, int32_t o_limit = INT32_MAX,
                  bool events = false)
{
    if (ctx->timing && hipEventRecord(ctx->ev0, st) != hipSuccess) return KVSCHED_EHIP;
    int rc;
    if (events) {
        rc = kvs_launch_event_rows(p, st);
        if (rc == KVSCHED_OK && p.todo) {
            SimParams rest = p;
            rest.scan_here = 0;  // (if the lengths have been looked over: with decodes above the limit no row is left)
            rc = kvs_launch_simulate_reg(rest, st);
        }
    } else {
        // profile in registers when the longest decode fits there, else the LDS ring
        rc = short_rows ? kvs_launch_short_rows(p, o_limit, st)
             : p.o_bound <= KVS_REG_MAX_O ? kvs_launch_simulate_reg(p, st) : kvs_launch_simulate(p, H, st);
    }
    if (rc != KVSCHED_OK) return rc;
    if (p.scan_here) ctx->status_turn = p.status_word - KVS_W_STATUS_TURN;  // (only now: a launch that failed has cleared nothing)
    if (ctx->timing) {
        if (hipEventRecord(ctx->ev1, st) != hipSuccess) return KVSCHED_EHIP;
        ctx->timed = 1;
    }
    return KVSCHED_OK;
}

int32_t ring_slots_for(int32_t o_max)
{
    int32_t h = 64;
    while (h < o_max) h <<= 1;
    return h;
}

int32_t next_seq(kvsched_ctx *ctx) { return ctx->scan_seq = (int32_t)((uint32_t)ctx->scan_seq + 1u); }

// A wait inside a captured stream would have nothing to wait for.
bool capturing(hipStream_t st)
{
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(st, &c) != hipSuccess || c != hipStreamCaptureStatusNone;
}

// Wait until the launch number ctx->scan_seq (length scan, or a batch of the exact DP) has left its results in pinned
// host memory.  (The scan is some microseconds of work, so the host polls; every so often it asks the stream, which
// has the runtime retire the launches behind it here, not in the caller's next copy: 126 launches of an exact DP left 65 us to it.
// Asking also ends the wait if the device has failed.)
int wait_for_scan(kvsched_ctx *ctx, hipStream_t st)
{
    const int32_t seq = ctx->scan_seq;
    for (;;) {
        for (int i = 0; i < 1000; ++i) {
            if (__atomic_load_n(&ctx->h_scan[KVS_H_SEQ], __ATOMIC_ACQUIRE) == seq) return KVSCHED_OK;
            __builtin_ia32_pause();
        }
        const hipError_t e = hipStreamQuery(st);
        if (e == hipErrorNotReady) continue;
        if (e != hipSuccess) return KVSCHED_EHIP;
        // everything enqueued has run
        return __atomic_load_n(&ctx->h_scan[KVS_H_SEQ], __ATOMIC_ACQUIRE) == seq ? KVSCHED_OK : KVSCHED_EHIP;
    }
}

// The longest decode that the length scan found (after wait_for_scan), 1 at least.
int32_t scanned_longest(const kvsched_ctx *ctx)
{
    const int32_t omax = ctx->h_scan[KVS_H_OMAX] & INT32_MAX;
    return omax < 1 ? 1 : omax;
}

int scanned_bound(const kvsched_ctx *ctx, int32_t *o_bound_out)
{
    const int32_t omax = scanned_longest(ctx);
    if (omax > KVSCHED_MAX_O) return KVSCHED_ERANGE;
    *o_bound_out = omax;
    return KVSCHED_OK;
}

// ... and whether the decode lengths are few (a scan_lengths_kernel that was asked to tell).
bool scanned_few(const kvsched_ctx *ctx) { return ctx->h_scan[KVS_H_OMAX] < 0; }

// Where a launch that looks the lengths over leaves whether they are few, which matters beyond kEventsFrom alone (by_events).
constexpr int32_t kEventsFrom = 2048;
int32_t *few_word(const kvsched_ctx *ctx, int32_t o_bound) { return o_bound > kEventsFrom ? ctx->h_scan + KVS_H_FEW : nullptr; }

// Enqueue the length scan; unless the caller supplied a bound, wait for the largest decode
// length.  *o_bound_out is what the timeline kernels size their ring from.
int scan_and_bound(kvsched_ctx *ctx, const int32_t *s, const int32_t *o, int32_t n, int64_t M, hipStream_t st,
                   int32_t *o_bound_out, const int32_t *moves = nullptr, int32_t K = 0,
                   int32_t *min_position_out = nullptr, int32_t *max_position_out = nullptr)
{
    if (max_position_out) *max_position_out = n - 1;
    if (min_position_out) *min_position_out = 0;
    if (ctx->o_max_bound > 0) {
        *o_bound_out = ctx->o_max_bound;
        return kvs_launch_scan_lengths(s, o, n, (int32_t)M, ctx->o_max_bound, ctx->d_words, st, moves, K, nullptr, 0,
                                       moves ? nullptr : few_word(ctx, ctx->o_max_bound));
    }
    if (capturing(st)) return KVSCHED_EHIP;
    // (the first and last position the moves touch come with it)
    int rc = kvs_launch_scan_lengths(s, o, n, (int32_t)M, 0, ctx->d_words, st, moves, K, ctx->h_scan,
                                     next_seq(ctx), moves ? nullptr : few_word(ctx, INT32_MAX));
    if (rc != KVSCHED_OK) return rc;
    rc = wait_for_scan(ctx, st);
    if (rc != KVSCHED_OK) return rc;
    rc = scanned_bound(ctx, o_bound_out);
    if (rc != KVSCHED_OK) return rc;
    if (moves && min_position_out) {
        const int32_t mp = ctx->h_scan[KVS_H_MINPOS];
        *min_position_out = (mp < 0 || mp > n) ? 0 : mp;  // INT_MAX: no move changes the order
        if (mp == INT32_MAX) *min_position_out = n;
        if (max_position_out) {
            const int32_t top = ctx->h_scan[KVS_H_MAXPOS];
            *max_position_out = (top < 0 || top >= n) ? n - 1 : top;
        }
    }
    return KVSCHED_OK;
}

constexpr int32_t kMinSharedPrefix = 64;  // shorter shared prefixes are not worth a launch
// Resuming rows from snapshots of row 0 costs the plan (which rows share what with row 0, sorted:
// some 50 us for 16384 rows) and the wait for row 0's wave; it pays when there is enough work to
// skip.  Measured on random one-swap neighbours of a base order, whole call, no resume / resumed in
// one launch / in two: n = 2000: 2048 rows 0.48 / 0.53 / 0.85 ms, 4096 rows 0.62 / 0.63 / 0.87, 6144 rows 0.78 / 0.75 / 0.96,
// 16384 rows 1.71 / 1.34 / 1.66; n = 1000: 8192 rows 0.54 / 0.54 / 0.64, 16384 rows 0.98 / 0.86 / 0.99; n = 500: 8192 rows 0.32 /
// 0.38 / 0.40, 16384 rows 0.57 / 0.58 / 0.62, 32768 rows 1.06 / 0.98 / 1.06; n = 200: never (16384 rows 0.37 / 0.51 / 0.45).
// Hence, unless the caller sets a row threshold of his own: at least 4096 rows, 6 blocks of 64
// positions and 8 million positions in all.  In two launches (the quarter of the rows that shares least,
// at most half a chip's worth, from the start next to row 0, then the others) the first launch lasts
// a whole timeline whatever it holds: that pays from 16384 rows on.
constexpr int32_t kResumeAutoMinRows = 4096;
constexpr int32_t kResumeAutoMinRowsTwoLaunches = 16384;
constexpr int32_t kResumeAutoMinBlocks = 6;
constexpr int64_t kResumeAutoMinPositions = 8000000;
constexpr int32_t kResumeFirstLaunchMax = 4096;
constexpr int32_t kResumeWaitPollsDefault = 4096;  // about 14 ms
// Streams of kvsched_online run one per wavefront, at most some 1500 to 3000 at once on 256 compute
// units (LDS-limited): below that every stream starts at once and their order is of no consequence.
constexpr int32_t kOnlineOrderMinStreams = 1024;

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }
size_t neighbor_scratch_bytes(int32_t K, int32_t n, int32_t o_bound);

// Are C timelines of n positions to be resumed from the states of the first of them?
static bool resume_pays(const kvsched_ctx *ctx, int32_t C, int32_t n, int32_t o_bound)
{
    if (n <= 2 * WAVE_POSITIONS || o_bound > KVS_REG_MAX_O) return false;
    if (ctx->resume_min_rows != KVSCHED_RESUME_AUTO) return ctx->resume_min_rows > 0 && C >= ctx->resume_min_rows;
    return (n - 1) / WAVE_POSITIONS >= kResumeAutoMinBlocks && (int64_t)C * (int64_t)n >= kResumeAutoMinPositions &&
           C >= (ctx->resume_wait_polls > 0 ? kResumeAutoMinRows : kResumeAutoMinRowsTwoLaunches);
}

__global__ void kvs_copy_i32(int32_t *dst, const int32_t *src, int32_t n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

__global__ void kvs_fill_zero_i32(int32_t *dst, int32_t n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = 0;
}
size_t state_bytes() { return align256(sizeof(int32_t) * KVS_STATE_MAX_WORDS); }

// The horizon step's own buffer (kept between steps).
HorizonKept horizon_kept(kvsched_ctx *ctx, int32_t n)
{
    const size_t row = align256(sizeof(int32_t) * (size_t)n);
    char *b = (char *)ctx->d_horizon;
    HorizonKept h;
    h.ctrl = (int32_t *)b;
    h.progress = h.ctrl + KVS_HZ_WORDS;
    b += align256(sizeof(int32_t) * (KVS_HZ_WORDS + KVS_PROGRESS_WORDS));
    h.order = (int32_t *)b;
    h.s = (int32_t *)(b + row);
    h.o = (int32_t *)(b + 2 * row);
    h.start = (int32_t *)(b + 3 * row);
    h.completion = (int32_t *)(b + 4 * row);
    h.snapshots = (int32_t *)(b + 5 * row);
    return h;
}

// ... for n positions with saved states of `stride` words.
size_t horizon_bytes(int32_t n, int32_t stride)
{
    return align256(sizeof(int32_t) * (KVS_HZ_WORDS + KVS_PROGRESS_WORDS)) + 5 * align256(sizeof(int32_t) * (size_t)n) +
           sizeof(int32_t) * (size_t)((n - 1) / WAVE_POSITIONS) * (size_t)stride + 256;
}

// Growing it forgets what was kept, unless `carry`: what is there moves along (its places depend on its own number of
// positions alone).
int ensure_horizon(kvsched_ctx *ctx, size_t bytes, bool carry = false)
{
    if (bytes <= ctx->horizon_bytes) return KVSCHED_OK;
    if (ctx->d_horizon && hipDeviceSynchronize() != hipSuccess) return KVSCHED_EHIP;
    if (!carry) {
        ctx->hz_kept = ctx->hz_completion = 0;
        (void)hipFree(ctx->d_horizon);
        ctx->d_horizon = nullptr;
        ctx->horizon_bytes = 0;
    }
    void *buf = nullptr;
    if (hipMalloc(&buf, bytes) != hipSuccess) return KVSCHED_ENOMEM;
    if ((ctx->d_horizon ? hipMemcpy(buf, ctx->d_horizon, ctx->horizon_bytes, hipMemcpyDeviceToDevice)
                        : hipMemset(buf, 0, sizeof(int32_t) * KVS_HZ_WORDS)) != hipSuccess ||
        hipDeviceSynchronize() != hipSuccess) {  // (the copies may run behind the call; the steps' streams do not wait for them)
        (void)hipFree(buf);
        return KVSCHED_EHIP;
    }
    (void)hipFree(ctx->d_horizon);
    ctx->d_horizon = buf;
    ctx->horizon_bytes = bytes;
    return KVSCHED_OK;
}

// Run positions [0, cp) of `row0` once and leave the timeline state in `state`;
// completion rounds of those positions (position order) go to prefix_completion if not NULL.
int run_shared_prefix(const int32_t *row0, int32_t cp, int32_t n, const int32_t *s, const int32_t *o, int64_t M,
                      int32_t o_bound, int32_t *d_words, int32_t *state, int32_t *prefix_completion, hipStream_t st)
{
    SimParams q;
    q.src.orders = row0;
    q.src.base = nullptr;
    q.src.moves = nullptr;
    q.C = 1;
    q.n = n;
    q.s = s;
    q.o = o;
    q.M = (int32_t)M;
    q.tel_out = nullptr;
    q.completion_out = prefix_completion;
    q.completion_by_position = 1;
    q.d_words = d_words;
    q.o_bound = o_bound;
    q.k_begin = 0;
    q.k_end = cp;
    q.state_out = state;
    return kvs_launch_simulate_reg(q, st);
}

int check_common(kvsched_ctx *ctx, int32_t n, const int32_t *s, const int32_t *o, int64_t M)
{
    if (!ctx || !s || !o || n < 1 || M < 1) return KVSCHED_EINVAL;
    if (M >= kMaxM) return KVSCHED_ERANGE;
    if (hipSetDevice(ctx->device) != hipSuccess) return KVSCHED_EHIP;
    return KVSCHED_OK;
}

}  // namespace

extern "C" {

int kvsched_create(kvsched_ctx **out, int device_id)
{
    if (!out) return KVSCHED_EINVAL;
    *out = nullptr;
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess) return KVSCHED_EHIP;
    if (device_id < 0 || device_id >= count) return KVSCHED_EINVAL;
    if (hipSetDevice(device_id) != hipSuccess) return KVSCHED_EHIP;
    kvsched_ctx *ctx = new (std::nothrow) kvsched_ctx();
    if (!ctx) return KVSCHED_ENOMEM;
    ctx->device = device_id;
    ctx->o_max_bound = 0;
    ctx->d_words = nullptr;
    ctx->h_words = nullptr;
    ctx->h_scan = nullptr;
    ctx->scan_seq = 0;
    ctx->d_scratch = nullptr;
    ctx->scratch_bytes = 0;
    ctx->static_scratch = nullptr;
    ctx->d_tables = nullptr;
    ctx->tables_bytes = 0;
    ctx->d_horizon = nullptr;
    ctx->horizon_bytes = 0;
    ctx->hz_kept = ctx->hz_n = ctx->hz_o_bound = ctx->hz_completion = 0;
    ctx->hz_M = 0;
    ctx->pad_outputs = 0;
    ctx->o_file = 0;
    ctx->status_turn = 0;
    ctx->timing = 0;
    ctx->timed = 0;
    ctx->resume_rows = 0;
    ctx->rejoin_offset = 0;
    ctx->neighbor_stop_offset = 0;
    ctx->neighbor_moves = 0;
    ctx->resume_first = 0;
    ctx->resume_min_rows = KVSCHED_RESUME_AUTO;
    ctx->resume_wait_polls = kResumeWaitPollsDefault;
    ctx->ev0 = nullptr;
    ctx->ev1 = nullptr;
    int32_t words[KVS_W_ALLOCATED] = {0};
    words[KVS_W_SCAN_MINPOS] = INT32_MAX;
    words[KVS_W_SCAN_MAXPOS] = -1;
    if (hipMalloc((void **)&ctx->d_words, sizeof(words)) != hipSuccess ||
        hipHostMalloc((void **)&ctx->h_words, sizeof(int32_t) * (KVS_W_COUNT + KVS_H_COUNT), hipHostMallocDefault) != hipSuccess ||
        hipMemcpy(ctx->d_words, words, sizeof(words), hipMemcpyHostToDevice) != hipSuccess) {
        kvsched_destroy(ctx);
        return KVSCHED_ENOMEM;
    }
    ctx->h_scan = ctx->h_words + KVS_W_COUNT;
    ctx->h_scan[KVS_H_SEQ] = 0;
    ctx->h_scan[KVS_H_FEW] = 0;
    // devices beyond the table simply cannot use kvsched_best_neighbor_static
    if (device_id < kMaxDevices) {
        const int rc = static_scratch_of_current_device(device_id, &ctx->static_scratch);
        if (rc != KVSCHED_OK) {
            kvsched_destroy(ctx);
            return rc;
        }
    }
    *out = ctx;
    return KVSCHED_OK;
}

void kvsched_destroy(kvsched_ctx *ctx)
{
    if (!ctx) return;
    (void)hipSetDevice(ctx->device);
    (void)hipDeviceSynchronize();
    if (ctx->d_words) (void)hipFree(ctx->d_words);
    if (ctx->h_words) (void)hipHostFree(ctx->h_words);
    if (ctx->d_scratch) (void)hipFree(ctx->d_scratch);
    if (ctx->d_tables) (void)hipFree(ctx->d_tables);
    if (ctx->d_horizon) (void)hipFree(ctx->d_horizon);
    if (ctx->ev0) (void)hipEventDestroy(ctx->ev0);
    if (ctx->ev1) (void)hipEventDestroy(ctx->ev1);
    delete ctx;
}

const char *kvsched_strerror(int status)
{
    switch (status) {
        case KVSCHED_OK: return "ok";
        case KVSCHED_EINVAL: return "invalid argument (null pointer, non-positive size or bad enum)";
        case KVSCHED_ERANGE: return "size outside the supported range";
        case KVSCHED_EHIP: return "HIP runtime call failed";
        case KVSCHED_ENOMEM: return "out of device or host memory";
        default: return "unknown status";
    }
}

int kvsched_reserve(kvsched_ctx *ctx, int32_t rows, int32_t n, int32_t moves)
{
    if (!ctx || rows < 0 || n < 1 || moves < 0) return KVSCHED_EINVAL;
    if (hipSetDevice(ctx->device) != hipSuccess) return KVSCHED_EHIP;
    // the largest of what the calls named in the header ask of the scratch buffer at these sizes
    const size_t nblk = (size_t)((n - 1) / WAVE_POSITIONS);
    const size_t row_bytes = align256(sizeof(int32_t) * (size_t)n);
    size_t need = kvs_sortedF_scratch_bytes(n);
    const size_t swap = kvs_local_swap_scratch_bytes(n);
    if (swap > need) need = swap;
    if (rows > 0) {
        const size_t sim = 6 * align256(sizeof(int32_t) * (size_t)rows) +
                           align256(sizeof(int32_t) * nblk * KVS_STATE_MAX_WORDS) +
                           align256(sizeof(int32_t) * KVS_PROGRESS_WORDS) + 2 * row_bytes;
        const size_t pre = state_bytes() + row_bytes;  // a declared common prefix
        if (sim > need) need = sim;
        if (pre > need) need = pre;
    }
    if (moves > 0) {
        // ... whatever the decode lengths (a bound set now may be lifted later): for the shortest decodes of each register
        // file, the most positions that a call may have with them
        size_t kept = 0;  // by the horizon step, between steps
        for (const int32_t o_bound : {1, 513, 2049, 4097, 8193}) {
            const int64_t most = (kMaxM - 1) / ring_slots_for(o_bound);
            const int32_t m = (int32_t)(most < n ? most : n);
            const size_t hor = neighbor_scratch_bytes(moves, m, o_bound) + align256(sizeof(int32_t) * (size_t)m) + 256;
            if (hor > need) need = hor;
            const size_t states = horizon_bytes(m, kvs_reg_state_words(o_bound));
            if (states > kept) kept = states;
        }
        const int rc = ensure_horizon(ctx, kept, true);
        if (rc != KVSCHED_OK) return rc;
    }
    const int32_t keep = ctx->resume_rows;  // reserving is no call: the last resume plan stays readable unless the buffer moves
    const size_t keep_rejoin = ctx->rejoin_offset, keep_neighbor = ctx->neighbor_stop_offset;
    const bool grows = need > ctx->scratch_bytes;
    const int rc = ensure_scratch(ctx, need);
    if (!grows) ctx->resume_rows = keep, ctx->rejoin_offset = keep_rejoin, ctx->neighbor_stop_offset = keep_neighbor;
    return rc;
}

int kvsched_set_o_max(kvsched_ctx *ctx, int32_t o_max_bound)
{
    if (!ctx || o_max_bound < 0) return KVSCHED_EINVAL;
    if (o_max_bound > KVSCHED_MAX_O) return KVSCHED_ERANGE;
    ctx->o_max_bound = o_max_bound;
    return KVSCHED_OK;
}

int kvsched_set_pad_outputs(kvsched_ctx *ctx, int on)
{
    if (!ctx) return KVSCHED_EINVAL;
    ctx->pad_outputs = on ? 1 : 0;
    return KVSCHED_OK;
}

int kvsched_set_resume_one_launch(kvsched_ctx *ctx, int32_t wait_polls)
{
    if (!ctx || wait_polls < 0) return KVSCHED_EINVAL;
    ctx->resume_wait_polls = wait_polls;
    return KVSCHED_OK;
}

int kvsched_set_resume_min_rows(kvsched_ctx *ctx, int32_t rows)
{
    if (!ctx || (rows < 0 && rows != KVSCHED_RESUME_AUTO)) return KVSCHED_EINVAL;
    ctx->resume_min_rows = rows;
    return KVSCHED_OK;
}

int kvsched_enable_timing(kvsched_ctx *ctx, int on)
{
    if (!ctx) return KVSCHED_EINVAL;
    if (hipSetDevice(ctx->device) != hipSuccess) return KVSCHED_EHIP;
    if (on && !ctx->ev0) {
        if (hipEventCreate(&ctx->ev0) != hipSuccess || hipEventCreate(&ctx->ev1) != hipSuccess) return KVSCHED_EHIP;
    }
    ctx->timing = on ? 1 : 0;
    ctx->timed = 0;
    return KVSCHED_OK;
}

int kvsched_last_timeline_ms(kvsched_ctx *ctx, float *ms_out)
{
    if (!ctx || !ms_out || !ctx->timing || !ctx->timed) return KVSCHED_EINVAL;
    if (hipEventSynchronize(ctx->ev1) != hipSuccess) return KVSCHED_EHIP;
    if (hipEventElapsedTime(ms_out, ctx->ev0, ctx->ev1) != hipSuccess) return KVSCHED_EHIP;
    return KVSCHED_OK;
}

int kvsched_device_status(kvsched_ctx *ctx, void *stream, int32_t *status_out)
{
    if (!ctx || !status_out) return KVSCHED_EINVAL;
    if (hipSetDevice(ctx->device) != hipSuccess) return KVSCHED_EHIP;
    hipStream_t st = (hipStream_t)stream;
    if (hipMemcpyAsync(ctx->h_words, ctx->d_words, sizeof(int32_t) * KVS_W_COUNT, hipMemcpyDeviceToHost, st) !=
        hipSuccess)
        return KVSCHED_EHIP;
    if (hipStreamSynchronize(st) != hipSuccess) return KVSCHED_EHIP;
    const int32_t at = ctx->h_words[KVS_W_STATUS_AT];
    *status_out = ctx->h_words[at == KVS_W_STATUS_TURN || at == KVS_W_STATUS_TURN + 1 ? at : KVS_W_STATUS];
    return KVSCHED_OK;
}

// May a simulate call whose timelines take the register file of o_bound do without a length scan ahead of it?  Its timelines look
// the lengths over themselves where those are few: rows that are placed in full and checked by their own wavefronts.  Not while
// the stream is captured, as a replay would find the status word of the replay before.  (A launch between others that
// depend on each other takes 4.7 us: 40321 rows of 8 11.6 -> 9.3 us a call, 4096 rows of 200 51.8 -> 48.6, with a bound 47.4 -> 46.1; one
// order of 61 requests 14.2 -> 14.4, which waits for the scan's result either way.)
static bool scans_here(const kvsched_ctx *ctx, int32_t C, int32_t n, int32_t o_bound, int32_t common_prefix, hipStream_t st)
{
    return n <= KVS_SCANNED_HERE && o_bound <= KVS_REG_MAX_O && !(common_prefix >= kMinSharedPrefix && C > 1) &&
           !resume_pays(ctx, C, n, o_bound) && !capturing(st);
}

// The status word of the next such call, whose launch clears the other one for the call after it.
static int32_t next_status_word(const kvsched_ctx *ctx) { return KVS_W_STATUS_TURN + (ctx->status_turn ^ 1); }

// Are timelines of n positions, no prefix shared, placed by the event kernel (eventrows.hip)?  Where the decodes are few, which the kernel
// sees for itself, and may be long.  If they are not few, or a row has too many completions ahead, the timeline kernel's launch behind it
// places the rows.  Not while the stream is captured, as the list of rows left lies in memory that later calls may replace
// (orders of up to 64 have none); not where the caller asks for rows to be resumed.
// few: by this call's scan, where the host has waited for it (no bound from the caller, or a wrong guess); -1: not known.  Then `hint` is what
// the context has seen last, of an earlier call, and may be out of date.  Orders that would not be resumed lose a launch by it, 3 us, or the
// other kernel's time; from 8192 positions on, 700 us and more, they take the launch unasked.  Rows that would be resumed could lose all that
// resuming saves (a hint out of date, 16384 rows of 2000 mixed requests: exchanges anywhere 1570 -> 1750, in the last tenth 890 -> 1780), so they
// are resumed while it is not known.
// Known few, such rows are placed here unless they differ from row 0 late (differ_late), as resumed rows cost the less the later they do.  One call
// (us, resumed and here): rows that exchange two positions anywhere, bimodal lengths, 16384 rows of 2000 2414 847, 8192 of 1000 1234 501, 32768 of
// 500 3187 1081, 4096 of 20000 2205 602; four lengths up to 4096, 16384 of 2000 1806 851, 32768 of 500 2115 969; all of 4096, 3463 1639 and
// 4320 1671; random orders, four lengths 3197 2160 and 2868 1877.
// Decodes up to 2048 stay with the timeline kernel's 33 rows.  The lengths decide which is faster there (us, 33 rows and here): of 1 and
// 2048, 1000 orders of 10000 1756 347, 4000 of 2000 831 398, 2 of 200 196 85; of 1, 300, 900 and 2048 1670 816, 714 896, 326 108; of 1, 300 and
// 1024 1360 854, 513 834, 412 104.
constexpr int32_t kEventsUnasked = 8192;
static bool by_events(const kvsched_ctx *ctx, int32_t C, int32_t n, int32_t o_bound, int few, bool hint, hipStream_t st)
{
    if (o_bound <= kEventsFrom || o_bound > KVS_REG_MAX_O || n > KVS_EVENTS_MAX_N) return false;
    const bool resume = resume_pays(ctx, C, n, o_bound);
    if (ctx->resume_min_rows != KVSCHED_RESUME_AUTO && resume) return false;
    if (few == 0 || (few < 0 && (resume || (!hint && n < kEventsUnasked)))) return false;
    return n <= WAVE_POSITIONS || !capturing(st);
}

// Rows that would be resumed and whose lengths are few: do they differ from row 0 so late that resuming them is the quicker way?  Looked up in
// KVS_AGREE_ROWS of them, for which the host waits once more (10 us); yes if half of these agree with row 0 over two thirds.  The event kernel pays for
// all of a row, and the more the fewer requests start together, that is the smaller the budget is against them.  (us, resumed and by events,
// exchanges in the last tenth, and over the last 0.3 alone: lengths 500 to 2500, 16384 rows of 4000, budgets of 12288 2960 7825, 7616 7860; of
// 160000 946 951, 1443 986; of 400000 818 451, 1062 472; 32768 of 1000, 12288 1382 3508, 3856 3540; 40000 770 1203, 2177 1212; 400000 576 434;
// bimodal, 32768 of 400, 12288 1123 1582, 2666 1576; 16000 910 920; 400000 462 130; four lengths from 2100 on, 32768 of 1000, 40000 1068 2015, 3224
// 2008; 400000 589 530, 988 543; of 1, 100 and 14000 the 225 rows always lose, 19606 5476 at the most.)  With a budget of 64 of the longest decodes, or
// decodes beyond 8192, the rows are not looked at.
constexpr int32_t kLateBudget = 64, kLateMaxO = 8192;
static int differ_late(kvsched_ctx *ctx, const int32_t *orders, int32_t C, int32_t n, int64_t M, int32_t o_bound, hipStream_t st, bool *late)
{
    *late = false;
    if (o_bound > kLateMaxO || M >= (int64_t)kLateBudget * o_bound) return KVSCHED_OK;
    const int32_t first = (int32_t)((int64_t)n * 2 / 3);
    int rc = kvs_launch_rows_agree(orders, C, n, first, ctx->d_words, ctx->h_scan, o_bound, next_seq(ctx), st);
    if (rc == KVSCHED_OK) rc = wait_for_scan(ctx, st);
    if (rc != KVSCHED_OK) return rc;
    *late = 2 * ctx->h_scan[KVS_H_AGREE] >= KVS_AGREE_ROWS;
    return KVSCHED_OK;
}

// kvsched_simulate for decodes of at most o_bound.  gated: nothing is written when the length scan enqueued before finds a
// longer one (only where rows are not resumed and no prefix is placed ahead).  scan: no length scan is enqueued before
// (scans_here), the launch does it and, if gated, leaves its result in pinned memory under number ctx->scan_seq.
// status_word: where faulty rows are reported.  few: whether the decode lengths are few, by this call's scan (-1: not known yet), and the rows, if they
// would be resumed, do not differ late (by_events).
static int simulate_within(kvsched_ctx *ctx, const int32_t *orders, int32_t C, int32_t n, const int32_t *s,
                           const int32_t *o, int64_t M, int32_t o_bound, bool gated, bool scan, int32_t status_word, int few, int64_t *tel_out,
                           int32_t *completion_out, int32_t common_prefix, hipStream_t st)
{
    const int32_t o_limit = gated ? o_bound : INT32_MAX;
    int rc;
    const int32_t H = ring_slots_for(o_bound);
    if ((int64_t)n * (int64_t)H >= kMaxM) return KVSCHED_ERANGE;  // rounds are int32
    SimParams p;
    p.src.orders = orders;
    p.src.base = nullptr;
    p.src.moves = nullptr;
    p.C = C;
    p.n = n;
    p.s = s;
    p.o = o;
    p.M = (int32_t)M;
    p.tel_out = tel_out;
    p.completion_out = completion_out;
    // Completion rounds leave the timeline kernel in position order (coalesced stores); a second
    // kernel permutes each row to request-id order through LDS.  Rows too long for LDS are
    // scattered by the timeline kernel itself.
    p.completion_by_position = (completion_out && n <= KVS_PERMUTE_MAX_N) ? 1 : 0;
    p.d_words = ctx->d_words;
    p.o_bound = o_bound;
    p.gate = gated && !scan ? ctx->d_words + KVS_W_OMAX : nullptr;
    p.status_word = status_word;
    if (scan) {
        p.scan_here = 1;
        p.scan_limit = o_limit;
        p.scan_bound = ctx->o_max_bound;
        if (gated) {
            p.host = ctx->h_scan;
            p.seq = ctx->scan_seq;
        }
    }
    // Declared common prefix: run it once (row 0), resume every row from its state.
    int32_t cp = 0;
    int32_t *prefix_comp = nullptr;
    if (common_prefix >= kMinSharedPrefix && C > 1 && o_bound <= KVS_REG_MAX_O &&
        (!completion_out || p.completion_by_position)) {
        cp = common_prefix;
        rc = ensure_scratch(ctx, state_bytes() + align256(sizeof(int32_t) * (size_t)cp));
        if (rc != KVSCHED_OK) return rc;
        int32_t *state = (int32_t *)ctx->d_scratch;
        if (completion_out) prefix_comp = (int32_t *)((char *)ctx->d_scratch + state_bytes());
        rc = run_shared_prefix(orders, cp, n, s, o, M, o_bound, ctx->d_words, state, prefix_comp, st);
        if (rc != KVSCHED_OK) return rc;
        p.k_begin = cp;
        p.state_in = state;
    }
    // No declared prefix: rows that agree with row 0 on their leading 64-position blocks resume
    // from snapshots of row 0's timeline, taken by row 0's own wave.
    ctx->resume_rows = 0;
    ctx->rejoin_offset = 0;
    const int32_t *resumed_blocks = nullptr, *resumed_row0 = nullptr, *rejoined = nullptr;
    p.few_out = few_word(ctx, o_bound);
    p.few_known = p.few_out ? __atomic_load_n(p.few_out, __ATOMIC_RELAXED) : 0;
    const bool events = cp == 0 && by_events(ctx, C, n, o_bound, few, p.few_known != 0, st);
    if (cp == 0 && !events && resume_pays(ctx, C, n, o_bound)) {
        const int32_t nblk = (n - 1) / WAVE_POSITIONS;
        const int32_t stride = kvs_reg_state_words(o_bound);
        const size_t list_bytes = align256(sizeof(int32_t) * (size_t)C);
        const size_t snap_bytes = align256(sizeof(int32_t) * (size_t)nblk * (size_t)stride);
        const size_t flag_bytes = align256(sizeof(int32_t) * KVS_PROGRESS_WORDS);  // the progress word of row 0's wave
        const size_t row_bytes = align256(sizeof(int32_t) * (size_t)n);
        rc = ensure_scratch(ctx, 6 * list_bytes + snap_bytes + flag_bytes + 2 * row_bytes);
        if (rc != KVSCHED_OK) return rc;
        int32_t *blocks = (int32_t *)ctx->d_scratch;
        int32_t *sorted = (int32_t *)((char *)ctx->d_scratch + list_bytes);
        int32_t *tmp = (int32_t *)((char *)ctx->d_scratch + 2 * list_bytes);
        int32_t *snaps = (int32_t *)((char *)ctx->d_scratch + 3 * list_bytes);
        int32_t *flags = (int32_t *)((char *)ctx->d_scratch + 3 * list_bytes + snap_bytes);
        int32_t *row0 = (int32_t *)((char *)ctx->d_scratch + 3 * list_bytes + snap_bytes + flag_bytes);
        // A row may also stop before its end, where its timeline has become row 0's again (see SimParams);
        // not when the timeline kernel itself scatters the completion rounds by request id.
        const bool rejoin = !completion_out || p.completion_by_position;
        char *more = (char *)ctx->d_scratch + 3 * list_bytes + snap_bytes + flag_bytes + row_bytes;
        int32_t *diff_first = (int32_t *)more, *diff_last = (int32_t *)(more + list_bytes);
        int32_t *rejoin_block = (int32_t *)(more + 2 * list_bytes);
        int32_t *start0 = (int32_t *)(more + 3 * list_bytes);
        rc = kvs_launch_shared_blocks(orders, C, n, blocks, rejoin ? diff_first : nullptr, diff_last, st);
        if (rc != KVSCHED_OK) return rc;
        if (rejoin) {
            p.diff_first = diff_first;
            p.diff_last = diff_last;
            p.rejoin_block = rejoin_block;
            p.start0 = start0;
        }
        rc = kvs_launch_sort_by_blocks(blocks, C, 0, tmp, sorted, flags, KVS_PROGRESS_WORDS, st);  // (clears the progress word too)
        if (rc != KVSCHED_OK) return rc;
        int32_t first = 0;
        if (ctx->resume_wait_polls > 0) {
            // All rows in one launch, those that share least with row 0 first: row 0's wave reports each
            // snapshot as it is written, the others wait for theirs (most find it there already).
            if (ctx->timing && hipEventRecord(ctx->ev0, st) != hipSuccess) return KVSCHED_EHIP;
            SimParams a = p;
            a.cand_list = sorted;
            a.resume_block = blocks;
            a.snapshots = snaps;
            a.snap_stride = stride;
            a.snap_blocks = nblk;
            a.snap_flags = flags;
            a.snap_wait_polls = ctx->resume_wait_polls;
            a.rejoin_blocks = rejoin ? nblk : 0;
            rc = kvs_launch_simulate_reg(a, st);
            if (rc != KVSCHED_OK) return rc;
        } else {
            rc = kvs_launch_mark_snapshots_unusable(snaps, nblk, stride, st);
            if (rc != KVSCHED_OK) return rc;
            first = (C + 3) / 4 < kResumeFirstLaunchMax ? (C + 3) / 4 : kResumeFirstLaunchMax;
            if (ctx->timing && hipEventRecord(ctx->ev0, st) != hipSuccess) return KVSCHED_EHIP;
            SimParams a = p;  // rows sorted[0 .. first): from the start; row 0 (sorted[0]) takes the snapshots
            a.C = first;
            a.cand_list = sorted;
            a.snapshots = snaps;
            a.snap_stride = stride;
            a.snap_blocks = nblk;
            rc = kvs_launch_simulate_reg(a, st);
            if (rc != KVSCHED_OK) return rc;
            SimParams b = p;  // rows sorted[first .. C): from their snapshot
            b.C = C - first;
            b.cand_list = sorted + first;
            b.resume_block = blocks;
            b.snapshots = snaps;
            b.snap_stride = stride;
            b.snap_blocks = 0;
            b.rejoin_blocks = rejoin ? nblk : 0;  // (the first launch has left every state and start round of row 0)
            rc = kvs_launch_simulate_reg(b, st);
            if (rc != KVSCHED_OK) return rc;
        }
        if (rejoin) {
            rc = kvs_launch_rejoin_finish(rejoin_block, C, 0, tel_out, st);
            if (rc != KVSCHED_OK) return rc;
            rejoined = rejoin_block;
            ctx->rejoin_offset = (size_t)((char *)rejoin_block - (char *)ctx->d_scratch);
        }
        if (ctx->timing) {
            if (hipEventRecord(ctx->ev1, st) != hipSuccess) return KVSCHED_EHIP;
            ctx->timed = 1;
        }
        if (completion_out && p.completion_by_position) {
            // the permute pass takes the positions a row did not place from this copy of row 0's row
            hipLaunchKernelGGL(kvs_copy_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, row0, completion_out, n);
            if (hipGetLastError() != hipSuccess) return KVSCHED_EHIP;
            resumed_blocks = blocks;
            resumed_row0 = row0;
        } else if (completion_out) {
            rc = kvs_launch_copy_row0_prefix(orders, C, n, sorted, first, blocks, p.completion_by_position,
                                             completion_out, st);
            if (rc != KVSCHED_OK) return rc;
        }
        ctx->resume_rows = C;
        ctx->resume_first = first;
    } else {
        const bool short_rows = cp == 0 && kvs_short_rows(C, n);
        if (events && n > WAVE_POSITIONS) {
            rc = ensure_scratch(ctx, sizeof(int32_t) * (size_t)C);
            if (rc != KVSCHED_OK) return rc;
            p.todo = (int32_t *)ctx->d_scratch;
        }
        if (cp == 0 && n <= KVS_CHECKED_ROW && o_bound <= KVS_REG_MAX_O) {
            p.check_rows = 1;
            p.completion_by_position = 0;
        }
        rc = run_timelines(ctx, p, H, st, short_rows, o_limit, events && !short_rows);
        if (rc != KVSCHED_OK || short_rows || p.check_rows) return rc;  // (these check the orders and write by request id)
    }
    if (prefix_comp) {
        rc = kvs_launch_broadcast_prefix(prefix_comp, cp, C, n, completion_out, st);
        if (rc != KVSCHED_OK) return rc;
    }
    if (p.completion_by_position) {  // this pass over the rows checks them as well
        rc = kvs_launch_permute_rows(orders, C, n, completion_out, tel_out, ctx->d_words, resumed_blocks, resumed_row0,
                                     resumed_row0 ? rejoined : nullptr, st, o_limit, p.todo);
    } else {
        rc = kvs_launch_check_orders(orders, C, n, tel_out, ctx->d_words, st, o_limit, p.todo);
    }
    if (rc != KVSCHED_OK || cp == 0) return rc;
    return kvs_launch_check_prefix(orders, C, n, cp, tel_out, ctx->d_words, st);
}

// Without a bound from the caller the largest decode length has to be found before the kernel can be chosen.  A small
// call does not let the GPU wait for the host meanwhile: its launches follow the scan at once, with the register file that
// the last call needed, and do nothing if the scan has found a longer decode; the host, which reads the scan's result
// while they run, then launches with the right file.  So a caller whose backlogs alternate pays for launches that end
// at once, not for timelines.  Nor does it get a file that lets fewer of its timelines run side by side than its own:
// the file has to be one of those with eight wavefronts per SIMD, or every timeline of the call in flight.
// (Up to a million positions, some 100 us of timelines, against 10 us of waiting in each call.  One order of 61 requests:
// 29 us with the wait, 18.5 without, 22 when two backlogs alternate; 4096 orders of 200, decodes up to 400 and up to 14000 in
// turn: 114 with the wait, 102 now, 114 when the launches of a wrong guess ran to their end; up to 2000 and up to 14000: 118,
// 105, 132.  4096 orders exceed what the 225-row file holds at once, so those of 14000 alone wait: 130.)
constexpr int64_t kGuessMaxPositions = 1 << 20;

int kvsched_simulate(kvsched_ctx *ctx, const int32_t *orders, int32_t C, int32_t n, const int32_t *s,
                     const int32_t *o, int64_t M, int64_t *tel_out, int32_t *completion_out, int32_t common_prefix,
                     void *stream)
{
    int rc = check_common(ctx, n, s, o, M);
    if (rc != KVSCHED_OK) return rc;
    if (!orders || !tel_out || C < 1 || common_prefix < 0 || common_prefix > n) return KVSCHED_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    int32_t guess = 0, status_word = KVS_W_STATUS;
    bool scan = false;
    if (ctx->o_max_bound == 0 && ctx->o_file > 0 && (int64_t)C * n <= kGuessMaxPositions &&
        common_prefix < kMinSharedPrefix && !resume_pays(ctx, C, n, ctx->o_file) &&
        (C <= kvs_reg_wavefronts(ctx->o_file) || kvs_reg_wavefronts(ctx->o_file) == kvs_reg_wavefronts(1)) &&
        (int64_t)n * ring_slots_for(ctx->o_file) < kMaxM && !capturing(st))
        guess = ctx->o_file;
    if (guess > 0) {
        next_seq(ctx);
        scan = scans_here(ctx, C, n, guess, common_prefix, st);
        if (scan) status_word = next_status_word(ctx);
        else rc = kvs_launch_scan_lengths(s, o, n, (int32_t)M, 0, ctx->d_words, st, nullptr, 0, ctx->h_scan, ctx->scan_seq,
                                          few_word(ctx, INT32_MAX));
        if (rc == KVSCHED_OK)
            rc = simulate_within(ctx, orders, C, n, s, o, M, guess, true, scan, status_word, -1, tel_out, completion_out, 0, st);
        if (rc == KVSCHED_OK) rc = wait_for_scan(ctx, st);
        if (rc != KVSCHED_OK) return rc;
    } else if (ctx->o_max_bound > 0 && scans_here(ctx, C, n, ctx->o_max_bound, common_prefix, st)) {
        ctx->o_file = kvs_reg_file_bound(ctx->o_max_bound);
        return simulate_within(ctx, orders, C, n, s, o, M, ctx->o_max_bound, false, true, next_status_word(ctx), -1, tel_out,
                               completion_out, common_prefix, st);
    }
    int32_t o_bound = 0;
    rc = guess > 0 ? scanned_bound(ctx, &o_bound) : scan_and_bound(ctx, s, o, n, M, st, &o_bound);
    if (rc != KVSCHED_OK) return rc;
    ctx->o_file = kvs_reg_file_bound(o_bound);
    if (guess >= o_bound) return KVSCHED_OK;
    int few = scan || ctx->o_max_bound > 0 ? -1 : scanned_few(ctx);
    if (few > 0 && common_prefix < kMinSharedPrefix && resume_pays(ctx, C, n, o_bound) && by_events(ctx, C, n, o_bound, few, false, st)) {
        bool late;
        rc = differ_late(ctx, orders, C, n, M, o_bound, st, &late);
        if (rc != KVSCHED_OK) return rc;
        if (late) few = 0;
    }
    if (scan && o_bound > KVS_REG_MAX_O) {  // (whose kernels report in the scan's word)
        status_word = KVS_W_STATUS;
        rc = kvs_launch_scan_lengths(s, o, n, (int32_t)M, 0, ctx->d_words, st);
        if (rc != KVSCHED_OK) return rc;
    }
    return simulate_within(ctx, orders, C, n, s, o, M, o_bound, false, false, status_word, few, tel_out, completion_out, common_prefix,
                           st);
}

// The three Phase-1 solvers; (ga, gb) = (0, 1) is the F-metric.
static int run_sortedF(kvsched_ctx *ctx, int32_t n, const int32_t *s, const int32_t *o, int64_t M, int32_t ga,
                       int32_t gb, int32_t tie_rule, int32_t feas_mode, int32_t *order_out, int32_t *batch_end_out,
                       double *F_out, int32_t *num_batches_out, void *stream)
{
    int rc = check_common(ctx, n, s, o, M);
    if (rc != KVSCHED_OK) return rc;
    if (!order_out || !batch_end_out || !F_out || !num_batches_out) return KVSCHED_EINVAL;
    if (tie_rule != KVSCHED_TIE_LARGER && tie_rule != KVSCHED_TIE_SMALLER) return KVSCHED_EINVAL;
    if (feas_mode != KVSCHED_FEAS_SUM_OF_PEAKS && feas_mode != KVSCHED_FEAS_PROFILE) return KVSCHED_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    rc = ensure_scratch(ctx, kvs_sortedF_scratch_bytes(n));
    if (rc != KVSCHED_OK) return rc;
    return kvs_launch_sortedF(n, s, o, (int32_t)M, ga, gb, tie_rule, feas_mode, ctx->pad_outputs, order_out, batch_end_out, F_out,
                              num_batches_out, ctx->d_scratch, ctx->d_words, st);
}

int kvsched_sortedF(kvsched_ctx *ctx, int32_t n, const int32_t *s, const int32_t *o, int64_t M, int32_t tie_rule,
                    int32_t feas_mode, int32_t *order_out, int32_t *batch_end_out, double *F_out,
                    int32_t *num_batches_out, void *stream)
{
    return run_sortedF(ctx, n, s, o, M, 0, 1, tie_rule, feas_mode, order_out, batch_end_out, F_out, num_batches_out,
                       stream);
}

static int run_local_swap(kvsched_ctx *ctx, int32_t n, const int32_t *s, const int32_t *o, int64_t M, int32_t ga,
                          int32_t gb, int32_t *order_out, int32_t *batch_end_out, double *F_out, int32_t *swaps_out,
                          int32_t *num_batches_out, void *stream)
{
    int rc = check_common(ctx, n, s, o, M);
    if (rc != KVSCHED_OK) return rc;
    if (!order_out || !batch_end_out || !F_out || !num_batches_out) return KVSCHED_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    rc = ensure_scratch(ctx, kvs_local_swap_scratch_bytes(n));
    if (rc != KVSCHED_OK) return rc;
    return kvs_launch_local_swap(n, s, o, (int32_t)M, ga, gb, ctx->pad_outputs, order_out, batch_end_out, F_out, swaps_out,
                                 num_batches_out, ctx->d_scratch, ctx->d_words, st);
}

int kvsched_local_swap(kvsched_ctx *ctx, int32_t n, const int32_t *s, const int32_t *o, int64_t M,
                       int32_t *order_out, int32_t *batch_end_out, double *F_out, int32_t *swaps_out,
                       int32_t *num_batches_out, void *stream)
{
    return run_local_swap(ctx, n, s, o, M, 0, 1, order_out, batch_end_out, F_out, swaps_out, num_batches_out, stream);
}

__global__ void kvs_zero_batches(int32_t *batch_end, double *F, int32_t n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) batch_end[i] = 0, F[i] = 0.0;
}

static int run_exact_dp(kvsched_ctx *ctx, int32_t n, const int32_t *s, const int32_t *o, int64_t M, int32_t ga,
                        int32_t gb, int32_t feas_mode, int32_t tie_rule, int32_t *order_out, int32_t *batch_end_out,
                        double *F_out, int32_t *num_batches_out, void *stream)
{
    int rc = check_common(ctx, n, s, o, M);
    if (rc != KVSCHED_OK) return rc;
    if (!order_out || !batch_end_out || !F_out || !num_batches_out) return KVSCHED_EINVAL;
    if (tie_rule != KVSCHED_TIE_LARGER && tie_rule != KVSCHED_TIE_SMALLER) return KVSCHED_EINVAL;
    if (feas_mode != KVSCHED_FEAS_SUM_OF_PEAKS && feas_mode != KVSCHED_FEAS_PROFILE) return KVSCHED_EINVAL;
    if (n > KVSCHED_EXACT_MAX_N) return KVSCHED_ERANGE;
    hipStream_t st = (hipStream_t)stream;
    rc = ensure_scratch(ctx, kvs_exact_dp_list_bytes(n));
    if (rc != KVSCHED_OK) return rc;
    // Small problems run in one workgroup with both tables in LDS; a batch holds at most M / 2
    // requests (each costs at least 2 of the budget), which may already show that they fit.
    const int32_t k_host = (int32_t)((M / 2 < n) ? M / 2 : n);
    if (const int lg = kvs_exact_dp_small_lg(n, k_host, (int32_t)M)) {
        rc = ensure_tables(ctx, kvs_exact_dp_small_record_bytes(n, k_host, lg));
        if (rc != KVSCHED_OK) return rc;
        if (ctx->pad_outputs) {
            hipLaunchKernelGGL(kvs_zero_batches, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, batch_end_out, F_out, n);
            if (hipGetLastError() != hipSuccess) return KVSCHED_EHIP;
        }
        return kvs_launch_exact_dp_small(n, s, o, (int32_t)M, ga, gb, feas_mode, tie_rule, lg, ctx->d_scratch, ctx->d_tables,
                                         order_out, batch_end_out, F_out, num_batches_out, ctx->d_words, st);
    }
    if (capturing(st)) return KVSCHED_EHIP;
    rc = kvs_launch_exact_dp_prepare(n, s, o, (int32_t)M, ga, gb, feas_mode, tie_rule, ctx->pad_outputs, kMaxExactTableBytes, ctx->d_scratch,
                                     order_out, batch_end_out, F_out, ctx->d_words, num_batches_out, ctx->h_scan, next_seq(ctx), st);
    if (rc != KVSCHED_OK) return rc;
    rc = wait_for_scan(ctx, st);
    if (rc != KVSCHED_OK) return rc;
    int32_t r = ctx->h_scan[KVS_H_REMAIN], kmax = ctx->h_scan[KVS_H_KMAX], kmin = ctx->h_scan[KVS_H_KMIN], nb = ctx->h_scan[KVS_H_BATCHES];
    if (r == 0) return KVSCHED_OK;  // all batches are found (or malformed lengths: reported in the device status, no batches)
    if (r < 0 || r > n || kmax < 1 || kmax > r || kmin < 1 || kmin > kmax || nb < 0 || nb > n - r) return KVSCHED_EHIP;
    if (r == n) {  // nothing found yet
        if (const int lg = kvs_exact_dp_small_lg(n, kmax, (int32_t)M)) {  // fits after all, with the true bound
            rc = ensure_tables(ctx, kvs_exact_dp_small_record_bytes(n, kmax, lg));
            if (rc != KVSCHED_OK) return rc;
            return kvs_launch_exact_dp_small(n, s, o, (int32_t)M, ga, gb, feas_mode, tie_rule, lg, ctx->d_scratch, ctx->d_tables,
                                             order_out, batch_end_out, F_out, num_batches_out, ctx->d_words, st);
        }
        if (kvs_exact_dp_counted_bytes(r, kmax, (int32_t)M) > kMaxExactTableBytes) return KVSCHED_ERANGE;
    }
    rc = ensure_tables(ctx, kvs_exact_dp_table_bytes(r, kmax, (int32_t)M));
    if (rc != KVSCHED_OK) return rc;
    // Requests of a few lengths leave most of a backlog undecided: once that has happened twice more than the search has found
    // a batch it is not tried again (150 requests of lengths up to 8: tried for every batch it cost 45 us of 970).
    int32_t tables = 0, failed = r <= KVS_EXACT_SEARCH_N ? 1 : 0;
    while (r > 0) {  // r falls by at least one per batch
        const bool search = failed <= 1 + nb - tables++;
        rc = kvs_launch_exact_dp_batch(n, r, kmin, kmax, s, o, (int32_t)M, ga, gb, feas_mode, tie_rule, nb, search, ctx->d_scratch,
                                       ctx->d_tables, order_out, batch_end_out, F_out, num_batches_out, ctx->d_words, ctx->h_scan,
                                       next_seq(ctx), st);
        if (rc != KVSCHED_OK) return rc;
        rc = wait_for_scan(ctx, st);
        if (rc != KVSCHED_OK) return rc;
        const int32_t r_next = ctx->h_scan[KVS_H_REMAIN], k_next = ctx->h_scan[KVS_H_KMAX], min_next = ctx->h_scan[KVS_H_KMIN];
        if (r_next < 0 || r_next >= r || k_next > kmax || (r_next > 0 && (k_next < 1 || min_next < 1 || min_next > k_next)))
            return KVSCHED_EHIP;
        r = r_next;
        kmax = k_next;
        kmin = min_next;
        nb = ctx->h_scan[KVS_H_BATCHES];
        if (search && r > 0 && r <= KVS_EXACT_SEARCH_N) ++failed;
    }
    return KVSCHED_OK;
}

int kvsched_exact_dp(kvsched_ctx *ctx, int32_t n, const int32_t *s, const int32_t *o, int64_t M, int32_t feas_mode,
                     int32_t tie_rule, int32_t *order_out, int32_t *batch_end_out, double *F_out,
                     int32_t *num_batches_out, void *stream)
{
    return run_exact_dp(ctx, n, s, o, M, 0, 1, feas_mode, tie_rule, order_out, batch_end_out, F_out, num_batches_out,
                        stream);
}

int kvsched_phase1_G(kvsched_ctx *ctx, int32_t solver, int32_t n, const int32_t *s, const int32_t *o, int64_t M,
                     int32_t alpha_num, int32_t alpha_den, int32_t tie_rule, int32_t feas_mode, int32_t *order_out,
                     int32_t *batch_end_out, double *G_out, int32_t *swaps_out, int32_t *num_batches_out, void *stream)
{
    if (alpha_num < 0 || alpha_den < 1 || M < 1) return KVSCHED_EINVAL;
    // Effective lengths alpha_num s_i + alpha_den o_i <= big (s_i + o_i) <= big M.  The sorted-prefix
    // kernel sums them in int64 (and needs alpha_den k^2 exact in a double); Local Swap Search keeps one
    // per request in an int32; the exact DP keeps sums over a batch in int32 (at most M under the sum of
    // peaks, 2 M under the profile constraint).
    const int64_t big = alpha_num > alpha_den ? alpha_num : alpha_den;
    const int64_t lim = (int64_t)1 << 31;
    if (big > 65535) return KVSCHED_ERANGE;
    if (solver == KVSCHED_SOLVER_LOCAL_SWAP && big * M >= lim) return KVSCHED_ERANGE;
    if (solver == KVSCHED_SOLVER_EXACT_DP && big * 2 * M >= lim) return KVSCHED_ERANGE;
    switch (solver) {
        case KVSCHED_SOLVER_SORTED_PREFIX:
            return run_sortedF(ctx, n, s, o, M, alpha_num, alpha_den, tie_rule, feas_mode, order_out, batch_end_out,
                               G_out, num_batches_out, stream);
        case KVSCHED_SOLVER_LOCAL_SWAP:
            if (feas_mode != KVSCHED_FEAS_SUM_OF_PEAKS) return KVSCHED_EINVAL;
            return run_local_swap(ctx, n, s, o, M, alpha_num, alpha_den, order_out, batch_end_out, G_out, swaps_out,
                                  num_batches_out, stream);
        case KVSCHED_SOLVER_EXACT_DP:
            return run_exact_dp(ctx, n, s, o, M, alpha_num, alpha_den, feas_mode, tie_rule, order_out, batch_end_out,
                                G_out, num_batches_out, stream);
        default: return KVSCHED_EINVAL;
    }
}

// Scratch of kvsched_best_neighbor: K + 1 latencies, the state of a shared prefix, where each move's timeline
// stopped because it had become the base order's again (K + 1 entries) with the base order's start rounds (n),
// and the plan for resuming each move's timeline from the base order's (three lists of K + 1 entries, a flag
// and a saved state of the largest kind per 64 positions).
namespace {
// o_bound: the caller's bound on the decode lengths if there is one (it fixes the size of a saved state), else 0: the
// longest that n positions allow (rounds are int32).
size_t neighbor_scratch_bytes(int32_t K, int32_t n, int32_t o_bound)
{
    const size_t nblk = (size_t)((n - 1) / WAVE_POSITIONS);
    if (o_bound == 0) {
        o_bound = KVS_REG_MAX_O;
        while (o_bound > 512 && (int64_t)n * ring_slots_for(o_bound) >= kMaxM) o_bound = ring_slots_for(o_bound) / 2;
    }
    const size_t words = o_bound > KVS_REG_MAX_O ? 0  // beyond the register kernel nothing is resumed
                                                 : (size_t)kvs_reg_state_words(o_bound);
    return align256(sizeof(int64_t) * ((size_t)K + 1)) + state_bytes() +
           4 * align256(sizeof(int32_t) * ((size_t)K + 1)) + align256(sizeof(int32_t) * (size_t)n) +
           align256(sizeof(int32_t) * KVS_PROGRESS_WORDS) + align256(sizeof(int32_t) * nblk * words);
}
}  // namespace

// kvsched_best_neighbor on working memory `work` of at least neighbor_scratch_bytes(K, n) bytes.
// o_bound_known > 0: the caller's bound on the decode lengths; nothing is read back from the device
// (so the lowest position the moves touch is not known either and no common prefix is placed ahead:
// moves far into the order start from the base order's saved states instead).
static int best_neighbor_on(kvsched_ctx *ctx, void *work, int32_t o_bound_known, const int32_t *base_order, int32_t n,
                            const int32_t *moves, int32_t K, const int32_t *s, const int32_t *o, int64_t M,
                            int64_t *tel_out, int64_t *result_out, hipStream_t st)
{
    // work: [K+1] latencies (neighbours, then the base order) | state of the shared prefix | resume plan
    const size_t tel_bytes = align256(sizeof(int64_t) * ((size_t)K + 1));
    int64_t *tel = (int64_t *)work;
    int32_t *state = (int32_t *)((char *)work + tel_bytes);
    const size_t list_bytes_all = align256(sizeof(int32_t) * ((size_t)K + 1));
    int32_t *rejoin_block = (int32_t *)((char *)work + tel_bytes + state_bytes());
    int32_t *start0 = (int32_t *)((char *)work + tel_bytes + state_bytes() + list_bytes_all);
    const size_t plan_offset = tel_bytes + state_bytes() + list_bytes_all + align256(sizeof(int32_t) * (size_t)n);
    int32_t o_bound = 0, min_pos = 0, max_pos = n - 1;
    bool stops_early = false;
    ctx->neighbor_stop_offset = 0;
    int rc;
    if (o_bound_known > 0) {
        rc = kvs_launch_scan_lengths(s, o, n, (int32_t)M, o_bound_known, ctx->d_words, st);
        o_bound = o_bound_known;
    } else {
        rc = scan_and_bound(ctx, s, o, n, M, st, &o_bound, moves, K, &min_pos, &max_pos);
    }
    if (rc != KVSCHED_OK) return rc;
    const int32_t H = ring_slots_for(o_bound);
    if ((int64_t)n * (int64_t)H >= kMaxM) return KVSCHED_ERANGE;
    SimParams p;
    p.src.orders = nullptr;
    p.src.base = base_order;
    p.src.moves = moves;
    p.C = K + 1;
    p.n = n;
    p.s = s;
    p.o = o;
    p.M = (int32_t)M;
    p.tel_out = tel;
    p.completion_out = nullptr;
    p.completion_by_position = 0;
    p.d_words = ctx->d_words;
    p.o_bound = o_bound;
    // No move touches a position before min_pos: that prefix of the base order is common to
    // every neighbour, so it is placed once and all timelines resume from its state.
    if (min_pos >= kMinSharedPrefix && o_bound <= KVS_REG_MAX_O) {
        rc = run_shared_prefix(base_order, min_pos, n, s, o, M, o_bound, ctx->d_words, state, nullptr, st);
        if (rc != KVSCHED_OK) return rc;
        p.k_begin = min_pos;
        p.state_in = state;
        // A move that only reorders requests the base order starts in one and the same round changes no
        // completion round (see the timeline kernel): the base order is placed once more, alone, through the last
        // position any move touches, and the moves found to be of that kind are not run at all.
        if (min_pos < n && max_pos >= min_pos) {
            SimParams q = p;
            q.src.orders = base_order;
            q.src.base = nullptr;
            q.src.moves = nullptr;
            q.C = 1;
            q.tel_out = nullptr;
            q.k_end = max_pos + 1;
            q.start0 = start0;  // (by position)
            rc = kvs_launch_simulate_reg(q, st);
            if (rc != KVSCHED_OK) return rc;
            rc = kvs_launch_mark_noop_moves(moves, K, n, min_pos, max_pos + 1 - min_pos, start0 + min_pos, state,
                                            rejoin_block, st);
            if (rc != KVSCHED_OK) return rc;
            p.skip = rejoin_block;
            stops_early = true;
        }
    }
    if (!p.state_in && ctx->resume_wait_polls > 0 && resume_pays(ctx, K + 1, n, o_bound)) {
        // Moves anywhere in the order (no prefix common to all): a move at positions i, j leaves the
        // positions before min(i, j) as they are, so its timeline starts from the state the base
        // order's timeline (run in the same launch) has saved at the last 64-position boundary before.
        const int32_t C = K + 1;
        const int32_t nblk = (n - 1) / WAVE_POSITIONS;
        const int32_t stride = kvs_reg_state_words(o_bound);
        const size_t list_bytes = align256(sizeof(int32_t) * (size_t)C);
        char *plan = (char *)work + plan_offset;
        int32_t *blocks = (int32_t *)plan;
        int32_t *sorted = (int32_t *)(plan + list_bytes);
        int32_t *tmp = (int32_t *)(plan + 2 * list_bytes);
        int32_t *flags = (int32_t *)(plan + 3 * list_bytes);
        int32_t *snaps = (int32_t *)(plan + 3 * list_bytes + align256(sizeof(int32_t) * KVS_PROGRESS_WORDS));
        rc = kvs_launch_move_blocks(moves, K, n, blocks, st);
        if (rc != KVSCHED_OK) return rc;
        rc = kvs_launch_sort_by_blocks(blocks, C, K, tmp, sorted, flags, KVS_PROGRESS_WORDS, st);  // (clears the progress word too)
        if (rc != KVSCHED_OK) return rc;
        p.cand_list = sorted;
        p.resume_block = blocks;
        p.snapshots = snaps;
        p.snap_stride = stride;
        p.snap_blocks = nblk;
        p.snap_flags = flags;
        p.snap_wait_polls = ctx->resume_wait_polls;
        p.snap_cand = K;
        p.rejoin_block = rejoin_block;  // a move's timeline stops where it has become the base order's again
        p.start0 = start0;
        p.rejoin_blocks = nblk;
        stops_early = true;
        if (ctx->timing && hipEventRecord(ctx->ev0, st) != hipSuccess) return KVSCHED_EHIP;
        rc = kvs_launch_simulate_reg(p, st);
        if (rc == KVSCHED_OK && ctx->timing) {
            if (hipEventRecord(ctx->ev1, st) != hipSuccess) return KVSCHED_EHIP;
            ctx->timed = 1;
        }
    } else {
        rc = run_timelines(ctx, p, H, st);
    }
    if (rc != KVSCHED_OK) return rc;
    if (stops_early && work == ctx->d_scratch) {
        ctx->neighbor_stop_offset = (size_t)((char *)rejoin_block - (char *)work);
        ctx->neighbor_moves = K;
    }
    rc = kvs_launch_check_orders(base_order, 1, n, tel + K, ctx->d_words, st);
    if (rc != KVSCHED_OK) return rc;
    return kvs_launch_neighbor_finish(tel, stops_early ? rejoin_block : nullptr, moves, K, n, tel_out, result_out,
                                      ctx->d_words, st);
}

// A horizon step without saved states: best neighbour, the move, the chosen timeline from its first position, commit point.
static int horizon_step_plain(kvsched_ctx *ctx, int32_t *order, int32_t n, const int32_t *moves, int32_t K, const int32_t *s,
                              const int32_t *o, int64_t M, int64_t completed_in, int32_t complete_every, int64_t *tel_out,
                              int32_t *completion_out, int64_t *result_out, hipStream_t st)
{
    char *base = (char *)ctx->d_scratch;
    const size_t tel_bytes = neighbor_scratch_bytes(K, n, ctx->o_max_bound);
    int32_t *new_order = (int32_t *)(base + tel_bytes);
    int64_t *tel1 = (int64_t *)(base + tel_bytes + align256(sizeof(int32_t) * (size_t)n));
    int32_t *comp = completion_out ? completion_out : horizon_kept(ctx, n).completion;
    int rc = best_neighbor_on(ctx, ctx->d_scratch, ctx->o_max_bound, order, n, moves, K, s, o, M, tel_out, result_out, st);
    if (rc != KVSCHED_OK) return rc;
    rc = kvs_launch_apply_best_move(order, n, moves, result_out, new_order, st);
    if (rc != KVSCHED_OK) return rc;
    hipLaunchKernelGGL(kvs_copy_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, order, new_order, n);
    if (hipGetLastError() != hipSuccess) return KVSCHED_EHIP;
    const int32_t o_bound = ctx->o_max_bound > 0 ? ctx->o_max_bound : scanned_longest(ctx);
    SimParams p;
    p.src.orders = order;
    p.src.base = nullptr;
    p.src.moves = nullptr;
    p.C = 1;
    p.n = n;
    p.s = s;
    p.o = o;
    p.M = (int32_t)M;
    p.tel_out = tel1;
    p.completion_out = comp;
    p.completion_by_position = 0;
    p.d_words = ctx->d_words;
    p.o_bound = o_bound;
    rc = p.o_bound <= KVS_REG_MAX_O ? kvs_launch_simulate_reg(p, st)
                                    : kvs_launch_simulate(p, ring_slots_for(o_bound), st);
    if (rc != KVSCHED_OK) return rc;
    if (!completion_out) {
        ctx->hz_completion = 2;
        ctx->hz_n = n;
    }
    return kvs_launch_horizon_advance_by_id(order, comp, o, n, completed_in, complete_every, result_out, st);
}

int kvsched_best_neighbor(kvsched_ctx *ctx, const int32_t *base_order, int32_t n, const int32_t *moves, int32_t K,
                          const int32_t *s, const int32_t *o, int64_t M, int64_t *tel_out, int64_t *result_out,
                          void *stream)
{
    int rc = check_common(ctx, n, s, o, M);
    if (rc != KVSCHED_OK) return rc;
    if (!base_order || !moves || !result_out || K < 1 || K == INT32_MAX) return KVSCHED_EINVAL;
    rc = ensure_scratch(ctx, neighbor_scratch_bytes(K, n, ctx->o_max_bound));
    if (rc != KVSCHED_OK) return rc;
    return best_neighbor_on(ctx, ctx->d_scratch, ctx->o_max_bound, base_order, n, moves, K, s, o, M, tel_out,
                            result_out, (hipStream_t)stream);
}

int kvsched_best_neighbor_static(kvsched_ctx *ctx, const int32_t *base_order, int32_t n, const int32_t *moves,
                                 int32_t K, const int32_t *s, const int32_t *o, int64_t M, int32_t o_max_bound,
                                 int64_t *tel_out, int64_t *result_out, void *stream)
{
    int rc = check_common(ctx, n, s, o, M);
    if (rc != KVSCHED_OK) return rc;
    if (!base_order || !moves || !result_out || K < 1 || K == INT32_MAX || o_max_bound < 1) return KVSCHED_EINVAL;
    if (o_max_bound > KVSCHED_MAX_O) return KVSCHED_ERANGE;
    if (!ctx->static_scratch) return KVSCHED_ERANGE;  // device number beyond the table of resolved addresses
    if (neighbor_scratch_bytes(K, n, o_max_bound) > KVS_STATIC_SCRATCH_BYTES) return KVSCHED_ERANGE;
    // Nothing in the array has to start at zero: the latencies, the prefix state and the plan's lists are
    // written before they are read, and the progress word of the hand-over is cleared by the kernel that
    // sorts the plan.
    return best_neighbor_on(ctx, ctx->static_scratch, o_max_bound, base_order, n, moves, K, s, o, M, tel_out,
                            result_out, (hipStream_t)stream);
}

int kvsched_horizon_step(kvsched_ctx *ctx, int32_t *order, int32_t n, const int32_t *moves, int32_t K,
                         const int32_t *s, const int32_t *o, int64_t M, int64_t completed_in, int32_t complete_every,
                         int64_t *tel_out, int32_t *completion_out, int64_t *result_out, void *stream)
{
    int rc = check_common(ctx, n, s, o, M);
    if (rc != KVSCHED_OK) return rc;
    if (!order || !moves || !result_out || completed_in < 0 || complete_every < 1) return KVSCHED_EINVAL;
    if (K < 1 || K == INT32_MAX) return KVSCHED_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    ctx->hz_completion = 0;
    // scratch: [K+1] latencies of best_neighbor and its plan | new order [n] | one latency
    const size_t tel_bytes = neighbor_scratch_bytes(K, n, ctx->o_max_bound);
    const size_t row_bytes = align256(sizeof(int32_t) * (size_t)n);
    rc = ensure_scratch(ctx, tel_bytes + row_bytes + 256);
    if (rc != KVSCHED_OK) return rc;
    char *base = (char *)ctx->d_scratch;
    int32_t o_bound = ctx->o_max_bound;
    const bool states_wanted = n > 2 * WAVE_POSITIONS && ctx->resume_wait_polls > 0 && ctx->resume_min_rows != 0;
    if (!(states_wanted && o_bound <= KVS_REG_MAX_O)) {  // short orders, and where saved states are ruled out: step by step
        ctx->hz_kept = 0;
        rc = ensure_horizon(ctx, horizon_bytes(n, 0));
        if (rc != KVSCHED_OK) return rc;
        return horizon_step_plain(ctx, order, n, moves, K, s, o, M, completed_in, complete_every, tel_out, completion_out,
                                  result_out, st);
    }
    rc = scan_and_bound(ctx, s, o, n, M, st, &o_bound, moves, K);
    if (rc != KVSCHED_OK) return rc;
    if ((int64_t)n * (int64_t)ring_slots_for(o_bound) >= kMaxM) return KVSCHED_ERANGE;
    if (o_bound > KVS_REG_MAX_O) {
        ctx->hz_kept = 0;
        rc = ensure_horizon(ctx, horizon_bytes(n, 0));
        if (rc != KVSCHED_OK) return rc;
        return horizon_step_plain(ctx, order, n, moves, K, s, o, M, completed_in, complete_every, tel_out, completion_out,
                                  result_out, st);
    }
    const int32_t stride = kvs_reg_state_words(o_bound), nblk = (n - 1) / WAVE_POSITIONS, C = K + 1;
    rc = ensure_horizon(ctx, horizon_bytes(n, stride));
    if (rc != KVSCHED_OK) return rc;
    const HorizonKept h = horizon_kept(ctx, n);
    // (a state holds the largest file's words or fewer: kept ones are of use only to the same file)
    const int32_t kept = ctx->hz_kept && ctx->hz_n == n && ctx->hz_M == M && kvs_reg_state_words(ctx->hz_o_bound) == stride;
    ctx->hz_kept = 0;  // (until this step has left its own)
    // 1. the candidates.  Each starts from the state saved at the last 64-position boundary before what its move
    //    touches: left there by the step before as far as that placed its order, and beyond by the wave that runs the
    //    order as it stands, in the same launch.
    const size_t list_bytes = align256(sizeof(int32_t) * (size_t)C);
    int64_t *tel = (int64_t *)base;
    char *lists = base + align256(sizeof(int64_t) * (size_t)C) + state_bytes();
    int32_t *rejoin_block = (int32_t *)lists;
    int32_t *blocks = (int32_t *)(lists + list_bytes + row_bytes);
    int32_t *sorted = (int32_t *)(lists + 2 * list_bytes + row_bytes);
    int32_t *tmp = (int32_t *)(lists + 3 * list_bytes + row_bytes);
    rc = kvs_launch_horizon_begin(h, kept, order, s, o, n, moves, K, blocks, st);
    if (rc != KVSCHED_OK) return rc;
    rc = kvs_launch_sort_by_blocks(blocks, C, K, tmp, sorted, nullptr, 0, st);
    if (rc != KVSCHED_OK) return rc;
    SimParams p;
    p.src.orders = nullptr;
    p.src.base = order;
    p.src.moves = moves;
    p.C = C;
    p.n = n;
    p.s = s;
    p.o = o;
    p.M = (int32_t)M;
    p.tel_out = tel;
    p.completion_out = nullptr;
    p.completion_by_position = 0;
    p.d_words = ctx->d_words;
    p.o_bound = o_bound;
    p.cand_list = sorted;
    p.resume_block = blocks;
    p.snapshots = h.snapshots;
    p.snap_stride = stride;
    p.snap_blocks = nblk;
    p.snap_flags = h.progress;
    p.snap_wait_polls = ctx->resume_wait_polls;
    p.snap_cand = K;
    p.snap_start = h.ctrl + KVS_HZ_AVAIL;
    p.rejoin_block = rejoin_block;
    p.start0 = h.start;
    p.rejoin_blocks = nblk;
    if (ctx->timing && hipEventRecord(ctx->ev0, st) != hipSuccess) return KVSCHED_EHIP;
    rc = kvs_launch_simulate_reg(p, st);
    if (rc != KVSCHED_OK) return rc;
    if (ctx->timing) {
        if (hipEventRecord(ctx->ev1, st) != hipSuccess) return KVSCHED_EHIP;
        ctx->timed = 1;
    }
    ctx->neighbor_stop_offset = (size_t)((char *)rejoin_block - base);
    ctx->neighbor_moves = K;
    rc = kvs_launch_check_orders(order, 1, n, tel + K, ctx->d_words, st);
    if (rc != KVSCHED_OK) return rc;
    rc = kvs_launch_neighbor_finish(tel, rejoin_block, moves, K, n, tel_out, result_out, ctx->d_words, st);
    if (rc != KVSCHED_OK) return rc;
    // 2. the best move is taken; 3. the new order's timeline, from the first block that changed, to its end if its
    //    completion rounds are asked for, else until the commit point is behind it; 4. the commit point
    rc = kvs_launch_horizon_choose(h, order, n, moves, result_out, ctx->d_words, stride, completed_in, complete_every,
                                   completion_out ? 1 : 0, st);
    if (rc != KVSCHED_OK) return rc;
    SimParams q;
    q.src.orders = order;
    q.src.base = nullptr;
    q.src.moves = nullptr;
    q.C = 1;
    q.n = n;
    q.s = s;
    q.o = o;
    q.M = (int32_t)M;
    q.tel_out = nullptr;
    q.completion_out = nullptr;
    q.completion_by_position = 0;
    q.d_words = ctx->d_words;
    q.o_bound = o_bound;
    q.cand_list = h.ctrl + KVS_HZ_ZERO;
    q.snapshots = h.snapshots;
    q.snap_stride = stride;
    q.snap_blocks = nblk;
    q.snap_start = h.ctrl + KVS_HZ_FIRST;
    q.t_limit = h.ctrl + KVS_HZ_LIMIT;
    q.placed_out = h.ctrl + KVS_HZ_PLACED;
    q.start0 = h.start;
    rc = kvs_launch_simulate_reg(q, st);
    if (rc != KVSCHED_OK) return rc;
    rc = kvs_launch_horizon_advance(h, order, n, nblk, completed_in, complete_every, completion_out, result_out + 3, st);
    if (rc != KVSCHED_OK) return rc;
    ctx->hz_kept = ctx->hz_completion = 1;
    ctx->hz_n = n;
    ctx->hz_M = M;
    ctx->hz_o_bound = o_bound;
    return KVSCHED_OK;
}

int kvsched_horizon_completion(kvsched_ctx *ctx, const int32_t *order, int32_t n, const int32_t *o, int32_t *completion_out,
                               void *stream)
{
    if (!ctx || !order || !o || !completion_out || n < 1 || !ctx->hz_completion || ctx->hz_n != n) return KVSCHED_EINVAL;
    if (hipSetDevice(ctx->device) != hipSuccess) return KVSCHED_EHIP;
    const HorizonKept h = horizon_kept(ctx, n);
    if (ctx->hz_completion == 1) return kvs_launch_horizon_completion(h, order, o, n, completion_out, (hipStream_t)stream);
    hipLaunchKernelGGL(kvs_copy_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, completion_out,
                       h.completion, n);
    return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
}

int kvsched_online(kvsched_ctx *ctx, int32_t B, const int32_t *streams, int32_t N, const int32_t *a,
                   const int32_t *s, const int32_t *o, int64_t M, int32_t backlog_cap, int32_t *completion_out,
                   int32_t out_len, int64_t *stats_out, void *stream)
{
    int rc = check_common(ctx, N, s, o, M);
    if (rc != KVSCHED_OK) return rc;
    if (!streams || !a || !completion_out || !stats_out || B < 1 || out_len < 1 || backlog_cap < 1)
        return KVSCHED_EINVAL;
    if (backlog_cap > KVSCHED_ONLINE_MAX_BACKLOG) return KVSCHED_ERANGE;
    hipStream_t st = (hipStream_t)stream;
    int32_t o_bound = 0;
    rc = scan_and_bound(ctx, s, o, N, M, st, &o_bound);
    if (rc != KVSCHED_OK) return rc;
    if (o_bound > KVSCHED_ONLINE_MAX_O) return KVSCHED_ERANGE;
    int32_t H = 64;  // ring of the running requests' future memory: a slot per round of the longest decode
    while (H < o_bound) H <<= 1;
    // More streams than run at once: those with most work go first (the order needs 2 B ints of scratch).
    int32_t *order_scratch = nullptr;
    if (B > kOnlineOrderMinStreams) {
        rc = ensure_scratch(ctx, 2 * sizeof(int32_t) * (size_t)B);
        if (rc != KVSCHED_OK) return rc;
        order_scratch = (int32_t *)ctx->d_scratch;
    }
    return kvs_launch_online(B, streams, N, a, s, o, (int32_t)M, backlog_cap, H, completion_out, out_len, stats_out,
                             order_scratch, ctx->d_words, st);
}

int kvsched_simulate_resume_positions(kvsched_ctx *ctx, int32_t C, int32_t *resume_pos_out, void *stream)
{
    if (!ctx || !resume_pos_out || C < 1) return KVSCHED_EINVAL;
    if (hipSetDevice(ctx->device) != hipSuccess) return KVSCHED_EHIP;
    hipStream_t st = (hipStream_t)stream;
    if (ctx->resume_rows == 0) {  // the last call placed every row from its first position
        hipLaunchKernelGGL(kvs_fill_zero_i32, dim3((unsigned)((C + 255) / 256)), dim3(256), 0, st, resume_pos_out, C);
        return hipGetLastError() == hipSuccess ? KVSCHED_OK : KVSCHED_EHIP;
    }
    if (C != ctx->resume_rows) return KVSCHED_EINVAL;
    const size_t list_bytes = align256(sizeof(int32_t) * (size_t)C);
    const int32_t *blocks = (const int32_t *)ctx->d_scratch;
    const int32_t *sorted = (const int32_t *)((const char *)ctx->d_scratch + list_bytes);
    return kvs_launch_resume_plan(sorted, C, ctx->resume_first, blocks, resume_pos_out, st);
}

int kvsched_simulate_stop_positions(kvsched_ctx *ctx, int32_t C, int32_t n, int32_t *stop_pos_out, void *stream)
{
    if (!ctx || !stop_pos_out || C < 1 || n < 1) return KVSCHED_EINVAL;
    if (hipSetDevice(ctx->device) != hipSuccess) return KVSCHED_EHIP;
    if (ctx->rejoin_offset != 0 && C != ctx->resume_rows) return KVSCHED_EINVAL;
    const int32_t *rejoin =
        ctx->rejoin_offset != 0 ? (const int32_t *)((const char *)ctx->d_scratch + ctx->rejoin_offset) : nullptr;
    return kvs_launch_stop_positions(rejoin, C, n, stop_pos_out, (hipStream_t)stream);
}

int kvsched_neighbor_stop_positions(kvsched_ctx *ctx, int32_t K, int32_t n, int32_t *stop_pos_out, void *stream)
{
    if (!ctx || !stop_pos_out || K < 1 || n < 1) return KVSCHED_EINVAL;
    if (hipSetDevice(ctx->device) != hipSuccess) return KVSCHED_EHIP;
    if (ctx->neighbor_stop_offset != 0 && K != ctx->neighbor_moves) return KVSCHED_EINVAL;
    const int32_t *rejoin = ctx->neighbor_stop_offset != 0
                                ? (const int32_t *)((const char *)ctx->d_scratch + ctx->neighbor_stop_offset)
                                : nullptr;
    return kvs_launch_stop_positions(rejoin, K, n, stop_pos_out, (hipStream_t)stream);
}

int kvsched_simulate_predicted(kvsched_ctx *ctx, const int32_t *orders, int32_t C, int32_t n, const int32_t *s,
                               const int32_t *o, const int32_t *est0, int32_t E, int64_t M, int64_t *tel_out,
                               int32_t *completion_out, int32_t *evictions_out, void *stream)
{
    int rc = check_common(ctx, n, s, o, M);
    if (rc != KVSCHED_OK) return rc;
    if (!orders || !est0 || !tel_out || C < 1 || (E != 1 && E != C)) return KVSCHED_EINVAL;
    if (n > 65535) return KVSCHED_ERANGE;
    hipStream_t st = (hipStream_t)stream;
    rc = kvs_launch_scan_lengths(s, o, n, (int32_t)M, ctx->o_max_bound, ctx->d_words, st);
    if (rc != KVSCHED_OK) return rc;
    int32_t bound = ctx->o_max_bound;
    if (bound <= 0) {
        rc = kvs_launch_scan_estimates(est0, (size_t)E * (size_t)n, ctx->d_words, st);
        if (rc != KVSCHED_OK) return rc;
        rc = read_words(ctx, st);
        if (rc != KVSCHED_OK) return rc;
        bound = ctx->h_words[KVS_W_OMAX] > ctx->h_words[KVS_W_ESTMAX] ? ctx->h_words[KVS_W_OMAX]
                                                                      : ctx->h_words[KVS_W_ESTMAX];
    }
    if (bound > KVSCHED_MAX_O) return KVSCHED_ERANGE;
    const int32_t H = ring_slots_for(bound < 1 ? 1 : bound);
    if (kvs_predicted_lds_bytes(n, H) > KVS_PREDICTED_MAX_LDS) return KVSCHED_ERANGE;
    // which candidates need the second launch; the estimates that stopped requests keep (written before read)
    const size_t retry_bytes = align256(sizeof(int32_t) * (size_t)C);
    rc = ensure_scratch(ctx, retry_bytes + sizeof(uint16_t) * (size_t)C * (size_t)n);
    if (rc != KVSCHED_OK) return rc;
    rc = kvs_launch_predicted(orders, C, n, s, o, est0, E, (int32_t)M, H, 1 << 26, tel_out, completion_out,
                              evictions_out, (int32_t *)ctx->d_scratch, (uint16_t *)((char *)ctx->d_scratch + retry_bytes),
                              ctx->d_words, st);
    if (rc != KVSCHED_OK) return rc;
    return kvs_launch_check_orders(orders, C, n, tel_out, ctx->d_words, st);
}

int kvsched_argmin(kvsched_ctx *ctx, const int64_t *tel, int32_t C, int64_t *result_out, void *stream)
{
    if (!ctx || !tel || !result_out || C < 1) return KVSCHED_EINVAL;
    if (hipSetDevice(ctx->device) != hipSuccess) return KVSCHED_EHIP;
    return kvs_launch_argmin(tel, C, result_out, ctx->d_words, (hipStream_t)stream);
}

}  // extern "C"
