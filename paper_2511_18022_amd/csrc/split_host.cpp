// C-ABI host layer of libsplitgpu.so: argument checking, device buffers, kernel launches, the
// autotuner, captured evaluation graphs, and the conversion of the exact device moments into
// the sample mean and variance.
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <utility>
#include <vector>

#include "split_internal.h"

using namespace splitgpu;

namespace {

constexpr int kStages = 8;              // pinned host slots for tour uploads
// SPLIT_FORM_AUTO takes the wave form for short tours over few scenarios, where the lane
// kernel's per-item prologue outweighs its per-state advantage. Measured crossover of whole
// evaluations (tours of 8..256 positions): the wave form is ahead up to n = 32 at S = 256, up to
// n = 24 at S = 1024 and up to n = 16 at S = 4096; the lane form everywhere else (at n = 1000
// from S = 1024 on, at 2.6x and more).
bool auto_wave(int64_t S, int32_t maxn)
{
    if (S <= 256) return maxn <= 32;
    if (S <= 1024) return maxn <= 24;
    if (S <= 4096) return maxn <= 16;
    return false;
}
// The lane kernel compares load differences in 16 bits, exact while 8 * max(q) + Q < 2^15;
// evaluations with a larger capacity run in the wave form, which is exact for any Q.
constexpr int32_t kLaneMaxQ = 16383;
constexpr int kMaxTimingPairs = 4096;
constexpr int kGraphSlots = 2;          // a graph's launches alternate between two host slots
constexpr int32_t kMaxLanePerCu = 8;    // the lane kernel's LDS allows 8 workgroups per CU
constexpr int32_t kLaneStaticPerCu = kMaxLanePerCu;  // fixed-stride grid: all resident at once
constexpr int64_t kLaneStaticMaxRounds = 16;         // and at most this many items each
constexpr int32_t kTailPerCu = 2;       // the tail kernel's LDS allows 2 workgroups per CU
constexpr int32_t kPairPerCu = 4;       // as many of the pair kernel's: two wavefronts a SIMD
constexpr int32_t kPairMaxQ = 2047;     // a demand of Q itself stays within the 16-bit bound
constexpr int64_t kClassMaxArc = 2047;  // 16 states times 2 max_arc: below 2^16

// Device buffers of one evaluation sequence. The context's grow with its calls; a graph owns
// a fixed set.
struct EvalBuffers {
    char *d_stage = nullptr;  // staged header, see TourDev
    int64_t cap_stage = 0;
    int64_t *d_rowoff = nullptr;
    uint32_t *d_rowoff32 = nullptr;
    int32_t *d_w = nullptr;
    uint32_t *d_rowoff32_back = nullptr;  // pair kernel only, as the two after it
    int32_t *d_w_back = nullptr;
    int64_t cap_back = 0;
    int64_t cap_pos = 0;      // entries of the per-tour arrays
    DevStats *d_stats = nullptr;
    int32_t cap_T = 0;
    char *d_sums = nullptr;
    int64_t cap_sums = 0;  // bytes
    BatchCtl *d_ctl = nullptr;
    int16_t *d_mask = nullptr;  // two-kernel form only: window starts [positions][S]
    int64_t cap_mask = 0;       // elements
};

void free_buffers(EvalBuffers &b)
{
    if (b.d_stage) (void)hipFree(b.d_stage);
    if (b.d_rowoff) (void)hipFree(b.d_rowoff);
    if (b.d_rowoff32) (void)hipFree(b.d_rowoff32);
    if (b.d_w) (void)hipFree(b.d_w);
    if (b.d_rowoff32_back) (void)hipFree(b.d_rowoff32_back);
    if (b.d_w_back) (void)hipFree(b.d_w_back);
    if (b.d_stats) (void)hipFree(b.d_stats);
    if (b.d_sums) (void)hipFree(b.d_sums);
    if (b.d_ctl) (void)hipFree(b.d_ctl);
    if (b.d_mask) (void)hipFree(b.d_mask);
    b = EvalBuffers();
}

// Byte offsets of the staged header for capacity capT tours and cap_n positions:
// int64 T at 0, int64 tptr[capT + 1] at 8, int32 order[capT], int32 tours[cap_n].
struct StageLayout {
    int32_t capT = 0;
    size_t off_order = 0, off_tours = 0, bytes = 0;
};

StageLayout stage_layout(int32_t capT, int64_t cap_n)
{
    StageLayout L;
    L.capT = capT;
    L.off_order = sizeof(int64_t) * (2 + (size_t)capT);
    L.off_tours = L.off_order + ((sizeof(int32_t) * (size_t)capT + 7) & ~(size_t)7);
    L.bytes = L.off_tours + sizeof(int32_t) * (size_t)cap_n;
    return L;
}

// Summary of a validated batch.
struct BatchInfo {
    int32_t T = 0, max_id = 0, maxn = 0, minn = 0;
    int64_t total_n = 0;
};

// What the kernels of one evaluation are launched with.
struct Plan {
    int form = SPLIT_FORM_LANE;
    int32_t lane_grid = 0, wave_grid = 0, maxn = 0, lane_block = 16;
    int32_t tail_grid = 0;
    bool lane_static = false, lane_uniform = false, pair = false;
    uint32_t lane_bytes = 0;
};

// A timed call: its DP kernel from start to dp, and (lane form: the tail kernel may do the DP) its
// tail kernel from dp to end.
struct TimedCall {
    hipEvent_t start = nullptr, dp = nullptr, end = nullptr;
    const char *name = "";
    bool tail = false;
};

// The instance as the kernels see it (a graph keeps its own copy).
struct Instance {
    int32_t N = 0;
    int kind = -1;  // 0 coordinates, 1 matrix
    int32_t *d_xy = nullptr;
    int32_t *d_dist = nullptr;
    int64_t max_arc = 0;
};

void free_instance(Instance &in)
{
    if (in.d_xy) (void)hipFree(in.d_xy);
    if (in.d_dist) (void)hipFree(in.d_dist);
    in = Instance();
}

}  // namespace

struct split_ctx {
    int device = 0;
    int cus = 0;
    std::string err;
    split_tuning tuning = {SPLIT_FORM_AUTO, 0, 0, 0, 0};

    Instance inst;
    std::vector<unsigned char> seen;

    EvalBuffers buf;

    // pinned host staging
    char *h_stage[kStages] = {};
    int64_t cap_h_stage = 0;
    hipEvent_t stage_ev[kStages] = {};
    bool stage_ev_used[kStages] = {};
    int stage = 0;
    TourResult *h_stats = nullptr;
    int32_t cap_h_stats = 0;
    hipEvent_t last_ev = nullptr;  // end of the latest call (one of stage_ev)
    bool have_call = false;
    int64_t last_S = 0;
    int32_t last_T = 0;
    int32_t last_parts = 0;  // nonzero: h_stats holds this many parts of one tour's result

    // timing of the dominant kernel
    bool timing = false;
    std::vector<TimedCall> timed;
    size_t timed_used = 0;
    double ms_acc = 0.0;
    int64_t launches = 0;
    std::vector<float> ms_samples;  // per timed launch since the last reset
    const char *tname = "";

    // device address of this GPU's fixed scratch (split_eval_noalloc), looked up at creation
    unsigned char *scratch = nullptr;
    void *topk = nullptr;  // device scratch of split_topk_smallest, kept between calls
};

struct split_graph {
    split_ctx *ctx = nullptr;  // for error messages and the device
    Instance inst;
    std::vector<unsigned char> seen;
    EvalBuffers buf;
    StageLayout layout;
    int32_t max_T = 0;
    int64_t max_total_n = 0;
    int64_t S = 0, ld = 0, ldc = 0;
    int32_t Q = 0;
    int order = 0;
    Plan plan;
    hipStream_t cap_stream = nullptr;
    char *h_stage[kGraphSlots] = {};
    TourResult *h_stats[kGraphSlots] = {};
    // per host slot; [1] with the pair kernel, for replays of long tours (where plan.pair)
    hipGraph_t graph[kGraphSlots][2] = {};
    hipGraphExec_t exec[kGraphSlots][2] = {};
    hipEvent_t done[kGraphSlots] = {};
    bool used[kGraphSlots] = {};
    int next = 0;
    int last = -1;
    int32_t last_T = 0;
};

namespace {

split_status fail(split_ctx *ctx, split_status st, const char *fmt, ...)
{
    if (ctx) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        ctx->err = buf;
    }
    return st;
}

split_status hip_fail(split_ctx *ctx, hipError_t e, const char *what)
{
    return fail(ctx, SPLIT_E_HIP, "%s: %s", what, hipGetErrorString(e));
}

#define HIP_TRY(ctx, expr)                                   \
    do {                                                     \
        hipError_t e_ = (expr);                              \
        if (e_ != hipSuccess) return hip_fail(ctx, e_, #expr); \
    } while (0)

// Makes ctx->device current for the scope of one API call and restores the caller's device.
struct DeviceGuard {
    int prev = -1;
    bool ok = false;
    explicit DeviceGuard(int dev)
    {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        ok = hipSetDevice(dev) == hipSuccess;
    }
    ~DeviceGuard()
    {
        if (prev >= 0) (void)hipSetDevice(prev);
    }
};

template <class P>
bool grow(P **ptr, size_t bytes)
{
    if (*ptr) (void)hipFree(*ptr);
    *ptr = nullptr;
    return hipMalloc(ptr, bytes) == hipSuccess;
}

// Device buffers for T tours with total_n positions in all, a header of stage_bytes and sum_bytes
// of cost sums (exact sizes, or with room to grow). Growing waits for
// enqueued work before replacing a buffer.
split_status ensure_buffers(split_ctx *ctx, EvalBuffers &b, int32_t T, int64_t total_n,
                            int64_t stage_bytes, int64_t sum_bytes, bool pair, bool exact)
{
    const int64_t pos = total_n + (int64_t)T * (1 + kRowPad);
    const bool g_pos = pos > b.cap_pos, g_stage = stage_bytes > b.cap_stage;
    const bool g_T = T > b.cap_T, g_sums = sum_bytes > b.cap_sums;
    const bool g_ctl = b.d_ctl == nullptr;
    const bool g_back = pair && pos > b.cap_back;
    if (!g_pos && !g_stage && !g_T && !g_sums && !g_ctl && !g_back) return SPLIT_OK;
    HIP_TRY(ctx, hipDeviceSynchronize());
    auto room = [exact](int64_t need, int64_t floor) {
        return exact ? need : (need < floor ? floor : need + need / 4);
    };
    if (g_pos) {
        const int64_t np = room(pos, 4096);
        b.cap_pos = 0;
        if (!grow(&b.d_rowoff, sizeof(int64_t) * np) ||
            !grow(&b.d_rowoff32, sizeof(uint32_t) * np) || !grow(&b.d_w, sizeof(int32_t) * np))
            return fail(ctx, SPLIT_E_NOMEM, "device allocation for %lld tour positions failed",
                        (long long)np);
        b.cap_pos = np;
    }
    if (g_back) {
        const int64_t np = room(pos, 4096);
        b.cap_back = 0;
        if (!grow(&b.d_rowoff32_back, sizeof(uint32_t) * np) ||
            !grow(&b.d_w_back, sizeof(int32_t) * np))
            return fail(ctx, SPLIT_E_NOMEM, "device allocation for %lld tour positions failed",
                        (long long)np);
        b.cap_back = np;
    }
    if (g_stage) {
        const int64_t nb = room(stage_bytes, 65536);
        b.cap_stage = 0;
        if (!grow(&b.d_stage, (size_t)nb))
            return fail(ctx, SPLIT_E_NOMEM, "device staging of %lld bytes failed", (long long)nb);
        b.cap_stage = nb;
    }
    if (g_T) {
        const int32_t nt = exact ? T : (T < 16 ? 16 : T);
        b.cap_T = 0;
        if (!grow(&b.d_stats, sizeof(DevStats) * nt))
            return fail(ctx, SPLIT_E_NOMEM, "allocation of %d result blocks failed", nt);
        b.cap_T = nt;
    }
    if (g_sums) {
        const int64_t nb = room(sum_bytes, 65536);
        b.cap_sums = 0;
        if (!grow(&b.d_sums, (size_t)nb))
            return fail(ctx, SPLIT_E_NOMEM, "allocation of the cost sums failed");
        b.cap_sums = nb;
    }
    if (g_ctl && hipMalloc(&b.d_ctl, sizeof(BatchCtl)) != hipSuccess)
        return fail(ctx, SPLIT_E_NOMEM, "allocation of the batch counters failed");
    return SPLIT_OK;
}

// Pinned host memory that kernels read and write themselves: coherent, so that neither side sees
// what a cache kept from an earlier call.
template <class P>
bool pinned(P **ptr, size_t bytes)
{
    return hipHostMalloc((void **)ptr, bytes, hipHostMallocCoherent) == hipSuccess;
}

// Pinned host staging of the context: kStages slots of stage_bytes and T result blocks.
split_status ensure_host(split_ctx *ctx, int64_t stage_bytes, int32_t T)
{
    if (stage_bytes > ctx->cap_h_stage) {
        HIP_TRY(ctx, hipDeviceSynchronize());
        const int64_t nb = stage_bytes < 65536 ? 65536 : stage_bytes + stage_bytes / 4;
        ctx->cap_h_stage = 0;
        for (int k = 0; k < kStages; ++k) {
            if (ctx->h_stage[k]) (void)hipHostFree(ctx->h_stage[k]);
            ctx->h_stage[k] = nullptr;
            ctx->stage_ev_used[k] = false;
            if (!pinned(&ctx->h_stage[k], (size_t)nb))
                return fail(ctx, SPLIT_E_NOMEM, "pinned staging of %lld bytes failed",
                            (long long)nb);
        }
        ctx->cap_h_stage = nb;
    }
    if (T > ctx->cap_h_stats) {
        HIP_TRY(ctx, hipDeviceSynchronize());
        const int32_t nt = T < 16 ? 16 : T;
        if (ctx->h_stats) (void)hipHostFree(ctx->h_stats);
        ctx->h_stats = nullptr;
        ctx->cap_h_stats = 0;
        if (!pinned(&ctx->h_stats, sizeof(TourResult) * nt))
            return fail(ctx, SPLIT_E_NOMEM, "pinned allocation of %d result blocks failed", nt);
        memset(ctx->h_stats, 0, sizeof(TourResult) * nt);
        ctx->cap_h_stats = nt;
    }
    return SPLIT_OK;
}

split_status collect_timing(split_ctx *ctx)
{
    for (size_t k = 0; k < ctx->timed_used; ++k) {
        const TimedCall &c = ctx->timed[k];
        HIP_TRY(ctx, hipEventSynchronize(c.tail ? c.end : c.dp));
        float ms = 0.f, tail_ms = 0.f;
        HIP_TRY(ctx, hipEventElapsedTime(&ms, c.start, c.dp));
        if (c.tail) HIP_TRY(ctx, hipEventElapsedTime(&tail_ms, c.dp, c.end));
        ctx->tname = c.name;
        if (tail_ms > ms) {
            ms = tail_ms;
            ctx->tname = tail_kernel_name();
        }
        ctx->ms_acc += ms;
        ctx->launches += 1;
        ctx->ms_samples.push_back(ms);
    }
    ctx->timed_used = 0;
    return SPLIT_OK;
}

// The events of a call whose DP kernel is `name`, the first one recorded; NULL when nothing is timed.
split_status timing_begin(split_ctx *ctx, hipStream_t stream, const char *name, TimedCall **out)
{
    *out = nullptr;
    if (!ctx->timing) return SPLIT_OK;
    if (ctx->timed_used == (size_t)kMaxTimingPairs) {
        split_status st = collect_timing(ctx);
        if (st != SPLIT_OK) return st;
    }
    if (ctx->timed_used == ctx->timed.size()) {
        TimedCall c;
        if (hipEventCreate(&c.start) != hipSuccess || hipEventCreate(&c.dp) != hipSuccess ||
            hipEventCreate(&c.end) != hipSuccess) {
            for (hipEvent_t e : {c.start, c.dp, c.end})
                if (e) (void)hipEventDestroy(e);
            return fail(ctx, SPLIT_E_HIP, "timing: hipEventCreate failed");
        }
        ctx->timed.push_back(c);
    }
    TimedCall &c = ctx->timed[ctx->timed_used];
    HIP_TRY(ctx, hipEventRecord(c.start, stream));
    c.name = name;
    c.tail = false;
    *out = &c;
    return SPLIT_OK;
}

// Counts a call whose kernels were all launched and whose events were all recorded.
void timing_end(split_ctx *ctx, const TimedCall *c)
{
    if (c) ++ctx->timed_used;
}

void fill_stats(const TourResult &d, int64_t S, split_stats *out)
{
    const unsigned __int128 sq = ((unsigned __int128)d.sq_h32 << 32) + d.sq_l32;
    out->sum = (int64_t)d.sum;
    out->sumsq_lo = (uint64_t)sq;
    out->sumsq_hi = (uint64_t)(sq >> 64);
    out->mean = (double)(int64_t)d.sum / (double)S;
    if (S == 1) {
        out->var = 0.0;
    } else {
        const unsigned __int128 sm = d.sum;
        const unsigned __int128 num = (unsigned __int128)(uint64_t)S * sq - sm * sm;
        out->var = ((double)num / (double)S) / (double)(S - 1);
    }
    out->n_fallback = d.ovf_count;
}

// The latest call's results (its end has been waited for): adds up the parts of a small evaluation.
const TourResult *last_results(split_ctx *ctx)
{
    TourResult &r = ctx->h_stats[0];
    for (int32_t k = 1; k < ctx->last_parts; ++k) {
        const TourResult &x = ctx->h_stats[k];
        r.sum += x.sum;
        r.sq_l32 += x.sq_l32;
        r.sq_h32 += x.sq_h32;
        r.err_demand |= x.err_demand;
        r.ovf_count += x.ovf_count;
    }
    ctx->last_parts = 0;
    return ctx->h_stats;
}

// Per-tour statistics and status of T result blocks; SPLIT_E_DEMAND names the first bad tour.
split_status report(split_ctx *ctx, const TourResult *h, int32_t T, int64_t S, split_stats *stats,
                    int32_t *tour_status)
{
    int bad = -1;
    for (int32_t t = 0; t < T; ++t) {
        if (stats) fill_stats(h[t], S, stats + t);
        if (tour_status) tour_status[t] = h[t].err_demand ? SPLIT_E_DEMAND : SPLIT_OK;
        if (h[t].err_demand && bad < 0) bad = t;
    }
    if (bad >= 0)
        return fail(ctx, SPLIT_E_DEMAND, "tour %d: a scenario has a demand q < 0 or q > Q on the "
                    "tour", bad);
    return SPLIT_OK;
}

split_status check_shape(split_ctx *ctx, const char *who, int64_t S, int64_t ld, int32_t Q,
                         int64_t ldc)
{
    if (S < 1 || S > INT32_MAX || ld < S || ldc < S)
        return fail(ctx, SPLIT_E_INVAL, "%s: need 1 <= S < 2^31, ld >= S and ldc >= S", who);
    if (Q < 1) return fail(ctx, SPLIT_E_INVAL, "%s: need Q >= 1", who);
    return SPLIT_OK;
}

// Tours against instance `in` (seen: scratch of N + 1 zeros, left zeroed), the work-item
// bound T * ceil(S / 64) < 2^31 and the int32 range of the DP.
split_status check_tours(split_ctx *ctx, const char *who, const Instance &in,
                         std::vector<unsigned char> &seen, const int32_t *tours,
                         const int64_t *tour_ptr, int32_t T, int64_t S, BatchInfo *info)
{
    if (!tours || !tour_ptr) return fail(ctx, SPLIT_E_INVAL, "%s: NULL pointer", who);
    if (T < 1) return fail(ctx, SPLIT_E_INVAL, "%s: need T >= 1", who);
    if (tour_ptr[0] != 0) return fail(ctx, SPLIT_E_INVAL, "%s: tour_ptr[0] must be 0", who);
    BatchInfo bi;
    bi.T = T;
    for (int32_t t = 0; t < T; ++t) {
        const int64_t n64 = tour_ptr[t + 1] - tour_ptr[t];
        if (n64 < 1 || n64 > in.N)
            return fail(ctx, SPLIT_E_INVAL, "%s: tour %d has length %lld (need 1..N)", who, t,
                        (long long)n64);
        const int32_t n = (int32_t)n64;
        bi.maxn = n > bi.maxn ? n : bi.maxn;
        bi.minn = (t == 0 || n < bi.minn) ? n : bi.minn;
        const int32_t *tour = tours + tour_ptr[t];
        for (int32_t k = 0; k < n; ++k) {
            const int32_t c = tour[k];
            if (c < 1 || c > in.N || seen[c]) {
                for (int32_t j = 0; j < k; ++j) seen[tour[j]] = 0;
                return fail(ctx, SPLIT_E_TOUR, "%s: tour %d position %d: id %d is out of range "
                            "or repeated", who, t, k, c);
            }
            seen[c] = 1;
            bi.max_id = c > bi.max_id ? c : bi.max_id;
        }
        for (int32_t k = 0; k < n; ++k) seen[tour[k]] = 0;
    }
    bi.total_n = tour_ptr[T];
    const int64_t nsb = (S + 63) / 64;
    if ((__int128)nsb * T >= ((__int128)1 << 31))
        return fail(ctx, SPLIT_E_INVAL, "%s: T * ceil(S / 64) must be below 2^31", who);
    // |g| and |w| stay below (2n+3) * max_arc; keep them below 2^30 with a margin.
    if ((__int128)4 * ((__int128)bi.maxn + 1) * in.max_arc >= ((__int128)1 << 31))
        return fail(ctx, SPLIT_E_RANGE, "%s: 4*(n+1)*max_arc = 4*%d*%lld exceeds 2^31", who,
                    bi.maxn + 1, (long long)in.max_arc);
    *info = bi;
    return SPLIT_OK;
}

// Header, work order and tours into host memory h laid out by L (T <= L.capT).
void stage_write(char *h, const StageLayout &L, const int32_t *tours, const int64_t *tour_ptr,
                 int32_t T, int order_mode)
{
    const int64_t T64 = T;
    memcpy(h, &T64, sizeof T64);
    memcpy(h + sizeof(int64_t), tour_ptr, sizeof(int64_t) * ((size_t)T + 1));
    int32_t *order = reinterpret_cast<int32_t *>(h + L.off_order);
    for (int32_t t = 0; t < T; ++t) order[t] = t;
    if (order_mode == 0) {
        // longest tours first (ties by index), so that short ones fill the tail
        std::stable_sort(order, order + T, [&](int32_t x, int32_t y) {
            return tour_ptr[x + 1] - tour_ptr[x] > tour_ptr[y + 1] - tour_ptr[y];
        });
    }
    memcpy(h + L.off_tours, tours, sizeof(int32_t) * (size_t)tour_ptr[T]);
}

// The cost sums of a launch of up to T_grid tours over S scenarios (their buffer left open).
SumSlots sum_slots(int form, int32_t T_grid, int64_t S)
{
    SumSlots s;
    s.base = nullptr;
    // an entry per item up to 128 MiB of them (or 64 a tour); batches beyond that, whose cost matrix
    // takes a GiB and more, keep 64 entries a tour
    const int64_t nsb = (S + 63) / 64;
    s.by_item = form == SPLIT_FORM_LANE && T_grid > 1 &&
                        (nsb <= kMaxSlots || nsb * T_grid <= ((int64_t)1 << 22))
                    ? 1
                    : 0;
    // several tours that add: a power of two that their additions per tour can fill, at most
    const int64_t adds = form == SPLIT_FORM_WAVE ? S : nsb;
    int64_t few = 1;
    while (few < adds && few < kMaxSlots) few *= 2;
    s.slots = s.by_item ? nsb : T_grid > 1 ? few : kMaxSlots;
    s.stride = s.by_item || T_grid > 1 ? (int32_t)sizeof(CostSums) : kSlotStride;
    return s;
}

// Shortest tour that two wavefronts an item pay for. The join takes what half of a tour of fewer than
// about 300 positions saves; past three items a compute unit the halves share their SIMDs, and it takes
// a little more. Whole calls, the pair kernel against the lane kernel, 512 items: 66.3 us against 70.7
// at 320 customers, 71.8 against 78.7 at 400; 768 items: 69.2 and 73.2 at 320, 72.9 and 74.0 at 340;
// 1024 items: 72.8 and 75.4 at 320, 74.3 and 74.1 at 340, 78.4 and 76.1 at 360, 73.3 and 80.4 at 380,
// 86.5 and 93.2 at 500. (Kernels alone, 64 items: 31 us against 25 at 128 positions, 39 and 37 at 256,
// 48 and 62 at 512, 71 and 108 at 1000.)
int32_t pair_min_n(const split_ctx *ctx, int64_t items) { return items <= 3ll * ctx->cus ? 320 : 380; }

// Launch configuration from the tuning. T_grid bounds T; maxn and max_id bound the tours;
// `uniform`: every tour of the launch has the same length (so has every work item).
Plan make_plan(const split_ctx *ctx, const split_tuning &tu, int64_t S, int64_t ld, int32_t Q,
               int32_t T_grid, int32_t maxn, int32_t max_id, bool uniform, int64_t max_arc)
{
    Plan p;
    p.form = tu.form;
    if (p.form == SPLIT_FORM_AUTO) p.form = auto_wave(S, maxn) ? SPLIT_FORM_WAVE : SPLIT_FORM_LANE;
    // past the lane kernel's 16-bit bound every scenario would be handed to the wave kernel
    if (p.form == SPLIT_FORM_LANE && Q > kLaneMaxQ) p.form = SPLIT_FORM_WAVE;
    // the lane kernel addresses demands with 32-bit buffer offsets
    const __int128 lane_bytes = ((__int128)(max_id - 1) * ld + S) * 2;
    const bool lane_addressable = lane_bytes <= (__int128)kRowAbsent;
    p.lane_bytes = lane_addressable ? (uint32_t)lane_bytes : 0u;
    if (p.form == SPLIT_FORM_LANE && !lane_addressable) p.form = SPLIT_FORM_WAVE;
    const int64_t items = (S + 63) / 64 * T_grid;
    // The library's choice (lane_per_cu 0): over one tour with at most kLaneStaticMaxRounds
    // items per workgroup, kLaneStaticPerCu resident workgroups per compute unit taking items
    // at a fixed stride (no dispatch gap between items, no queue); otherwise one workgroup per
    // item. Measured: 8, 12 and 16 items per workgroup of one tour gain about 1%; over several
    // tours, even of one length, their items differ enough that a fixed split lost 2-3%.
    const bool lib_choice = tu.lane_per_cu <= 0;
    const int64_t sgrid = (int64_t)ctx->cus * kLaneStaticPerCu;
    const bool fixed = lib_choice && T_grid == 1 && items <= sgrid * kLaneStaticMaxRounds;
    const int64_t lg = !lib_choice ? (int64_t)ctx->cus * tu.lane_per_cu : fixed ? sgrid : items;
    p.lane_grid = (int32_t)(lg < items ? lg : items);
    p.lane_static = fixed;
    p.lane_uniform = uniform;
    // Left to the library, the block length follows the windows of each item's first positions,
    // where arcs this short keep every suffix offset of either length within 16 bits (at most
    // 2 max_arc a state): n_fallback then does not depend on the length chosen.
    const bool by_class = tu.lane_block == 0 && max_arc <= kClassMaxArc;
    p.lane_block = by_class ? 0 : tu.lane_block == 8 ? 8 : 16;
    p.tail_grid = ctx->cus * kTailPerCu;
    // Two wavefronts per item where they all run at once, at most two on a SIMD: more items than
    // that keep the chip busy with one each.
    p.pair = p.form == SPLIT_FORM_LANE && lib_choice && p.lane_block != 8 &&
             maxn >= pair_min_n(ctx, items) && max_arc <= kClassMaxArc && Q <= kPairMaxQ && items <= (int64_t)ctx->cus * kPairPerCu;
    p.wave_grid = tu.wave_grid > 0 ? tu.wave_grid : 65536;
    p.maxn = maxn;
    return p;
}

// The kernels of one evaluation on `stream`, reading the header `src` (host or device memory, laid
// out by L) and reporting the tours' results to `out`: prep, the Split DP (lane kernel or wave
// kernel), tail. The dominant kernel is timed when ctx->timing and `timed` are set.
split_status enqueue_kernels(split_ctx *ctx, const Instance &in, const EvalBuffers &b,
                             const StageLayout &L, const char *src, TourResult *out,
                             const Plan &p, const int16_t *demand,
                             int64_t S, int64_t ld, int32_t Q, int32_t *cost, int64_t ldc,
                             hipStream_t stream, bool timed)
{
    TourDev td;
    td.nt = reinterpret_cast<int64_t *>(b.d_stage);
    td.tptr = td.nt + 1;
    td.order = reinterpret_cast<int32_t *>(b.d_stage + L.off_order);
    td.T_grid = L.capT;
    td.rowoff = b.d_rowoff;
    td.rowoff32 = b.d_rowoff32;
    td.w = b.d_w;
    td.rowoff32_back = b.d_rowoff32_back;
    td.w_back = b.d_w_back;

    PrepArgs pa;
    pa.tour = td;
    pa.src_nt = reinterpret_cast<const int64_t *>(src);
    pa.src_tptr = pa.src_nt + 1;
    pa.src_order = reinterpret_cast<const int32_t *>(src + L.off_order);
    pa.src_tours = reinterpret_cast<const int32_t *>(src + L.off_tours);
    pa.sums = sum_slots(p.form, L.capT, S);
    pa.sums.base = b.d_sums;
    pa.pair = p.pair ? 1 : 0;
    pa.threads = L.capT > 2 * ctx->cus && p.maxn <= 256 ? 256 : 1024;
    pa.N = in.N;
    pa.kind = in.kind;
    pa.xy = in.d_xy;
    pa.dist = in.d_dist;
    pa.ld = ld;
    pa.stats = b.d_stats;
    pa.ctl = b.d_ctl;
    HIP_TRY(ctx, launch_prep(pa, stream));

    EvalArgs ea;
    ea.demand = reinterpret_cast<const uint16_t *>(demand);
    ea.ld = ld;
    ea.S = S;
    ea.Q = Q;
    ea.tour = td;
    ea.cost = cost;
    ea.ldc = ldc;
    ea.stats = b.d_stats;
    ea.sums = pa.sums;
    ea.out = out;
    ea.ctl = b.d_ctl;
    ea.lane_bytes = p.lane_bytes;
    ea.lane_grid = p.lane_grid;
    ea.lane_static = p.lane_static ? 1 : 0;
    ea.lane_uniform = p.lane_uniform ? 1 : 0;
    ea.lane_block = p.lane_block;
    ea.recount = p.form == SPLIT_FORM_LANE && p.lane_block != 8 ? 1 : 0;
    // blocks of 16 in one wavefront hold every window of a tour of fewer than 64 customers (blocks of 8
    // do not, and the pair kernel marks more than it has to)
    ea.history_min_n = p.form == SPLIT_FORM_LANE && p.lane_block == 16 && !p.pair ? 64 : 0;
    ea.tail_grid = p.tail_grid;
    ea.wave_grid = p.wave_grid;
    ea.maxn = p.maxn;

    const char *name = p.form == SPLIT_FORM_WAVE   ? wave_kernel_name()
                       : p.form == SPLIT_FORM_MASK ? mask_kernel_name()
                       : p.pair                    ? pair_kernel_name()
                                                   : lane_kernel_name();
    ctx->tname = name;
    TimedCall *tc = nullptr;
    if (timed) {
        split_status st = timing_begin(ctx, stream, name, &tc);
        if (st != SPLIT_OK) return st;
    }
    if (p.form == SPLIT_FORM_WAVE) {
        HIP_TRY(ctx, launch_wave_all(ea, stream));
    } else if (p.form == SPLIT_FORM_MASK) {
        HIP_TRY(ctx, launch_mask(ea, b.d_mask, S, stream));
        HIP_TRY(ctx, launch_masked_dp(ea, b.d_mask, S, stream));
    } else {
        HIP_TRY(ctx, p.pair ? launch_pair(ea, stream) : launch_lane(ea, stream));
    }
    if (tc) HIP_TRY(ctx, hipEventRecord(tc->dp, stream));
    HIP_TRY(ctx, launch_tail(ea, stream));
    if (tc && p.form == SPLIT_FORM_LANE) {
        HIP_TRY(ctx, hipEventRecord(tc->end, stream));
        tc->tail = true;
    }
    timing_end(ctx, tc);
    return SPLIT_OK;
}

// One short tour in one launch. The tour travels with the arguments; a slot's event marks the end.
split_status eval_small(split_ctx *ctx, const int32_t *tour, int32_t n, const Plan &p,
                        const int16_t *demand, int64_t S, int64_t ld, int32_t Q, int32_t *cost,
                        hipStream_t stream)
{
    const int32_t parts = (int32_t)((S + kSmallPer - 1) / kSmallPer);
    split_status st = ensure_host(ctx, 1, parts);
    if (st != SPLIT_OK) return st;
    SmallArgs a;
    a.demand = reinterpret_cast<const uint16_t *>(demand);
    a.ld = ld;
    a.S = S;
    a.Q = Q;
    a.n = n;
    a.N = ctx->inst.N;
    a.kind = ctx->inst.kind;
    a.xy = ctx->inst.d_xy;
    a.dist = ctx->inst.d_dist;
    a.cost = cost;
    a.out = ctx->h_stats;
    a.count_bound = p.form == SPLIT_FORM_LANE ? 1 : 0;
    for (int32_t k = 0; k < kSmallN; ++k) a.tour[k] = tour[k < n ? k : n - 1];
    const int slot = ctx->stage;
    ctx->stage = (ctx->stage + 1) % kStages;
    // timed under the name of the form that the rule for several launches takes
    ctx->tname = p.form == SPLIT_FORM_LANE ? lane_kernel_name() : wave_kernel_name();
    TimedCall *tc = nullptr;
    st = timing_begin(ctx, stream, ctx->tname, &tc);
    if (st != SPLIT_OK) return st;
    HIP_TRY(ctx, launch_small(a, stream));
    if (tc) HIP_TRY(ctx, hipEventRecord(tc->dp, stream));
    timing_end(ctx, tc);
    HIP_TRY(ctx, hipEventRecord(ctx->stage_ev[slot], stream));
    ctx->stage_ev_used[slot] = true;
    ctx->last_ev = ctx->stage_ev[slot];
    ctx->have_call = true;
    ctx->last_S = S;
    ctx->last_T = 1;
    ctx->last_parts = parts;
    return SPLIT_OK;
}

// The common path of split_eval and split_eval_batch on the context's own buffers.
split_status eval_batch(split_ctx *ctx, const char *who, const int32_t *tours,
                        const int64_t *tour_ptr, int32_t T, const int16_t *demand, int64_t S,
                        int64_t ld, int32_t Q, int32_t *cost, int64_t ldc, hipStream_t stream)
{
    if (ctx->inst.kind < 0) return fail(ctx, SPLIT_E_INVAL, "%s: no instance set", who);
    if (!demand || !cost) return fail(ctx, SPLIT_E_INVAL, "%s: NULL pointer", who);
    split_status st = check_shape(ctx, who, S, ld, Q, ldc);
    if (st != SPLIT_OK) return st;
    BatchInfo bi;
    st = check_tours(ctx, who, ctx->inst, ctx->seen, tours, tour_ptr, T, S, &bi);
    if (st != SPLIT_OK) return st;

    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, SPLIT_E_HIP, "hipSetDevice failed");
    const StageLayout L = stage_layout(T, bi.total_n);
    const Plan p = make_plan(ctx, ctx->tuning, S, ld, Q, T, bi.maxn, bi.max_id,
                             bi.minn == bi.maxn, ctx->inst.max_arc);
    // A short tour over few scenarios, all choices left to the library: one launch instead of three,
    // which take longer than the work (1 to 32 customers, S = 256 to 32,768: 23 to 30 us a call against
    // 32 to 47, 1.4 to 1.6 times at every corner; the bounds keep the scan of 32 predecessors and the
    // 128 parts to add up small). Short arcs keep every suffix offset within 16 bits, so only the
    // demand bound can count towards n_fallback.
    const split_tuning &tu = ctx->tuning;
    if (T == 1 && bi.maxn <= kSmallN && S <= kSmallS && ctx->inst.max_arc <= kClassMaxArc &&
        tu.form == SPLIT_FORM_AUTO && tu.lane_per_cu == 0 && tu.lane_block == 0 && tu.wave_grid == 0)
        return eval_small(ctx, tours, bi.maxn, p, demand, S, ld, Q, cost, stream);
    // on the device the header ends before the tours
    const SumSlots ss = sum_slots(p.form, T, S);
    st = ensure_buffers(ctx, ctx->buf, T, bi.total_n, (int64_t)L.off_tours,
                        ss.slots * ss.stride * T, p.pair, false);
    if (st != SPLIT_OK) return st;
    st = ensure_host(ctx, (int64_t)L.bytes, T);
    if (st != SPLIT_OK) return st;

    // The header in a pinned slot, reused only after the call that read it completed.
    const int slot = ctx->stage;
    ctx->stage = (ctx->stage + 1) % kStages;
    if (ctx->stage_ev_used[slot]) HIP_TRY(ctx, hipEventSynchronize(ctx->stage_ev[slot]));
    stage_write(ctx->h_stage[slot], L, tours, tour_ptr, T, ctx->tuning.order);

    if (p.form == SPLIT_FORM_MASK && (__int128)ctx->buf.cap_pos * S > ctx->buf.cap_mask) {
        // one int16 window start per (position row, scenario)
        HIP_TRY(ctx, hipDeviceSynchronize());
        if (ctx->buf.d_mask) (void)hipFree(ctx->buf.d_mask);
        ctx->buf.d_mask = nullptr;
        ctx->buf.cap_mask = 0;
        const int64_t elems = ctx->buf.cap_pos * S;
        if (hipMalloc(&ctx->buf.d_mask, sizeof(int16_t) * (size_t)elems) != hipSuccess)
            return fail(ctx, SPLIT_E_NOMEM, "%s: the two-kernel form's %lld-byte mask matrix "
                        "could not be allocated", who, (long long)(2 * elems));
        ctx->buf.cap_mask = elems;
    }
    st = enqueue_kernels(ctx, ctx->inst, ctx->buf, L, ctx->h_stage[slot], ctx->h_stats, p, demand,
                         S, ld, Q, cost, ldc, stream, true);
    // recorded after a failed launch too: what was enqueued reads the slot
    const hipError_t ev = hipEventRecord(ctx->stage_ev[slot], stream);
    ctx->stage_ev_used[slot] = true;
    if (st != SPLIT_OK) return st;
    HIP_TRY(ctx, ev);
    ctx->last_ev = ctx->stage_ev[slot];
    ctx->have_call = true;
    ctx->last_S = S;
    ctx->last_T = T;
    ctx->last_parts = 0;
    return SPLIT_OK;
}

split_status check_tuning(split_ctx *ctx, const split_tuning &t)
{
    if (t.form != SPLIT_FORM_AUTO && t.form != SPLIT_FORM_LANE && t.form != SPLIT_FORM_WAVE &&
        t.form != SPLIT_FORM_MASK)
        return fail(ctx, SPLIT_E_INVAL, "tuning: unknown form %d", t.form);
    if (t.lane_per_cu < 0 || t.lane_per_cu > kMaxLanePerCu)
        return fail(ctx, SPLIT_E_INVAL, "tuning: lane_per_cu must be in 0..%d", kMaxLanePerCu);
    if (t.order != 0 && t.order != 1)
        return fail(ctx, SPLIT_E_INVAL, "tuning: order must be 0 or 1");
    if (t.wave_grid < 0) return fail(ctx, SPLIT_E_INVAL, "tuning: wave_grid must be >= 0");
    if (t.lane_block != 0 && t.lane_block != 8 && t.lane_block != 16)
        return fail(ctx, SPLIT_E_INVAL, "tuning: lane_block must be 0, 8 or 16");
    return SPLIT_OK;
}

}  // namespace

namespace splitgpu {

int ctx_device(const split_ctx *ctx) { return ctx->device; }

bool ctx_instance(const split_ctx *ctx, int32_t *N, int *kind, const int32_t **xy,
                  const int32_t **dist, int64_t *max_arc)
{
    if (ctx->inst.kind < 0) return false;
    *N = ctx->inst.N;
    *kind = ctx->inst.kind;
    *xy = ctx->inst.d_xy;
    *dist = ctx->inst.d_dist;
    *max_arc = ctx->inst.max_arc;
    return true;
}

void **ctx_topk_scratch(split_ctx *ctx) { return &ctx->topk; }

split_status ctx_fail(split_ctx *ctx, split_status st, const char *fmt, ...)
{
    if (ctx) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        ctx->err = buf;
    }
    return st;
}

}  // namespace splitgpu

extern "C" {

split_status split_ctx_create(int hip_device, split_ctx **out)
{
    if (!out) return SPLIT_E_INVAL;
    *out = nullptr;
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || hip_device < 0 || hip_device >= count)
        return SPLIT_E_INVAL;
    split_ctx *ctx = new (std::nothrow) split_ctx();
    if (!ctx) return SPLIT_E_NOMEM;
    ctx->device = hip_device;
    DeviceGuard g(hip_device);
    hipDeviceProp_t prop;
    if (!g.ok || hipGetDeviceProperties(&prop, hip_device) != hipSuccess) {
        split_ctx_destroy(ctx);
        return SPLIT_E_NOMEM;
    }
    ctx->cus = prop.multiProcessorCount;
    void *scr = nullptr;
    if (scratch_address(hip_device, &scr) != hipSuccess) {
        split_ctx_destroy(ctx);
        return SPLIT_E_HIP;
    }
    ctx->scratch = static_cast<unsigned char *>(scr);
    for (int k = 0; k < kStages; ++k) {
        if (hipEventCreateWithFlags(&ctx->stage_ev[k], hipEventDisableTiming) != hipSuccess) {
            split_ctx_destroy(ctx);
            return SPLIT_E_NOMEM;
        }
    }
    *out = ctx;
    return SPLIT_OK;
}

void split_ctx_destroy(split_ctx *ctx)
{
    if (!ctx) return;
    {
        DeviceGuard g(ctx->device);
        (void)hipDeviceSynchronize();
        free_instance(ctx->inst);
        free_buffers(ctx->buf);
        if (ctx->topk) (void)hipFree(ctx->topk);
        for (int k = 0; k < kStages; ++k) {
            if (ctx->h_stage[k]) (void)hipHostFree(ctx->h_stage[k]);
            if (ctx->stage_ev[k]) (void)hipEventDestroy(ctx->stage_ev[k]);
        }
        if (ctx->h_stats) (void)hipHostFree(ctx->h_stats);
        for (const TimedCall &c : ctx->timed)
            for (hipEvent_t e : {c.start, c.dp, c.end}) (void)hipEventDestroy(e);
    }
    delete ctx;
}

const char *split_last_error(const split_ctx *ctx)
{
    if (!ctx) return "null context";
    return ctx->err.c_str();
}

split_status split_instance_set_coords(split_ctx *ctx, int32_t N, const int32_t *xy)
{
    if (!ctx) return SPLIT_E_INVAL;
    if (!xy || N < 1 || N > SPLIT_MAX_N)
        return fail(ctx, SPLIT_E_INVAL, "set_coords: need xy != NULL and 1 <= N <= %d", SPLIT_MAX_N);
    int64_t lo[2] = {INT64_MAX, INT64_MAX}, hi[2] = {INT64_MIN, INT64_MIN};
    for (int64_t v = 0; v <= N; ++v)
        for (int c = 0; c < 2; ++c) {
            const int64_t x = xy[2 * v + c];
            if (x < -(1 << 20) || x > (1 << 20))
                return fail(ctx, SPLIT_E_INVAL, "set_coords: |coordinate| must be <= 2^20");
            lo[c] = x < lo[c] ? x : lo[c];
            hi[c] = x > hi[c] ? x : hi[c];
        }
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, SPLIT_E_HIP, "hipSetDevice failed");
    HIP_TRY(ctx, hipDeviceSynchronize());
    free_instance(ctx->inst);
    HIP_TRY(ctx, hipMalloc(&ctx->inst.d_xy, sizeof(int32_t) * 2 * ((size_t)N + 1)));
    HIP_TRY(ctx, hipMemcpy(ctx->inst.d_xy, xy, sizeof(int32_t) * 2 * ((size_t)N + 1),
                           hipMemcpyHostToDevice));
    const double dx = (double)(hi[0] - lo[0]), dy = (double)(hi[1] - lo[1]);
    ctx->inst.max_arc = (int64_t)ceil(sqrt(dx * dx + dy * dy)) + 1;  // bound on any rounded distance
    ctx->inst.N = N;
    ctx->inst.kind = 0;
    ctx->seen.assign((size_t)N + 1, 0);
    return SPLIT_OK;
}

split_status split_instance_set_dist(split_ctx *ctx, int32_t N, const int32_t *d)
{
    if (!ctx) return SPLIT_E_INVAL;
    if (!d || N < 1 || N > SPLIT_MAX_N)
        return fail(ctx, SPLIT_E_INVAL, "set_dist: need d != NULL and 1 <= N <= %d", SPLIT_MAX_N);
    const size_t V = (size_t)N + 1;
    int64_t mx = 0;
    for (size_t k = 0; k < V * V; ++k) {
        if (d[k] < 0) return fail(ctx, SPLIT_E_INVAL, "set_dist: negative entry at %zu", k);
        mx = d[k] > mx ? d[k] : mx;
    }
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, SPLIT_E_HIP, "hipSetDevice failed");
    HIP_TRY(ctx, hipDeviceSynchronize());
    free_instance(ctx->inst);
    HIP_TRY(ctx, hipMalloc(&ctx->inst.d_dist, sizeof(int32_t) * V * V));
    HIP_TRY(ctx, hipMemcpy(ctx->inst.d_dist, d, sizeof(int32_t) * V * V, hipMemcpyHostToDevice));
    ctx->inst.max_arc = mx;
    ctx->inst.N = N;
    ctx->inst.kind = 1;
    ctx->seen.assign(V, 0);
    return SPLIT_OK;
}

split_status split_eval(split_ctx *ctx, const int32_t *tour, int32_t n, const int16_t *demand,
                        int64_t S, int64_t ld, int32_t Q, int32_t *cost, split_stats *stats,
                        void *hip_stream)
{
    if (!ctx) return SPLIT_E_INVAL;
    const int64_t tour_ptr[2] = {0, n};
    split_status st = eval_batch(ctx, "split_eval", tour, tour_ptr, 1, demand, S, ld, Q, cost, S,
                                 (hipStream_t)hip_stream);
    if (st != SPLIT_OK) return st;
    if (stats) return split_stats_get(ctx, stats);
    return SPLIT_OK;
}

// The largest call (a tour of SPLIT_MAX_N positions) fits the scratch.
static_assert(((32 + 4 * (size_t)SPLIT_MAX_N + 255) & ~(size_t)255) +
                  ((8 * ((size_t)SPLIT_MAX_N + 1 + kRowPad) + 255) & ~(size_t)255) +
                  2 * ((4 * ((size_t)SPLIT_MAX_N + 1 + kRowPad) + 255) & ~(size_t)255) +
                  3 * 256 + kSlotStride * kMaxSlots <= kScratchBytes,
              "split_eval_noalloc: the scratch does not hold a maximal tour");

split_status split_eval_noalloc(split_ctx *ctx, const int32_t *tour, int32_t n,
                                const int16_t *demand, int64_t S, int64_t ld, int32_t Q,
                                int32_t *cost, split_stats *stats, void *hip_stream)
{
    if (!ctx) return SPLIT_E_INVAL;
    const char *who = "split_eval_noalloc";
    if (ctx->inst.kind < 0) return fail(ctx, SPLIT_E_INVAL, "%s: no instance set", who);
    if (!demand || !cost) return fail(ctx, SPLIT_E_INVAL, "%s: NULL pointer", who);
    split_status st = check_shape(ctx, who, S, ld, Q, S);
    if (st != SPLIT_OK) return st;
    const int64_t tour_ptr[2] = {0, n};
    BatchInfo bi;
    st = check_tours(ctx, who, ctx->inst, ctx->seen, tour, tour_ptr, 1, S, &bi);
    if (st != SPLIT_OK) return st;
    split_tuning tu = ctx->tuning;
    if (tu.form == SPLIT_FORM_MASK)
        return fail(ctx, SPLIT_E_INVAL, "%s: the two-kernel form needs a mask matrix in device "
                    "memory and is not available without allocation", who);

    // Carve the call's device buffers from the scratch, each 256-byte aligned.
    const StageLayout L = stage_layout(1, n);
    const int64_t pos = (int64_t)n + 1 + kRowPad;
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t o_stage = 0;
    const size_t o_rowoff = o_stage + up(L.bytes);
    const size_t o_rowoff32 = o_rowoff + up(sizeof(int64_t) * (size_t)pos);
    const size_t o_w = o_rowoff32 + up(sizeof(uint32_t) * (size_t)pos);
    const size_t o_stats = o_w + up(sizeof(int32_t) * (size_t)pos);
    const size_t o_ctl = o_stats + up(sizeof(DevStats));
    const size_t o_out = o_ctl + up(sizeof(BatchCtl));
    const size_t o_sums = o_out + up(sizeof(TourResult));
    const size_t need = o_sums + (size_t)kSlotStride * kMaxSlots;
    if (need > kScratchBytes)
        return fail(ctx, SPLIT_E_INVAL, "%s: a tour of %d positions needs %zu bytes of device "
                    "scratch, above the fixed %zu", who, n, need, kScratchBytes);

    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, SPLIT_E_HIP, "hipSetDevice failed");
    EvalBuffers b;  // views of the scratch; nothing here is owned or freed
    b.d_stage = reinterpret_cast<char *>(ctx->scratch + o_stage);
    b.cap_stage = (int64_t)L.bytes;
    b.d_rowoff = reinterpret_cast<int64_t *>(ctx->scratch + o_rowoff);
    b.d_rowoff32 = reinterpret_cast<uint32_t *>(ctx->scratch + o_rowoff32);
    b.d_w = reinterpret_cast<int32_t *>(ctx->scratch + o_w);
    b.cap_pos = pos;
    b.d_stats = reinterpret_cast<DevStats *>(ctx->scratch + o_stats);
    b.cap_T = 1;
    b.d_ctl = reinterpret_cast<BatchCtl *>(ctx->scratch + o_ctl);
    b.d_sums = reinterpret_cast<char *>(ctx->scratch + o_sums);
    b.cap_sums = (int64_t)kSlotStride * kMaxSlots;
    TourResult *d_out = reinterpret_cast<TourResult *>(ctx->scratch + o_out);

    // The staged header of a batch of one: T, tptr, order, then the tour itself, copied from
    // pageable host memory (the runtime stages it before the call returns).
    const hipStream_t stream = (hipStream_t)hip_stream;
    const int64_t head[3] = {1, 0, n};
    const int32_t order0 = 0;
    HIP_TRY(ctx, hipMemcpyAsync(b.d_stage, head, sizeof head, hipMemcpyHostToDevice, stream));
    HIP_TRY(ctx, hipMemcpyAsync(b.d_stage + L.off_order, &order0, sizeof order0,
                                hipMemcpyHostToDevice, stream));
    HIP_TRY(ctx, hipMemcpyAsync(b.d_stage + L.off_tours, tour, sizeof(int32_t) * (size_t)n,
                                hipMemcpyHostToDevice, stream));
    Plan p = make_plan(ctx, tu, S, ld, Q, 1, bi.maxn, bi.max_id, true, ctx->inst.max_arc);
    p.pair = false;  // the scratch does not hold the mirrored arrays of a maximal tour
    // the prep kernel zeroes the sums and the counters of every call
    st = enqueue_kernels(ctx, ctx->inst, b, L, b.d_stage, d_out, p, demand, S, ld, Q, cost, S,
                         stream, false);
    if (st != SPLIT_OK) return st;
    if (!stats) return SPLIT_OK;
    TourResult d;
    HIP_TRY(ctx, hipMemcpyAsync(&d, d_out, sizeof d, hipMemcpyDeviceToHost, stream));
    HIP_TRY(ctx, hipStreamSynchronize(stream));
    fill_stats(d, S, stats);
    if (d.err_demand)
        return fail(ctx, SPLIT_E_DEMAND, "%s: a scenario has a demand q < 0 or q > Q on the tour",
                    who);
    return SPLIT_OK;
}

split_status split_eval_batch(split_ctx *ctx, const int32_t *tours, const int64_t *tour_ptr,
                              int32_t T, const int16_t *demand, int64_t S, int64_t ld, int32_t Q,
                              int32_t *cost, int64_t ldc, split_stats *stats,
                              int32_t *tour_status, void *hip_stream)
{
    if (!ctx) return SPLIT_E_INVAL;
    split_status st = eval_batch(ctx, "split_eval_batch", tours, tour_ptr, T, demand, S, ld, Q,
                                 cost, ldc, (hipStream_t)hip_stream);
    if (st != SPLIT_OK) return st;
    if (stats || tour_status) return split_batch_stats_get(ctx, stats, tour_status);
    return SPLIT_OK;
}

split_status split_batch_stats_get(split_ctx *ctx, split_stats *stats, int32_t *tour_status)
{
    if (!ctx) return SPLIT_E_INVAL;
    if (!ctx->have_call) return fail(ctx, SPLIT_E_INVAL, "split_batch_stats_get: no evaluation yet");
    DeviceGuard g(ctx->device);
    HIP_TRY(ctx, hipEventSynchronize(ctx->last_ev));
    return report(ctx, last_results(ctx), ctx->last_T, ctx->last_S, stats, tour_status);
}

split_status split_stats_get(split_ctx *ctx, split_stats *stats)
{
    if (!ctx) return SPLIT_E_INVAL;
    if (!stats) return fail(ctx, SPLIT_E_INVAL, "split_stats_get: NULL stats");
    if (!ctx->have_call) return fail(ctx, SPLIT_E_INVAL, "split_stats_get: no evaluation yet");
    DeviceGuard g(ctx->device);
    HIP_TRY(ctx, hipEventSynchronize(ctx->last_ev));
    const TourResult d = last_results(ctx)[0];
    fill_stats(d, ctx->last_S, stats);
    if (d.err_demand)
        return fail(ctx, SPLIT_E_DEMAND,
                    "split_eval: a scenario has a demand q < 0 or q > Q on the tour");
    return SPLIT_OK;
}

split_status split_set_form(split_ctx *ctx, int form)
{
    if (!ctx) return SPLIT_E_INVAL;
    if (form != SPLIT_FORM_AUTO && form != SPLIT_FORM_LANE && form != SPLIT_FORM_WAVE &&
        form != SPLIT_FORM_MASK)
        return fail(ctx, SPLIT_E_INVAL, "split_set_form: unknown form %d", form);
    ctx->tuning.form = form;
    return SPLIT_OK;
}

split_status split_tuning_set(split_ctx *ctx, const split_tuning *tuning)
{
    if (!ctx) return SPLIT_E_INVAL;
    if (!tuning) return fail(ctx, SPLIT_E_INVAL, "split_tuning_set: NULL tuning");
    split_status st = check_tuning(ctx, *tuning);
    if (st != SPLIT_OK) return st;
    ctx->tuning = *tuning;
    return SPLIT_OK;
}

split_status split_tuning_get(split_ctx *ctx, split_tuning *tuning)
{
    if (!ctx) return SPLIT_E_INVAL;
    if (!tuning) return fail(ctx, SPLIT_E_INVAL, "split_tuning_get: NULL tuning");
    *tuning = ctx->tuning;
    return SPLIT_OK;
}

split_status split_autotune(split_ctx *ctx, const int32_t *tours, const int64_t *tour_ptr,
                            int32_t T, const int16_t *demand, int64_t S, int64_t ld, int32_t Q,
                            int32_t *cost, int64_t ldc, int32_t reps, void *hip_stream,
                            split_tuning *best, double *best_ms)
{
    if (!ctx) return SPLIT_E_INVAL;
    if (reps < 1 || reps > 1000)
        return fail(ctx, SPLIT_E_INVAL, "split_autotune: need 1 <= reps <= 1000");
    if (ctx->inst.kind < 0) return fail(ctx, SPLIT_E_INVAL, "split_autotune: no instance set");
    if (!demand || !cost) return fail(ctx, SPLIT_E_INVAL, "split_autotune: NULL pointer");
    split_status st = check_shape(ctx, "split_autotune", S, ld, Q, ldc);
    if (st != SPLIT_OK) return st;
    BatchInfo bi;
    st = check_tours(ctx, "split_autotune", ctx->inst, ctx->seen, tours, tour_ptr, T, S, &bi);
    if (st != SPLIT_OK) return st;
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, SPLIT_E_HIP, "hipSetDevice failed");
    hipStream_t stream = (hipStream_t)hip_stream;

    const split_tuning saved = ctx->tuning;
    const bool saved_timing = ctx->timing;
    ctx->timing = false;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    auto finish = [&](split_status s) {
        ctx->timing = saved_timing;
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
        if (s != SPLIT_OK) ctx->tuning = saved;
        return s;
    };
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
        return finish(fail(ctx, SPLIT_E_HIP, "split_autotune: hipEventCreate failed"));

    // mean milliseconds of one whole evaluation (upload, kernels, statistics) under tuning c,
    // on the first s_eval scenarios
    auto measure = [&](const split_tuning &c, int64_t s_eval, double *ms) -> split_status {
        ctx->tuning = c;
        split_status s = eval_batch(ctx, "split_autotune", tours, tour_ptr, T, demand, s_eval, ld,
                                    Q, cost, ldc, stream);  // warm-up
        if (s != SPLIT_OK) return s;
        s = split_batch_stats_get(ctx, nullptr, nullptr);
        if (s != SPLIT_OK) return s;
        if (hipEventRecord(e0, stream) != hipSuccess)
            return fail(ctx, SPLIT_E_HIP, "split_autotune: hipEventRecord failed");
        for (int r = 0; r < reps; ++r) {
            s = eval_batch(ctx, "split_autotune", tours, tour_ptr, T, demand, s_eval, ld, Q, cost,
                           ldc, stream);
            if (s != SPLIT_OK) return s;
        }
        if (hipEventRecord(e1, stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess)
            return fail(ctx, SPLIT_E_HIP, "split_autotune: timing events failed");
        float el = 0.f;
        if (hipEventElapsedTime(&el, e0, e1) != hipSuccess)
            return fail(ctx, SPLIT_E_HIP, "split_autotune: hipEventElapsedTime failed");
        *ms = (double)el / reps;
        return split_batch_stats_get(ctx, nullptr, nullptr);
    };

    // scenarios left to the wave kernel, over the first s_eval scenarios, under tuning c
    std::vector<split_stats> fb_stats((size_t)T);
    auto fallbacks = [&](const split_tuning &c, int64_t s_eval, int64_t *n) -> split_status {
        ctx->tuning = c;
        split_status s = eval_batch(ctx, "split_autotune", tours, tour_ptr, T, demand, s_eval, ld,
                                    Q, cost, ldc, stream);
        if (s != SPLIT_OK) return s;
        s = split_batch_stats_get(ctx, fb_stats.data(), nullptr);
        if (s != SPLIT_OK) return s;
        *n = 0;
        for (const split_stats &x : fb_stats) *n += x.n_fallback;
        return SPLIT_OK;
    };

    // The library's own choice (block length by window, one launch for short tours) is one of the
    // candidates. Where an explicit one comes within kTie of it, the explicit one is taken: that much
    // is noise, and it spares later calls the look at the windows.
    constexpr double kTie = 1.04;
    const split_tuning own = {SPLIT_FORM_AUTO, 0, 0, 0, 0};
    double own_ms = 0.0;
    st = measure(own, S, &own_ms);
    if (st != SPLIT_OK) return finish(st);
    split_tuning win = own;
    double win_ms = 1e300;
    const Plan lane_probe = make_plan(ctx, split_tuning{SPLIT_FORM_LANE, 0, 0, 0, 0}, S, ld, Q,
                                      T, bi.maxn, bi.max_id, bi.minn == bi.maxn, ctx->inst.max_arc);
    if (lane_probe.form == SPLIT_FORM_LANE) {
        // the block length first (it follows the window lengths, so the demand law), then the
        // grid and the order with that block length. 8-state blocks leave windows longer than
        // about 24 positions to the tail kernel, which costs far more than any block saves: a
        // probe on the first scenarios drops them when they leave more scenarios there.
        const int64_t s_fb = S < 4096 ? S : 4096;
        int64_t fb16 = 0, fb8 = 0;
        st = fallbacks(split_tuning{SPLIT_FORM_LANE, 0, 0, 0, 16}, s_fb, &fb16);
        if (st != SPLIT_OK) return finish(st);
        st = fallbacks(split_tuning{SPLIT_FORM_LANE, 0, 0, 0, 8}, s_fb, &fb8);
        if (st != SPLIT_OK) return finish(st);
        int32_t block = 16;
        for (int32_t lb : {16, 8, 0}) {
            if (lb == 8 && fb8 > fb16) continue;
            const split_tuning c = {SPLIT_FORM_LANE, 0, 0, 0, lb};
            double ms = 0.0;
            st = measure(c, S, &ms);
            if (st != SPLIT_OK) return finish(st);
            if (lb != 0 ? ms < win_ms : kTie * ms < win_ms) {
                win_ms = ms;
                win = c;
                block = lb;
            }
        }
        const int32_t per_cu[] = {0, 8, 4, 2};
        for (int32_t pc : per_cu)
            for (int32_t order = 0; order < 2; ++order) {
                if (T == 1 && order == 1) continue;  // one tour: the order is moot
                if (pc == 0 && order == 0) continue;  // timed above
                const split_tuning c = {SPLIT_FORM_LANE, pc, order, 0, block};
                double ms = 0.0;
                st = measure(c, S, &ms);
                if (st != SPLIT_OK) return finish(st);
                if (ms < win_ms) {
                    win_ms = ms;
                    win = c;
                }
            }
    }
    // The wave form costs about S times one scenario's evaluation: try it in full only when a
    // run on at most 256 scenarios, scaled to S, is within 1.5x of the best so far.
    const int64_t s_probe = S < 256 ? S : 256;
    double probe_ms = 0.0;
    st = measure(split_tuning{SPLIT_FORM_WAVE, 0, 0, 0, 0}, s_probe, &probe_ms);
    if (st != SPLIT_OK) return finish(st);
    if (probe_ms * ((double)S / (double)s_probe) < 1.5 * win_ms) {
        const int32_t grids[] = {0, ctx->cus * 8};
        for (int32_t wg : grids) {
            const split_tuning c = {SPLIT_FORM_WAVE, 0, 0, wg, 0};
            double ms = 0.0;
            st = measure(c, S, &ms);
            if (st != SPLIT_OK) return finish(st);
            if (ms < win_ms) {
                win_ms = ms;
                win = c;
            }
        }
    }
    if (win_ms > own_ms) {
        // once more, side by side, before the library's own choice is taken
        double ms = 0.0;
        st = measure(win, S, &ms);
        if (st != SPLIT_OK) return finish(st);
        win_ms = ms < win_ms ? ms : win_ms;
        st = measure(own, S, &ms);
        if (st != SPLIT_OK) return finish(st);
        own_ms = ms < own_ms ? ms : own_ms;
        if (win_ms > kTie * own_ms) {
            win = own;
            win_ms = own_ms;
        }
    }
    // leave the context's latest evaluation the full one under the chosen tuning
    ctx->tuning = win;
    st = eval_batch(ctx, "split_autotune", tours, tour_ptr, T, demand, S, ld, Q, cost, ldc, stream);
    if (st != SPLIT_OK) return finish(st);
    st = split_batch_stats_get(ctx, nullptr, nullptr);
    if (st != SPLIT_OK) return finish(st);
    if (best) *best = win;
    if (best_ms) *best_ms = win_ms;
    return finish(SPLIT_OK);
}

split_status split_timing_enable(split_ctx *ctx, int enable)
{
    if (!ctx) return SPLIT_E_INVAL;
    ctx->timing = enable != 0;
    return SPLIT_OK;
}

split_status split_timing_get(split_ctx *ctx, double *ms_total, int64_t *launches,
                              const char **kernel_name)
{
    if (!ctx) return SPLIT_E_INVAL;
    DeviceGuard g(ctx->device);
    split_status st = collect_timing(ctx);
    if (st != SPLIT_OK) return st;
    if (ms_total) *ms_total = ctx->ms_acc;
    if (launches) *launches = ctx->launches;
    if (kernel_name) *kernel_name = ctx->tname;
    return SPLIT_OK;
}

split_status split_timing_reset(split_ctx *ctx)
{
    if (!ctx) return SPLIT_E_INVAL;
    DeviceGuard g(ctx->device);
    split_status st = collect_timing(ctx);
    ctx->ms_acc = 0.0;
    ctx->launches = 0;
    ctx->ms_samples.clear();
    return st;
}

split_status split_timing_samples(split_ctx *ctx, float *ms, int64_t cap, int64_t *count)
{
    if (!ctx) return SPLIT_E_INVAL;
    if (cap < 0 || (cap > 0 && !ms))
        return fail(ctx, SPLIT_E_INVAL, "split_timing_samples: need cap >= 0 and ms for cap > 0");
    DeviceGuard g(ctx->device);
    split_status st = collect_timing(ctx);
    if (st != SPLIT_OK) return st;
    const int64_t n = (int64_t)ctx->ms_samples.size();
    for (int64_t k = 0; k < n && k < cap; ++k) ms[k] = ctx->ms_samples[(size_t)k];
    if (count) *count = n;
    return SPLIT_OK;
}

// ------------------------------------------------------------------------- graphs

void split_graph_destroy(split_graph *gr)
{
    if (!gr) return;
    {
        DeviceGuard g(gr->ctx->device);
        for (int k = 0; k < kGraphSlots; ++k)
            if (gr->used[k]) (void)hipEventSynchronize(gr->done[k]);
        for (int k = 0; k < kGraphSlots; ++k) {
            for (int pair = 0; pair < 2; ++pair) {
                if (gr->exec[k][pair]) (void)hipGraphExecDestroy(gr->exec[k][pair]);
                if (gr->graph[k][pair]) (void)hipGraphDestroy(gr->graph[k][pair]);
            }
            if (gr->done[k]) (void)hipEventDestroy(gr->done[k]);
            if (gr->h_stage[k]) (void)hipHostFree(gr->h_stage[k]);
            if (gr->h_stats[k]) (void)hipHostFree(gr->h_stats[k]);
        }
        if (gr->cap_stream) (void)hipStreamDestroy(gr->cap_stream);
        free_buffers(gr->buf);
        free_instance(gr->inst);
    }
    delete gr;
}

split_status split_graph_create(split_ctx *ctx, int32_t max_T, int64_t max_total_n,
                                const int16_t *demand, int64_t S, int64_t ld, int32_t Q,
                                int32_t *cost, int64_t ldc, split_graph **out)
{
    if (!ctx) return SPLIT_E_INVAL;
    if (!out) return fail(ctx, SPLIT_E_INVAL, "split_graph_create: NULL out");
    *out = nullptr;
    if (ctx->inst.kind < 0) return fail(ctx, SPLIT_E_INVAL, "split_graph_create: no instance set");
    if (!demand || !cost) return fail(ctx, SPLIT_E_INVAL, "split_graph_create: NULL pointer");
    split_status st = check_shape(ctx, "split_graph_create", S, ld, Q, ldc);
    if (st != SPLIT_OK) return st;
    if (max_T < 1 || max_total_n < max_T || max_total_n > (int64_t)max_T * ctx->inst.N)
        return fail(ctx, SPLIT_E_INVAL, "split_graph_create: need 1 <= max_T <= max_total_n <= "
                    "max_T * N");
    if ((__int128)((S + 63) / 64) * max_T >= ((__int128)1 << 31))
        return fail(ctx, SPLIT_E_INVAL, "split_graph_create: max_T * ceil(S / 64) must be below "
                    "2^31");
    const int32_t N = ctx->inst.N;
    if ((__int128)4 * ((__int128)N + 1) * ctx->inst.max_arc >= ((__int128)1 << 31))
        return fail(ctx, SPLIT_E_RANGE, "split_graph_create: 4*(N+1)*max_arc exceeds 2^31");
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, SPLIT_E_HIP, "hipSetDevice failed");

    split_graph *gr = new (std::nothrow) split_graph();
    if (!gr) return fail(ctx, SPLIT_E_NOMEM, "split_graph_create: out of host memory");
    gr->ctx = ctx;
    bool capturing = false;
    auto bail = [&](split_status s) {
        if (capturing) {
            hipGraph_t dropped = nullptr;
            (void)hipStreamEndCapture(gr->cap_stream, &dropped);
            if (dropped) (void)hipGraphDestroy(dropped);
        }
        split_graph_destroy(gr);
        return s;
    };
    // the graph's own copy of the instance: later changes to the context's do not reach it
    gr->inst.N = N;
    gr->inst.kind = ctx->inst.kind;
    gr->inst.max_arc = ctx->inst.max_arc;
    const size_t V = (size_t)N + 1;
    if (ctx->inst.kind == 0) {
        if (hipMalloc(&gr->inst.d_xy, sizeof(int32_t) * 2 * V) != hipSuccess ||
            hipMemcpy(gr->inst.d_xy, ctx->inst.d_xy, sizeof(int32_t) * 2 * V,
                      hipMemcpyDeviceToDevice) != hipSuccess)
            return bail(fail(ctx, SPLIT_E_NOMEM, "split_graph_create: instance copy failed"));
    } else {
        if (hipMalloc(&gr->inst.d_dist, sizeof(int32_t) * V * V) != hipSuccess ||
            hipMemcpy(gr->inst.d_dist, ctx->inst.d_dist, sizeof(int32_t) * V * V,
                      hipMemcpyDeviceToDevice) != hipSuccess)
            return bail(fail(ctx, SPLIT_E_NOMEM, "split_graph_create: instance copy failed"));
    }
    gr->seen.assign(V, 0);
    gr->max_T = max_T;
    gr->max_total_n = max_total_n;
    gr->S = S;
    gr->ld = ld;
    gr->ldc = ldc;
    gr->Q = Q;
    gr->order = ctx->tuning.order;
    gr->layout = stage_layout(max_T, max_total_n);
    // any tour of the instance: lengths up to N, ids up to N
    // the tours of a replay are known only then: a fixed item stride only for one tour
    gr->plan = make_plan(ctx, ctx->tuning, S, ld, Q, max_T, N, N, max_T == 1,
                         gr->inst.max_arc);
    const SumSlots ss = sum_slots(gr->plan.form, max_T, S);
    st = ensure_buffers(ctx, gr->buf, max_T, max_total_n, (int64_t)gr->layout.off_tours,
                        ss.slots * ss.stride * max_T, gr->plan.pair, true);
    if (st != SPLIT_OK) return bail(st);
    if (gr->plan.form == SPLIT_FORM_MASK)
        return bail(fail(ctx, SPLIT_E_INVAL, "split_graph_create: the two-kernel form is an "
                         "ablation and is not captured"));
    if (hipStreamCreateWithFlags(&gr->cap_stream, hipStreamNonBlocking) != hipSuccess) {
        gr->cap_stream = nullptr;
        return bail(fail(ctx, SPLIT_E_HIP, "split_graph_create: hipStreamCreate failed"));
    }
    for (int k = 0; k < kGraphSlots; ++k) {
        if (!pinned(&gr->h_stage[k], gr->layout.bytes) ||
            !pinned(&gr->h_stats[k], sizeof(TourResult) * (size_t)max_T))
            return bail(fail(ctx, SPLIT_E_NOMEM, "split_graph_create: pinned allocation failed"));
        memset(gr->h_stage[k], 0, gr->layout.bytes);
        if (hipEventCreateWithFlags(&gr->done[k], hipEventDisableTiming) != hipSuccess)
            return bail(fail(ctx, SPLIT_E_HIP, "split_graph_create: hipEventCreate failed"));
    }
    // One graph per host slot: the kernels read the slot's header and report to its results. Where
    // the instance's tours may run in the pair kernel, one with it and one without: which is faster
    // follows the tours of a replay (S = 10,000, graph of one tour over 1000 customers: 8 customers
    // 62 us with it, 47 without; 100 customers 64 and 56; eight tours of 8 to 300 over 5,000
    // scenarios 111 and 87).
    for (int v = 0; v < kGraphSlots * 2; ++v) {
        const int k = v / 2, pair = v % 2;
        if (pair && !gr->plan.pair) continue;
        Plan plan = gr->plan;
        plan.pair = pair != 0;
        if (hipStreamBeginCapture(gr->cap_stream, hipStreamCaptureModeThreadLocal) != hipSuccess)
            return bail(fail(ctx, SPLIT_E_HIP, "split_graph_create: hipStreamBeginCapture failed"));
        capturing = true;
        st = enqueue_kernels(ctx, gr->inst, gr->buf, gr->layout, gr->h_stage[k], gr->h_stats[k],
                             plan, demand, S, ld, Q, cost, ldc, gr->cap_stream, false);
        if (st != SPLIT_OK) return bail(st);
        hipGraph_t graph = nullptr;
        const hipError_t e = hipStreamEndCapture(gr->cap_stream, &graph);
        capturing = false;
        gr->graph[k][pair] = graph;
        if (e != hipSuccess || !graph)
            return bail(hip_fail(ctx, e, "split_graph_create: hipStreamEndCapture"));
        if (hipGraphInstantiate(&gr->exec[k][pair], graph, nullptr, nullptr, 0) != hipSuccess) {
            gr->exec[k][pair] = nullptr;
            return bail(fail(ctx, SPLIT_E_HIP, "split_graph_create: hipGraphInstantiate failed"));
        }
    }
    *out = gr;
    return SPLIT_OK;
}

split_status split_graph_launch(split_graph *gr, const int32_t *tours, const int64_t *tour_ptr,
                                int32_t T, void *hip_stream)
{
    if (!gr) return SPLIT_E_INVAL;
    split_ctx *ctx = gr->ctx;
    if (T > gr->max_T)
        return fail(ctx, SPLIT_E_INVAL, "split_graph_launch: T = %d exceeds the graph's %d", T,
                    gr->max_T);
    BatchInfo bi;
    split_status st = check_tours(ctx, "split_graph_launch", gr->inst, gr->seen, tours, tour_ptr,
                                  T, gr->S, &bi);
    if (st != SPLIT_OK) return st;
    if (bi.total_n > gr->max_total_n)
        return fail(ctx, SPLIT_E_INVAL, "split_graph_launch: %lld positions exceed the graph's "
                    "%lld", (long long)bi.total_n, (long long)gr->max_total_n);
    DeviceGuard g(ctx->device);
    if (!g.ok) return fail(ctx, SPLIT_E_HIP, "hipSetDevice failed");
    const int k = gr->next;
    if (gr->used[k]) HIP_TRY(ctx, hipEventSynchronize(gr->done[k]));
    stage_write(gr->h_stage[k], gr->layout, tours, tour_ptr, T, gr->order);
    hipStream_t stream = (hipStream_t)hip_stream;
    const int pair = gr->plan.pair && bi.maxn >= pair_min_n(ctx, (gr->S + 63) / 64 * gr->max_T) ? 1 : 0;
    HIP_TRY(ctx, hipGraphLaunch(gr->exec[k][pair], stream));
    HIP_TRY(ctx, hipEventRecord(gr->done[k], stream));
    gr->used[k] = true;
    gr->last = k;
    gr->last_T = T;
    gr->next = (k + 1) % kGraphSlots;
    return SPLIT_OK;
}

split_status split_graph_stats(split_graph *gr, split_stats *stats, int32_t *tour_status)
{
    if (!gr) return SPLIT_E_INVAL;
    split_ctx *ctx = gr->ctx;
    if (gr->last < 0) return fail(ctx, SPLIT_E_INVAL, "split_graph_stats: no launch yet");
    DeviceGuard g(ctx->device);
    HIP_TRY(ctx, hipEventSynchronize(gr->done[gr->last]));
    return report(ctx, gr->h_stats[gr->last], gr->last_T, gr->S, stats, tour_status);
}

}  // extern "C"
