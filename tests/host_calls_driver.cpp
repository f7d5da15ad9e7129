// The library's host code over a stand-in for the HIP runtime and for its own kernels, on the CPU:
// memory is host memory, a launch is a line in a trace and an advance of a simulated clock, a
// captured graph replays its lines, and any allocation or launch can be made to fail. What a call
// launches, allocates, waits for and reports can be checked without a GPU, and so can its error
// paths. Usage: host_calls_driver SCENARIO; exit code 0 when the scenario holds.
#include <hip/hip_runtime.h>

#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

#include "../include/split.h"
#include "../include/split_nn.h"
#include "../include/split_search.h"
#include "../paper_2511_18022_amd/csrc/nn_internal.h"
#include "../paper_2511_18022_amd/csrc/split_internal.h"

using namespace splitgpu;

namespace {

std::vector<std::string> trace;          // launches and copies, in order
std::map<std::string, double> cost_us;   // simulated duration of a launch
std::map<std::string, int> fail_launch;  // launches of this name that fail from now on
int fail_malloc = 0;                     // the fail_malloc-th device allocation from now fails
int mallocs = 0, syncs = 0;
size_t malloc_bytes = 0;
int prep_threads = 0;
double clock_us = 0.0;
std::vector<std::string> *capture = nullptr;

hipError_t launched(const char *name)
{
    if (fail_launch[name] > 0) {
        --fail_launch[name];
        return hipErrorLaunchFailure;
    }
    if (capture) {
        capture->push_back(name);
        return hipSuccess;
    }
    trace.push_back(name);
    clock_us += cost_us.count(name) ? cost_us[name] : 1.0;
    return hipSuccess;
}

int count(const char *name)
{
    int k = 0;
    for (const std::string &s : trace) k += s == name;
    return k;
}

int failures = 0;
#define CHECK(cond)                                                             \
    do {                                                                        \
        if (!(cond)) {                                                          \
            ++failures;                                                         \
            printf("line %d: %s does not hold\n", __LINE__, #cond);             \
        }                                                                       \
    } while (0)

}  // namespace

// ------------------------------------------------------------------------- HIP runtime

struct ihipEvent_t {
    double at = 0.0;
};
struct ihipGraph {
    std::vector<std::string> lines;
};

extern "C" {
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "a failure that the test asked for"; }
hipError_t hipMalloc(void **p, size_t n)
{
    ++mallocs;
    malloc_bytes += n;
    if (fail_malloc > 0 && --fail_malloc == 0) {
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    *p = calloc(n ? n : 1, 1);
    return hipSuccess;
}
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(n ? n : 1, 1); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipDeviceSynchronize() { ++syncs; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    memcpy(d, s, n);
    return launched("copy");
}
hipError_t hipMemset(void *d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = new ihipEvent_t; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = new ihipEvent_t; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { e->at = clock_us; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b)
{
    *ms = (float)((b->at - a->at) * 1e-3);
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode)
{
    capture = new std::vector<std::string>;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    *g = new ihipGraph{*capture};
    delete capture;
    capture = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t g, hipGraphNode_t *, char *, size_t)
{
    *e = reinterpret_cast<hipGraphExec_t>(new ihipGraph{g->lines});
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t)
{
    for (const std::string &s : reinterpret_cast<ihipGraph *>(e)->lines)
        if (launched(s.c_str()) != hipSuccess) return hipErrorLaunchFailure;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete g; return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { delete reinterpret_cast<ihipGraph *>(e); return hipSuccess; }
}

// ------------------------------------------------------------------------- kernels

namespace splitgpu {

hipError_t launch_prep(const PrepArgs &a, hipStream_t)
{
    prep_threads = a.threads;
    return launched("prep");
}
hipError_t launch_lane(const EvalArgs &a, hipStream_t)
{
    return launched(a.lane_block == 0 ? "lane0" : a.lane_block == 8 ? "lane8" : "lane16");
}
hipError_t launch_pair(const EvalArgs &a, hipStream_t)
{
    return launched(a.lane_block == 0 ? "pair0" : "pair16");
}
hipError_t launch_wave_all(const EvalArgs &, hipStream_t) { return launched("wave"); }
hipError_t launch_small(const SmallArgs &a, hipStream_t)
{
    for (int64_t k = 0; k < (a.S + kSmallPer - 1) / kSmallPer; ++k) a.out[k] = TourResult{};
    return launched("small");
}
hipError_t launch_tail(const EvalArgs &, hipStream_t) { return launched("tail"); }
hipError_t launch_mask(const EvalArgs &, int16_t *, long long, hipStream_t) { return launched("mask"); }
hipError_t launch_masked_dp(const EvalArgs &, const int16_t *, long long, hipStream_t)
{
    return launched("masked_dp");
}
const char *lane_kernel_name() { return "split_lane_kernel"; }
const char *pair_kernel_name() { return "split_pair_kernel"; }
const char *tail_kernel_name() { return "split_tail_kernel"; }
const char *wave_kernel_name() { return "split_wave_kernel"; }
const char *mask_kernel_name() { return "split_mask_kernel+split_masked_dp_kernel"; }
hipError_t scratch_address(int, void **p)
{
    static std::vector<char> s(1 << 20);
    *p = s.data();
    return hipSuccess;
}

static void ids(const int32_t *tours, long long n, int32_t N, int32_t *err)
{
    for (long long k = 0; k < n; ++k)
        if (tours[k] < 1 || tours[k] > N) *err = 1;
}
hipError_t nn_launch_dstats(const int16_t *, int64_t, int64_t, int32_t, double *, hipStream_t)
{
    return launched("dstats");
}
hipError_t nn_launch_features(const NnInstance &in, const int32_t *tours, int32_t T, int32_t n,
                              const double *, int32_t, double, const uint16_t *, uint16_t *, bool,
                              int32_t *err, hipStream_t)
{
    ids(tours, (long long)T * n, in.N, err);
    return launched("features");
}
hipError_t nn_launch_customers(const NnInstance &in, const double *, int32_t, double,
                               uint16_t *table, hipStream_t)
{
    CHECK(table != nullptr);
    if (table) memset(table, 0, sizeof(uint16_t) * kNnFeatures * (size_t)in.N);
    return launched("customers");
}
hipError_t nn_launch_conv_back(const uint16_t *, const uint16_t *, const uint16_t *, uint16_t *,
                               int32_t, int32_t, hipStream_t)
{
    return launched("conv_back");
}
int32_t nn_pool_groups(int32_t n) { return (n + 63) / 64; }
hipError_t nn_launch_fwd_fused(const uint16_t *, const NnWeights &, const float *, int32_t, int32_t,
                               float *, const NnHidden *, hipStream_t)
{
    return launched("fwd");
}
hipError_t nn_launch_head_pool(const float *, int32_t, int32_t, const float *, float *, float *,
                               float *, float *, double, double, int32_t *err, int32_t *host_err,
                               hipStream_t)
{
    const hipError_t e = launched("head");
    if (e == hipSuccess && host_err) {
        *host_err = *err;
        *err = 0;
    }
    return e;
}
hipError_t nn_launch_head_bwd(const float *, int32_t, int32_t, const float *, const float *,
                              const float *, const float *, double, double, float *, float *,
                              float *, float *, float *, const uint16_t *, uint16_t *, float *,
                              hipStream_t)
{
    return launched("head_bwd");
}
int32_t nn_wgrad_chunks(int32_t T, int32_t n, int32_t chunk)
{
    return (int32_t)(((int64_t)T * (n + 4) + chunk - 1) / chunk);
}
hipError_t nn_launch_wgrad(int, const uint16_t *, const uint16_t *, int32_t, int32_t, int32_t,
                           int32_t, float *, float *, float *, int, int, hipStream_t)
{
    return launched("wgrad");
}
hipError_t nn_launch_adam(float *, float *, float *, const float *, float, float, float,
                          hipStream_t)
{
    return launched("adam");
}
hipError_t nn_launch_pack(const float *, const NnWeights &, hipStream_t) { return launched("pack"); }
hipError_t nn_launch_gather(const int32_t *src, const float *, const int32_t *idx, int32_t B,
                            int32_t n, int32_t *dst, float *, hipStream_t)
{
    for (int32_t b = 0; b < B; ++b) memcpy(dst + (int64_t)b * n, src + (int64_t)idx[b] * n, sizeof(int32_t) * n);
    return launched("gather");
}
hipError_t nn_launch_moves(const int32_t *, const int32_t *, int32_t, int32_t, int32_t *, hipStream_t)
{
    return launched("moves");
}
hipError_t nn_launch_check_ids(const int32_t *t, long long n, int32_t N, int32_t *err, hipStream_t)
{
    ids(t, n, N, err);
    return launched("check_ids");
}
hipError_t nn_launch_topk(const float *, long long, long long K, NnTopk *, int32_t *idx, hipStream_t)
{
    for (long long k = 0; k < K; ++k) idx[k] = (int32_t)k;
    return launched("topk");
}

}  // namespace splitgpu

// ------------------------------------------------------------------------- scenarios

namespace {

struct Ctx {
    split_ctx *c = nullptr;
    explicit Ctx(int N, int grid = 1000)
    {
        CHECK(split_ctx_create(0, &c) == SPLIT_OK);
        coords(N, grid);
    }
    ~Ctx() { split_ctx_destroy(c); }
    void coords(int N, int grid = 1000)
    {
        std::vector<int32_t> xy;
        for (int v = 0; v <= 2 * N + 1; ++v) xy.push_back((int32_t)((v * 7919LL) % grid));
        CHECK(split_instance_set_coords(c, N, xy.data()) == SPLIT_OK);
    }
};

// The surrogate with customers 1..N known.
struct Nn {
    Ctx ctx;
    split_nn *nn = nullptr;
    std::vector<int16_t> dem;
    explicit Nn(int N) : ctx(N), dem((size_t)4096 * 4, 5)
    {
        CHECK(split_nn_create(ctx.c, 1, 1000.0, &nn) == SPLIT_OK);
        CHECK(scenarios() == SPLIT_OK);
    }
    ~Nn() { split_nn_destroy(nn); }
    split_status scenarios() { return split_nn_set_scenarios(nn, dem.data(), 4, 4, 100); }
};

// A pass that fails between the feature kernel and the head keeps its flag of bad ids to itself.
void flag_of_a_failed_pass()
{
    Nn s(20);
    const int32_t bad[4] = {1, 2, 99, 4}, good[4] = {1, 2, 3, 4};
    const float lab[2] = {1.f, 2.f};
    float pred[2];
    double loss;
    auto fails = [&](int how) {
        fail_launch["fwd"] = 1;
        split_status st = SPLIT_OK;
        if (how == 0) st = split_nn_gradient(s.nn, bad, lab, 2, 2, nullptr, &loss, nullptr);
        if (how == 1) st = split_nn_train_step(s.nn, bad, lab, 2, 2, 1e-3f, &loss, nullptr);
        if (how == 2) st = split_nn_predict(s.nn, bad, 2, 2, pred, nullptr);
        CHECK(st == SPLIT_E_HIP);
    };
    for (int how = 0; how < 3; ++how) {
        fails(how);
        CHECK(split_nn_gradient(s.nn, good, lab, 2, 2, nullptr, &loss, nullptr) == SPLIT_OK);
        fails(how);
        CHECK(split_nn_train_step(s.nn, good, lab, 2, 2, 1e-3f, &loss, nullptr) == SPLIT_OK);
        fails(how);
        CHECK(split_nn_predict(s.nn, good, 2, 2, pred, nullptr) == SPLIT_OK);
        fails(how);
        CHECK(split_nn_train(s.nn, good, lab, 2, 2, 1, 1, 1e-3f, 1, &loss, nullptr) == SPLIT_OK);
    }
    fail_launch["copy"] = 1;  // the flag's copy in split_nn_train
    CHECK(split_nn_train(s.nn, bad, lab, 2, 2, 1, 1, 1e-3f, 1, &loss, nullptr) == SPLIT_E_HIP);
    CHECK(split_nn_predict(s.nn, good, 2, 2, pred, nullptr) == SPLIT_OK);
    CHECK(split_nn_predict(s.nn, bad, 2, 2, pred, nullptr) == SPLIT_E_TOUR);
    CHECK(split_nn_predict(s.nn, good, 2, 2, pred, nullptr) == SPLIT_OK);
}

// An allocation that fails while the customers' statistics grow leaves no scenario set behind (and
// no half of the buffers): predictions are refused until a call has made both.
void scenarios_after_a_failed_allocation()
{
    for (int at = 1; at <= 2; ++at) {
        Nn s(20);
        std::vector<int32_t> tours((size_t)1 << 20, 1);
        std::vector<float> pred((size_t)1 << 18);
        s.ctx.coords(60);
        fail_malloc = at;
        CHECK(s.scenarios() == SPLIT_E_NOMEM);
        CHECK(fail_malloc == 0);
        s.ctx.coords(20);
        CHECK(split_nn_predict(s.nn, tours.data(), 2, 2, pred.data(), nullptr) == SPLIT_E_INVAL);
        // fewer customers than before the failure, and a call large enough to read the table
        CHECK(s.scenarios() == SPLIT_OK);
        CHECK(split_nn_predict(s.nn, tours.data(), 1 << 18, 4, pred.data(), nullptr) == SPLIT_OK);
        CHECK(count("customers") == at);
    }
}

// One tour 1..n over S scenarios of 5 units each.
split_tuning autotuned(int n, int64_t S, int Q, double *ms)
{
    Ctx c(n);
    std::vector<int32_t> tour, cost((size_t)S);
    for (int k = 1; k <= n; ++k) tour.push_back(k);
    const int64_t ptr[2] = {0, n};
    std::vector<int16_t> dem((size_t)n * S, 5);
    split_tuning best = {}, now = {};
    CHECK(split_autotune(c.c, tour.data(), ptr, 1, dem.data(), S, S, Q, cost.data(), S, 2, nullptr,
                         &best, ms) == SPLIT_OK);
    CHECK(split_tuning_get(c.c, &now) == SPLIT_OK);
    CHECK(memcmp(&best, &now, sizeof now) == 0);
    return best;
}

// The autotuner times the library's own choice too and installs nothing slower.
void autotune_times_the_own_choice()
{
    double ms = 0.0;
    // a short tour: one launch against three
    cost_us = {{"prep", 5}, {"tail", 5}, {"small", 8}, {"wave", 12},
               {"lane0", 20}, {"lane8", 20}, {"lane16", 20}};
    split_tuning t = autotuned(20, 1000, 100, &ms);
    CHECK(t.form == SPLIT_FORM_AUTO && t.lane_block == 0 && t.lane_per_cu == 0 && t.wave_grid == 0);
    CHECK(ms > 0.0079 && ms < 0.0081);
    // long windows: blocks of 16 run the tour before the tail kernel does it again
    cost_us = {{"prep", 5}, {"tail", 100}, {"pair0", 5}, {"pair16", 70}, {"lane0", 5},
               {"lane8", 105}, {"lane16", 105}, {"wave", 9000}};
    t = autotuned(700, 20000, 1200, &ms);
    CHECK(t.form != SPLIT_FORM_WAVE && t.lane_block == 0);
    CHECK(ms < 0.1101);
    // a difference within the noise: an explicit choice
    cost_us = {{"prep", 5}, {"tail", 5}, {"lane0", 40}, {"lane8", 40.5}, {"lane16", 60},
               {"wave", 9000}};
    t = autotuned(200, 65536, 60, &ms);
    CHECK(t.form == SPLIT_FORM_LANE && t.lane_block == 8);
    cost_us.clear();
}

// A replay takes the two-wavefront kernel where its own tours are long enough for it, not where the
// instance is.
void graph_replays_choose_by_their_tours()
{
    const int N = 400;
    const int64_t S = 640;
    for (int32_t block : {0, 16, 8}) {
        Ctx c(N);
        const split_tuning tu = {SPLIT_FORM_AUTO, 0, 0, 0, block};
        CHECK(split_tuning_set(c.c, &tu) == SPLIT_OK);
        std::vector<int16_t> dem((size_t)N * S, 5);
        std::vector<int32_t> cost((size_t)4 * S), tours;
        split_graph *g = nullptr;
        CHECK(split_graph_create(c.c, 4, 4 * N, dem.data(), S, S, 100, cost.data(), S, &g) == SPLIT_OK);
        const std::string lane = "lane" + std::to_string(block), pair = "pair" + std::to_string(block);
        auto replay = [&](std::vector<int> lens, bool two) {
            std::vector<int64_t> ptr = {0};
            tours.clear();
            for (int n : lens) {
                for (int k = 1; k <= n; ++k) tours.push_back(k);
                ptr.push_back((int64_t)tours.size());
            }
            trace.clear();
            CHECK(split_graph_launch(g, tours.data(), ptr.data(), (int32_t)lens.size(), nullptr) == SPLIT_OK);
            CHECK(split_graph_stats(g, nullptr, nullptr) == SPLIT_OK);
            two = two && block != 8;  // 8-state blocks are never halved
            CHECK(count(pair.c_str()) == (two ? 1 : 0) && count(lane.c_str()) == (two ? 0 : 1));
            CHECK(count("prep") == 1 && count("tail") == 1);
        };
        for (int rep = 0; rep < 3; ++rep) {  // both host slots
            replay({8}, false);
            replay({400}, true);
            replay({100, 300, 319}, false);
            replay({12, 320}, true);
        }
        split_graph_destroy(g);
    }
}

// Two wavefronts an item: where the tours are long enough for the number of items.
void two_wavefronts_by_length_and_items()
{
    const struct { int n; int64_t items; bool two; } cases[] = {
        {319, 768, false}, {320, 1, true}, {320, 768, true}, {320, 769, false}, {379, 1024, false},
        {380, 769, true}, {380, 1024, true}, {380, 1025, false}, {1000, 1024, true}};
    for (const auto &x : cases) {
        Ctx c(x.n);
        const int64_t S = 64 * x.items;
        std::vector<int32_t> tour, cost((size_t)S);
        for (int k = 1; k <= x.n; ++k) tour.push_back(k);
        std::vector<int16_t> dem((size_t)x.n * S, 5);
        trace.clear();
        CHECK(split_eval(c.c, tour.data(), x.n, dem.data(), S, S, 100, cost.data(), nullptr, nullptr) == SPLIT_OK);
        CHECK(count("pair0") == (x.two ? 1 : 0) && count("lane0") == (x.two ? 0 : 1));
    }
}

// The cost sums of a batch follow its scenarios, and grow with room to spare.
void sums_of_batches()
{
    const int N = 20, T = 4000;
    Ctx one(N), c(N);
    std::vector<int32_t> tours, cost((size_t)8 * 20000);
    std::vector<int64_t> ptr = {0};
    for (int t = 0; t < T; ++t) {
        for (int k = 1; k <= 5; ++k) tours.push_back(k);
        ptr.push_back((int64_t)tours.size());
    }
    std::vector<int16_t> dem((size_t)N * 20000, 5);
    auto batch = [&](const Ctx &on, int32_t n_tours, int64_t S) {
        return split_eval_batch(on.c, tours.data(), ptr.data(), n_tours, dem.data(), S, 20000, 100,
                                cost.data(), S, nullptr, nullptr, nullptr);
    };
    // per tour 16 bytes a position with its padding (and a quarter to spare), flags, and for one
    // scenario one entry of sums
    malloc_bytes = 0;
    CHECK(batch(one, T, 1) == SPLIT_OK);
    CHECK(malloc_bytes <= (size_t)T * ((16 * (6 + kRowPad) + 64) * 5 / 4 + 80));
    // a batch over ever more scenarios: the device is synchronized and buffers replaced now and then
    CHECK(batch(c, 8, 5000) == SPLIT_OK);
    syncs = mallocs = 0;
    for (int64_t S = 5000; S <= 20000; S += 64) CHECK(batch(c, 8, S) == SPLIT_OK);
    CHECK(syncs <= 8 && mallocs <= 8);  // four times as much, a quarter to spare each time
}

// Workgroups of the prep kernel: small ones where more short tours come than it has places.
void prep_workgroups()
{
    Ctx c(300);
    auto threads = [&](int T, int n) {
        std::vector<int32_t> tours, cost((size_t)T);
        std::vector<int64_t> ptr = {0};
        for (int t = 0; t < T; ++t) {
            for (int k = 1; k <= n; ++k) tours.push_back(k);
            ptr.push_back((int64_t)tours.size());
        }
        std::vector<int16_t> dem(300, 5);
        CHECK(split_eval_batch(c.c, tours.data(), ptr.data(), T, dem.data(), 1, 1, 100, cost.data(), 1,
                               nullptr, nullptr, nullptr) == SPLIT_OK);
        return prep_threads;
    };
    CHECK(threads(512, 100) == 1024 && threads(513, 100) == 256);
    CHECK(threads(513, 256) == 256 && threads(513, 257) == 1024 && threads(2, 10) == 1024);
}

// The timed interval is that of the kernel that took longest, and has its name.
void timing_names_the_dominant_kernel()
{
    const struct { int n; int64_t S; double lane, pair, tail; const char *name; double us; } cases[] = {
        {100, 10000, 50, 1, 5, "split_lane_kernel", 50},
        {700, 10000, 1, 60, 5, "split_pair_kernel", 60},
        {700, 10000, 1, 6, 140, "split_tail_kernel", 140},   // windows past the lane kernel's
        {100, 100000, 30, 1, 400, "split_tail_kernel", 400}};
    for (const auto &x : cases) {
        cost_us = {{"prep", 7}, {"lane0", x.lane}, {"pair0", x.pair}, {"tail", x.tail}, {"wave", 90}};
        Ctx c(x.n);
        std::vector<int32_t> tour, cost((size_t)x.S);
        for (int k = 1; k <= x.n; ++k) tour.push_back(k);
        std::vector<int16_t> dem((size_t)x.n * x.S, 5);
        CHECK(split_timing_enable(c.c, 1) == SPLIT_OK);
        double ms = 0.0;
        int64_t launches = 0, samples = 0;
        const char *name = nullptr;
        auto eval = [&] {
            CHECK(split_eval(c.c, tour.data(), x.n, dem.data(), x.S, x.S, 100, cost.data(), nullptr,
                             nullptr) == SPLIT_OK);
        };
        for (int k = 0; k < 3; ++k) eval();
        CHECK(split_timing_get(c.c, &ms, &launches, &name) == SPLIT_OK);
        CHECK(launches == 3 && ms > 2.999e-3 * x.us && ms < 3.001e-3 * x.us);
        CHECK(strcmp(name, x.name) == 0);
        float one[3];
        CHECK(split_timing_samples(c.c, one, 3, &samples) == SPLIT_OK && samples == 3);
        CHECK(one[2] > 0.999e-3 * x.us && one[2] < 1.001e-3 * x.us);
        // the wave form's tail only reports
        CHECK(split_set_form(c.c, SPLIT_FORM_WAVE) == SPLIT_OK);
        CHECK(split_timing_reset(c.c) == SPLIT_OK);
        eval();
        CHECK(split_timing_get(c.c, &ms, &launches, &name) == SPLIT_OK);
        CHECK(strcmp(name, "split_wave_kernel") == 0 && launches == 1 && ms > 0.0899 && ms < 0.0901);
    }
    cost_us.clear();
}

struct Scenario {
    const char *name;
    void (*run)();
};
const Scenario kScenarios[] = {
    {"flag-of-a-failed-pass", flag_of_a_failed_pass},
    {"scenarios-after-a-failed-allocation", scenarios_after_a_failed_allocation},
    {"autotune-times-the-own-choice", autotune_times_the_own_choice},
    {"graph-replays-choose-by-their-tours", graph_replays_choose_by_their_tours},
    {"two-wavefronts-by-length-and-items", two_wavefronts_by_length_and_items},
    {"sums-of-batches", sums_of_batches},
    {"prep-workgroups", prep_workgroups},
    {"timing-names-the-dominant-kernel", timing_names_the_dominant_kernel},
};

}  // namespace

int main(int argc, char **argv)
{
    for (const Scenario &s : kScenarios) {
        if (argc < 2) printf("%s\n", s.name);
        if (argc < 2 || strcmp(argv[1], s.name) != 0) continue;
        s.run();
        return failures ? 1 : 0;
    }
    return argc < 2 ? 0 : 2;
}
