// Internal interface between the C-ABI host layer (split_host.cpp) and the HIP kernels
// (split_kernels.hip). Not installed; callers use include/split.h.
//
// Every evaluation is a batch of T >= 1 giant tours over one instance and one demand matrix
// (split_eval is the batch of one). Per-tour arrays are concatenated: tour t's positions are
// tours[tptr[t] .. tptr[t+1]) and its derived arrays start at abase(t) = tptr[t] + t * (1 +
// kRowPad), each holding n_t + 1 + kRowPad entries.
//
// The kernels read T from device memory (the staged header), and their grids are sized for an
// upper bound of T: one captured HIP graph then serves every batch up to its capacity.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/split.h"

namespace splitgpu {

// Context accessors for the other host modules of the library (defined in split_host.cpp).
int ctx_device(const split_ctx *ctx);
// false when no instance is set
bool ctx_instance(const split_ctx *ctx, int32_t *N, int *kind, const int32_t **xy,
                  const int32_t **dist, int64_t *max_arc);
// the context's device scratch of split_topk_smallest (NULL until its first call; freed with the
// context)
void **ctx_topk_scratch(split_ctx *ctx);
// records the message as the context's last error and returns st
split_status ctx_fail(split_ctx *ctx, split_status st, const char *fmt, ...);

// "Infinity" for DP values. Host checks guarantee |DP value| + |weight| < 2^30.
constexpr int32_t kInf = 0x3fffffff;

// Cost mark of a scenario that a DP kernel leaves to the tail kernel (costs are >= 0).
constexpr int32_t kCostOvf = INT32_MIN;

// Device-side flags of one tour (zeroed by the prep kernel of each call).
struct DevStats {
    int32_t err_demand;  // nonzero: some scenario has q > Q (or q < 0) on the tour
    int32_t ovf_count;   // scenarios of this tour past the lane kernel's history
    uint32_t done;       // the tour's items that the tail kernel has finished
};

// Sums of some of a tour's costs: of the costs, and of their squares' low and high 32 bits (each
// below 2^63: a cost is below 2^30 and S below 2^31).
struct __attribute__((aligned(32))) CostSums {
    unsigned long long sum, sq_l32, sq_h32;
};

// Where the DP kernels leave them: slots entries per tour, `stride` bytes apart.
//  by item   one entry per work item, stored by it. For several tours: a workgroup that ends on
//            atomic additions holds its place until they are done, which made 256 tours over 65,536
//            scenarios 1.7% slower (8,710 us against 8,560).
//  added     a power of two of entries, kMaxSlots for one tour and as many as its additions can fill
//            for several; zeroed by the prep kernel and added to by the scenario's block (or the
//            scenario), each on a memory channel of its own: additions to one line, or to lines of
//            one channel, follow each other at about 11 ns. For one tour, whose workgroups go on to
//            their next item meanwhile, and for the other forms.
struct SumSlots {
    char *base;
    int64_t slots;
    int32_t stride;
    int32_t by_item;
};
constexpr int32_t kMaxSlots = 64;
constexpr int32_t kSlotStride = 256;
__host__ __device__ inline CostSums *sums_at(const SumSlots &s, int64_t t, int64_t k)
{
    return reinterpret_cast<CostSums *>(s.base + (t * s.slots + k) * s.stride);
}

// What the tail kernel reports of one tour (pinned host memory, or device memory where the caller
// copies it): sumsq = sq_l32 + 2^32 sq_h32.
struct TourResult {
    unsigned long long sum, sq_l32, sq_h32;
    int32_t err_demand, ovf_count;
};

// Batch-wide counters (reset by the prep kernel of each call).
struct BatchCtl {
    uint32_t head;       // next work item of the lane kernel's queue
    uint32_t ovf_total;  // nonzero: some scenario is marked kCostOvf
    uint32_t tail_head;  // next chunk of items of the tail kernel's queue
};

// Per-tour arrays built on the device by the prep kernel from the tours and the instance.
//   w[0]   = c(0, s_1)                                    (g_0 = f_0 + a_0)
//   w[i]   = c(s_i, 0) + c(0, s_{i+1}) - c(s_i, s_{i+1})   1 <= i <= n-1
//   w[n]   = D[n] + c(s_n, 0)                             (turns g back into f at i = n)
//   rowoff[i] = (s_i - 1) * ld * 2   (byte offset of position i's int16 demand row), 1 <= i <= n
// With g_p = f_p + c(0, s_{p+1}) - D[p+1] (D[k] = tour arc sum up to position k), Eq. (3)
// becomes g_i = w_i + min_{p in window(i)} g_p, and f_n = w_n + min_{p in window(n)} g_p.
// Each array carries kRowPad entries past position n (rowoff: a valid row; rowoff32: absent;
// w: zero) so that the kernels can read whole blocks of positions, up to six blocks past n,
// without guards.
constexpr int kRowPad = 128;

// rowoff32 value of a position without a demand (position 0, positions past n): beyond every
// lane_bytes, so the lane kernel's range-checked buffer loads return 0 for it.
constexpr uint32_t kRowAbsent = 0xFFFFFF00u;

__host__ __device__ inline int64_t tour_abase(const int64_t *tptr, int t)
{
    return tptr[t] + (int64_t)t * (1 + kRowPad);
}

// Header of an evaluation: int64 T, int64 tptr[T + 1], int32 order[T] (the lane kernel's work
// order), int32 tours[tptr[T]], each part at an offset fixed by the capacity the buffers were laid
// out for. The prep kernel reads it where the host wrote it (pinned host memory, or device memory
// that it was copied to) and leaves all but the tours in device memory for the other kernels.
struct TourDev {
    int64_t *nt;           // [1] number of tours T of this evaluation
    int64_t *tptr;         // [T + 1]
    int32_t *order;        // [T] work order of the lane kernel
    int32_t T_grid;        // upper bound of T that the launch grids are sized for
    int64_t *rowoff;       // concatenated, see above
    uint32_t *rowoff32;    // rowoff mod 2^32 (exact where it is used), kRowAbsent where absent
    int32_t *w;
    uint32_t *rowoff32_back;  // the pair kernel's mirrored half, indexed like rowoff32 and w
    int32_t *w_back;
};

struct PrepArgs {
    TourDev tour;
    const int64_t *src_nt;     // the header as the host wrote it
    const int64_t *src_tptr;
    const int32_t *src_order;
    const int32_t *src_tours;
    SumSlots sums;
    int32_t pair;              // 1: also the arrays of the mirrored half
    int32_t threads;           // of a workgroup: a multiple of 64, 64 (kMaxSlots) to 1024
    int32_t N;
    int32_t kind;          // 0: coordinates, 1: distance matrix
    const int32_t *xy;     // device [(N+1)*2]
    const int32_t *dist;   // device [(N+1)^2]
    int64_t ld;
    DevStats *stats;       // [T]
    BatchCtl *ctl;
};

struct EvalArgs {
    const uint16_t *demand;  // device, row-major [N][ld], read as unsigned (q > Q rejects q < 0)
    int64_t ld;
    int64_t S;
    int32_t Q;
    TourDev tour;
    int32_t *cost;           // device [T][ldc]
    int64_t ldc;
    DevStats *stats;         // [T]
    SumSlots sums;
    TourResult *out;         // [T] the tail kernel's report
    BatchCtl *ctl;
    uint32_t lane_bytes;     // lane kernel: bytes of demand it may address, <= kRowAbsent
    int32_t lane_grid;       // lane kernel workgroups (>= the work items: one item each)
    int32_t lane_static;     // lane kernel, fewer workgroups than items: 1 = each takes items
                             // at a fixed stride of lane_grid, 0 = from the queue
    int32_t lane_uniform;    // lane kernel: 1 = every tour of the launch has the same length
    int32_t lane_block;      // lane kernel block length: 16 or 8 states, 0 by the windows
    int32_t recount;         // 1: the tail kernel counts the scenarios past the lane kernel's history
    int32_t history_min_n;   // tail kernel: no mark of a shorter tour is for its windows
    int32_t tail_grid;       // tail kernel workgroups (at most)
    int32_t wave_grid;       // wave kernel workgroups of a full evaluation (form wave)
    int32_t maxn;            // bound on the tour lengths (sizes the wave kernel's LDS)
};

// A whole evaluation of one short tour over few scenarios in one launch.
constexpr int32_t kSmallN = 32;        // customers at most
constexpr int64_t kSmallS = 32768;     // scenarios at most: 128 workgroups
constexpr int32_t kSmallPer = 256;     // scenarios per workgroup
struct SmallArgs {
    const uint16_t *demand;
    int64_t ld, S;
    int32_t Q, n, N, kind;
    const int32_t *xy, *dist;
    int32_t *cost;                     // [S]
    TourResult *out;                   // one per workgroup
    int32_t count_bound;               // 1: count demands past the lane kernel's bound (n_fallback)
    int32_t tour[kSmallN];             // past n: the last customer again
};

// Kernel launchers (split_kernels.hip). All are asynchronous on `stream`.
hipError_t launch_prep(const PrepArgs &a, hipStream_t stream);
hipError_t launch_lane(const EvalArgs &a, hipStream_t stream);
hipError_t launch_small(const SmallArgs &a, hipStream_t stream);
hipError_t launch_pair(const EvalArgs &a, hipStream_t stream);
hipError_t launch_wave_all(const EvalArgs &a, hipStream_t stream);
hipError_t launch_tail(const EvalArgs &a, hipStream_t stream);
// two-kernel form: mask int16 [rows][mask_ld], row abase(t) + i
hipError_t launch_mask(const EvalArgs &a, int16_t *mask, long long mask_ld, hipStream_t stream);
hipError_t launch_masked_dp(const EvalArgs &a, const int16_t *mask, long long mask_ld,
                            hipStream_t stream);
const char *mask_kernel_name();
const char *lane_kernel_name();
const char *pair_kernel_name();
const char *tail_kernel_name();
const char *wave_kernel_name();

// Device scratch of the allocation-free evaluation: kScratchBytes per GPU, 256-byte aligned.
// scratch_address returns its device address on `device`, which must be the current device
// (looked up once per device, then cached).
constexpr size_t kScratchBytes = 192 * 1024;
constexpr int kMaxScratchDevices = 64;
hipError_t scratch_address(int device, void **out);

}  // namespace splitgpu
