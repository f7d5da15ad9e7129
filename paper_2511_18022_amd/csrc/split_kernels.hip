// HIP kernels for the scenario-batched Split (arXiv 2511.18022, Section 3) on gfx950.
//
// Notation (Section 3): positions 1..n of the giant tour s_1..s_n, DP states f(0..n),
// capacity window of state i = predecessors p in [mask(i), i-1] (Eq. (2)), Eq. (3) minimum
// over that window. The route cost of segment p+1..i splits into a term of p and a term of i,
// so with
//     g_p = f_p + c(0, s_{p+1}) - D[p+1]       (D[k] = sum of tour arcs up to position k)
// Eq. (3) becomes a sliding-window minimum:  g_i = w_i + min_{p in window(i)} g_p,
// where w_i depends on the tour only (built by split_prep_kernel) and f_n = g_n.
// All DP arithmetic is int32 and exact.
//
// Kernels:
//  split_prep_kernel      per-tour w_i and demand row offsets; zeroes the result block.
//  split_lane_kernel      one scenario per lane (scenario-level parallelism of Section 3);
//                         the window minimum is answered in O(1) per state from block
//                         suffix minima held in LDS; windows longer than its LDS history are
//                         left to the long kernel.
//  split_pair_kernel      the lane kernel with two wavefronts per 64 scenarios, from both ends of the
//                         tour, for launches of few work items.
//  split_small_kernel     a whole evaluation of a short tour over few scenarios.
//  split_tail_kernel      what the DP kernels left: the lane kernel's blocks over a history of 256
//                         positions for windows that outgrow the lane kernel's 64, then one
//                         scenario per wavefront for what outgrows that too; reports the sums.
//  split_wave_kernel      one scenario per wavefront; lanes cover the window's predecessors
//                         (transition-level parallelism of Section 3) and the minimum is a
//                         DPP reduction. Exact for any window length; used for small S.
// The DP kernels also add up the costs and their squares, exactly; the tail kernel reports them.
#include "split_internal.h"

#include <limits.h>

#include <mutex>
#include <type_traits>

namespace splitgpu {

// ------------------------------------------------------------------------- distances

// Nearest integer to the Euclidean distance between integer points (|coord| <= 2^20, so
// m < 2^43 and the double square root is within one unit of floor(sqrt(m))).
__device__ __forceinline__ int32_t dist_coords(const int32_t *xy, int u, int v)
{
    const long long dx = (long long)xy[2 * u] - xy[2 * v];
    const long long dy = (long long)xy[2 * u + 1] - xy[2 * v + 1];
    const long long m = dx * dx + dy * dy;
    long long k = (long long)sqrt((double)m);
    while (k * k > m) --k;
    while ((k + 1) * (k + 1) <= m) ++k;
    // m - k^2 > k  <=>  sqrt(m) > k + 1/2 (m integer: no exact halves)
    return (int32_t)(m - k * k > k ? k + 1 : k);
}

template <class A>
__device__ __forceinline__ int32_t arc_cost(const A &a, int u, int v)
{
    if (a.kind == 0) return dist_coords(a.xy, u, v);
    return a.dist[(long long)u * (a.N + 1) + v];
}

// The pair kernel (below) splits a tour in two halves.
// Last forward state of a tour of n >= 16 customers: about half of them, less the blocks that the
// join takes, one state short of a multiple of 16.
__host__ __device__ inline int pair_middle(int n)
{
    const int a = ((n + 1) >> 5) - 1;
    return 16 * (a > 1 ? a : 1) - 1;
}
__host__ __device__ inline int pair_shift(int n) { return (14 - n) & 15; }

// One workgroup per tour: the weights w, the row offsets and the padding of tour t, and the
// zeroed result block of the tour. Workgroup 0 also resets the batch counters. Workgroups
// past the call's T return at once.
// Bound by the round trips to the header in host memory. A workgroup of 1024 threads takes a tour of
// 1000 in one step, two of them fill a compute unit: where more short tours wait for a place,
// workgroups of 256 let eight at a time wait for theirs (65,536 tours of 40
// customers over 64 scenarios, from the launches to their end: 1.21 ms; 1.80 with 1024 threads, 1.40
// with 1024 and a header copied to the device before).
__global__ __launch_bounds__(1024) void split_prep_kernel(PrepArgs a)
{
    __shared__ long long red[16];
    __shared__ int32_t ends[2];  // c(0, first customer), c(last customer, 0)
    const int tid = threadIdx.x, threads = blockDim.x;
    const int t = blockIdx.x;
    // the header may lie in host memory: one round trip for these four, one for the tour
    const int64_t T = *a.src_nt, p0 = a.src_tptr[t], p1 = a.src_tptr[t + 1];
    const int32_t ord = a.src_order[t];
    if (t >= T) return;
    const int32_t *tour = a.src_tours + p0;
    const int n = (int)(p1 - p0);
    const int64_t ab = p0 + (int64_t)t * (1 + kRowPad);
    if (!a.sums.by_item && tid < a.sums.slots) *sums_at(a.sums, t, tid) = CostSums{0, 0, 0};
    int64_t *rowoff = a.tour.rowoff + ab;
    uint32_t *rowoff32 = a.tour.rowoff32 + ab;
    int32_t *w = a.tour.w + ab;
    long long link_sum = 0;
    for (int k = tid + 1; k <= n; k += threads) {
        const int sk = tour[k - 1];
        rowoff[k] = (long long)(sk - 1) * a.ld * (long long)sizeof(uint16_t);
        rowoff32[k] = (uint32_t)rowoff[k];
        // the two depot arcs of w_0 and w_n, from the threads that hold their customers
        if (k == 1) ends[0] = arc_cost(a, 0, sk);
        if (k == n) ends[1] = arc_cost(a, sk, 0);
        if (k < n) {
            const int sn = tour[k];
            const int link = arc_cost(a, sk, sn);
            link_sum += link;
            w[k] = arc_cost(a, sk, 0) + arc_cost(a, 0, sn) - link;
        }
    }
    // sum of the links: within each wavefront, then over the wavefronts (integers: the order does
    // not change the result)
    for (int off = 32; off > 0; off >>= 1) link_sum += __shfl_xor(link_sum, off, 64);
    if ((tid & 63) == 0) red[tid >> 6] = link_sum;
    __syncthreads();
    if (tid == 0) {
        for (int i = 1; i < threads / 64; ++i) red[0] += red[i];
    }
    __syncthreads();
    if (a.pair && n >= 16) {
        // the mirrored half: position k stands for break n - k + d (break n up to k = d); its demand
        // is that of the customer after the break
        uint32_t *rb = a.tour.rowoff32_back + ab;
        int32_t *wb = a.tour.w_back + ab;
        const int d = pair_shift(n);
        for (int k = tid; k <= n + kRowPad; k += threads) {
            const int i = n - k + d;  // break
            rb[k] = k <= d || i < 0 ? kRowAbsent : rowoff32[i + 1];
            wb[k] = k == 0 ? ends[1] : k <= d || i < 1 ? 0 : w[i];
        }
    }
    // positions n+1 .. n+kRowPad: row 0 (valid memory), absent for the lane kernel, weight 0,
    // so that kernels can load whole blocks of positions past n without guards
    for (int k = n + 1 + tid; k <= n + kRowPad; k += threads) {
        rowoff[k] = 0;
        rowoff32[k] = kRowAbsent;
        w[k] = 0;
    }
    if (tid == 0) {
        rowoff[0] = 0;
        rowoff32[0] = kRowAbsent;
        w[0] = ends[0];
        w[n] = (int32_t)(red[0] + ends[1]);
        a.stats[t] = DevStats{0, 0, 0};
        a.tour.tptr[t] = p0;
        a.tour.order[t] = ord;
        if (t == T - 1) a.tour.tptr[T] = p1;
        if (t == 0) {
            *a.tour.nt = T;
            *a.ctl = BatchCtl{0, 0, 0};
        }
    }
}

// ------------------------------------------------------------------------- sums of the costs

// Sum over the 64 lanes of a wavefront, in lane 63 (DPP row shifts and row broadcasts).
__device__ __forceinline__ uint32_t wave_sum_last(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return v;
}

// The sums of the 64 lanes' costs (each below 2^30; 0 where a lane has none) and their squares,
// in lane 63: 16-bit parts, whose sums over the lanes fit 32 bits.
__device__ __forceinline__ CostSums wave_costs(uint32_t c)
{
    const unsigned long long q = (unsigned long long)c * c;
    const uint32_t c0 = wave_sum_last(c & 0xFFFFu), c1 = wave_sum_last(c >> 16);
    const uint32_t q0 = wave_sum_last((uint32_t)q & 0xFFFFu);
    const uint32_t q1 = wave_sum_last((uint32_t)q >> 16);
    const uint32_t q2 = wave_sum_last((uint32_t)(q >> 32) & 0xFFFFu);
    const uint32_t q3 = wave_sum_last((uint32_t)(q >> 48));
    return CostSums{c0 + ((unsigned long long)c1 << 16), q0 + ((unsigned long long)q1 << 16),
                    q2 + ((unsigned long long)q3 << 16)};
}

__device__ __forceinline__ void add_sums(CostSums *to, const CostSums &v)
{
    atomicAdd(&to->sum, v.sum);
    atomicAdd(&to->sq_l32, v.sq_l32);
    atomicAdd(&to->sq_h32, v.sq_h32);
}

// Leaves the costs of work item (t, sb) in its slot. Two launches over the cost matrix did this
// before: 10 us of a call at 10^5 scenarios, 24 us of 256 tours over 65,536.
__device__ __forceinline__ void item_costs(const SumSlots &s, int t, long long sb, uint32_t c)
{
    const CostSums v = wave_costs(c);
    if ((threadIdx.x & 63) == 63) {
        if (s.by_item)
            *sums_at(s, t, sb) = v;
        else
            add_sums(sums_at(s, t, sb & (s.slots - 1)), v);
    }
}

// ------------------------------------------------------------------------- lane kernel
//
// One lane = one scenario; a workgroup is one wavefront of 64 scenarios. States 0..n are
// processed in blocks of LB states (block c = states LB*c .. LB*c + LB-1), LB = 16 or 8, a
// launch choice. A block's windows may reach back over the three blocks before it (windows
// of up to 3 * LB - 1 positions always fit): 16-state blocks suit windows of about 16 to 47
// positions; shorter windows mostly start inside a 16-state block, which takes the slow
// state-by-state path, and 8-state blocks keep them in older blocks. For state i, Eq. (3)'s
// window is [s_i, i-1] with s_i = #{p : P_p < P_i - Q} (Eq. (2); P = prefix loads).
//
// LDS per wavefront, every array interleaved by lane:
//   rec : per block slot c & 3, the pair (minimum of g over block c, minimum of the block
//         minima strictly between block c and the block being evaluated);
//   dl  : suffix minima of g inside each block of the last 64 positions, as 16-bit offsets
//         from the block minimum (row = position & 63);
//   pp  : prefix loads P mod 2^16 of the last 64 positions, positions (2k, 2k+1) in dword row
//         k & 31; rows 0 .. kMirror-1 repeated after the ring so that an 8-row read never wraps.
// The window minimum of a state of block c whose window starts at s in an older block b is
//   min(rec[b].bm + dl[s], rec[b].bs, minimum of g over block c before the state).
// Window starts advance by counting expired positions as packed 16-bit differences: the two
// states of a pair share one read of 12 positions starting at the even position below the
// previous start; in a fast block the first counts 8 of them and the second 10 (12 elsewhere).
// A block where some lane's last counted position expired (the count may be short), or where a
// count reached past the written prefix loads, has its starts redone. The counts are exact while
// 8 * max(q) + Q < 2^15 (every compared difference then fits a signed 16-bit value).
// Scenarios the kernel cannot finish exactly (that demand bound broken, a window longer than
// its history, suffix offsets beyond 16 bits) are queued for the general kernel.
//
// A window start s is carried as S = (s << 7) | (lane << 1): the dl offset, the pp row, the
// rec slot and the even base below s take one or two instructions each. The block loop is
// unrolled 64 / LB times so that every LDS store has a constant offset.

constexpr int kMirror = 7;  // ring rows repeated after the ring

// Blocks of LB states over a history of H positions: kRing = blocks in the history, kRecs = block
// records kept, kSteps = blocks unrolled in the block loop, kLog = log2(LB). The ring, the suffix
// offsets and the records hold every window start that lies at most kRecs - 1 blocks back.
// H = 64 (the lane kernel) unrolls its whole history, so that every LDS store has a constant
// offset; H = 256 (the long kernel, blocks of 16) adds the block's ring position to them.
template <int LB, int H>
struct LaneCfg {
    static_assert((H == 64 && (LB == 16 || LB == 8)) || (H == 256 && LB == 16),
                  "blocks of 16 or 8 states over 64 positions, of 16 over 256");
    static constexpr int kRing = H / LB;
    static constexpr int kRecs = H == 64 ? 4 : kRing;
    static constexpr int kSteps = H == 64 ? kRing : 4;
    static constexpr int kLog = LB == 16 ? 4 : 3;
    static constexpr int kPairs = H / 2;  // rows of the prefix-load ring, two positions each
    static constexpr uint32_t kDlMask = (uint32_t)(H * 128 - 1) & ~1u;
    static constexpr uint32_t kPpMask = (uint32_t)(kPairs * 256 - 1) & ~255u;
    static constexpr uint32_t kRecMask = (uint32_t)(kRecs - 1) * 512u;
};

template <int H>
struct __attribute__((aligned(16))) LaneLds {
    uint64_t rec[LaneCfg<16, H>::kRecs][64];
    uint16_t dl[H][64];
    uint32_t pp[H / 2 + kMirror][64];
    static constexpr uint32_t kDlOff = sizeof(uint64_t) * LaneCfg<16, H>::kRecs * 64;
    static constexpr uint32_t kPpOff = kDlOff + sizeof(uint16_t) * H * 64;
};

// Read-only per-tour arrays (written by the prep kernel, a previous launch): the constant
// address space lets every uniform read of them be a scalar load.
typedef __attribute__((address_space(4))) const uint32_t cu32;
typedef __attribute__((address_space(4))) const int32_t ci32;
typedef __attribute__((address_space(4))) const int64_t ci64;

typedef __attribute__((address_space(3))) uint64_t lds_u64;
typedef __attribute__((address_space(3))) uint32_t lds_u32;
typedef __attribute__((address_space(3))) uint16_t lds_u16;
typedef __attribute__((address_space(3))) char lds_char;
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int s_of(int S) { return S >> 7; }
__device__ __forceinline__ int S_of(int s, int lane) { return (s << 7) | (lane << 1); }

template <int H>
__device__ __forceinline__ const lds_char *lds_base(LaneLds<H> &L)
{
    return (const lds_char *)(&L);
}

// Window-minimum lookup of a start S (in an older block): the 16-bit suffix offset and the
// block record; combined later by query_min so that the reads are in flight meanwhile.
// The record slot (s / LB) & (kRecs - 1), 512 bytes a slot, is bits 9 and up of
// S >> (log2(LB) - 2).
template <int LB, int H>
__device__ __forceinline__ void query_issue(LaneLds<H> &L, int S, uint32_t lane8, uint32_t &dlv,
                                            uint64_t &recv)
{
    using C = LaneCfg<LB, H>;
    constexpr int kSh = C::kLog - 2;
    dlv = *(const lds_u16 *)(lds_base(L) + LaneLds<H>::kDlOff + ((uint32_t)S & C::kDlMask));
    recv = *(const lds_u64 *)(lds_base(L) + ((((uint32_t)S >> kSh) & C::kRecMask) | lane8));
}
__device__ __forceinline__ int query_min(uint32_t dlv, uint64_t recv, int pre)
{
    const int bm = (int)(uint32_t)recv;
    const int bs = (int)(uint32_t)(recv >> 32);
    return min(min(bm + (int)dlv, bs), pre);
}

// Offset of the ring row that holds a start S (and of the lane within it).
template <int H>
__device__ __forceinline__ uint32_t pp_off(int S, uint32_t lane4)
{
    return ((uint32_t)S & LaneCfg<16, H>::kPpMask) | lane4;
}
template <int H>
__device__ __forceinline__ uint32_t pp_at(LaneLds<H> &L, uint32_t off, int row)
{
    return *(const lds_u32 *)(lds_base(L) + LaneLds<H>::kPpOff + off + row * 256);
}
// 16-bit ring value of position p
template <int H>
__device__ __forceinline__ uint32_t pp_pos(LaneLds<H> &L, int lane, int p)
{
    const lds_u16 *h = (const lds_u16 *)(lds_base(L) + LaneLds<H>::kPpOff);
    return h[(((p >> 1) & (H / 2 - 1)) * 64 + lane) * 2 + (p & 1)];
}

// Packed 16-bit a - t in both halves, t a 16-bit value (no borrow between the halves).
__device__ __forceinline__ uint32_t pk_sub16(uint32_t a, uint32_t t)
{
    const u16x2 av = __builtin_bit_cast(u16x2, a);
    const u16x2 tv = {(unsigned short)t, (unsigned short)t};
    return __builtin_bit_cast(uint32_t, av - tv);
}
// Bytes 0..3 = 0xFF where the matching 16-bit half of (lo.lo, lo.hi, hi.lo, hi.hi) is negative.
__device__ __forceinline__ uint32_t sign_bytes(uint32_t hi, uint32_t lo)
{
    return __builtin_amdgcn_perm(hi, lo, 0x0b0a0908u);
}

// Exact start of a state with threshold T, advancing one position at a time from a start that
// is not past it. Bounded: position i of the state is never expired, and the ring holds it.
template <int H>
__device__ __forceinline__ int exact_start(LaneLds<H> &L, int lane, int S, uint32_t T)
{
    int s = s_of(S);
    for (int k = 0; k < H; ++k) {
        if ((int16_t)(uint16_t)(pp_pos(L, lane, s) - T) >= 0) break;
        ++s;
    }
    return S_of(s, lane);
}

// Prefix loads of block c (R = c mod kRing): q[j] is the demand of position LB*c + j (zero
// where a position does not exist). Writes the ring rows of the block and returns the packed
// thresholds TT[k] = (P_{LB*c+2k} - Q, P_{LB*c+2k+1} - Q) mod 2^16.
template <int LB, int H>
__device__ __forceinline__ void lane_prefix(LaneLds<H> &L, int lane, int R,
                                            const uint16_t (&q)[LB], uint32_t QQ,
                                            uint32_t &Plast, uint32_t &qor,
                                            uint32_t (&TT)[LB / 2])
{
    const int row0 = (LB / 2) * R;
    uint32_t prev = Plast;
#pragma unroll
    for (int k = 0; k < LB / 2; ++k) {
        // (q0, q1) packed by one byte permutation, then (q0, q0 + q1): the low half shifted
        // into the high half adds q0 there and leaves the low half alone
        const u16x2 qv = {q[2 * k], q[2 * k + 1]};
        const uint32_t Qp = __builtin_bit_cast(uint32_t, qv);
        const uint32_t E = Qp + (Qp << 16);
        const u16x2 ev = __builtin_bit_cast(u16x2, E);
        const u16x2 pv = __builtin_bit_cast(u16x2, prev);
        const u16x2 bc = {pv.y, pv.y};
        const uint32_t PP = __builtin_bit_cast(uint32_t, ev + bc);
        prev = PP;
        TT[k] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, PP) -
                                                 __builtin_bit_cast(u16x2, QQ));
        qor |= Qp;  // both halves: the bound below takes the larger
        L.pp[row0 + k][lane] = PP;
        if (row0 + k < kMirror) L.pp[row0 + k + H / 2][lane] = PP;
    }
    Plast = prev;
}

template <int LB>
__device__ __forceinline__ uint32_t tt_half(const uint32_t (&TT)[LB / 2], int t)
{
    return (t & 1) ? (TT[t >> 1] >> 16) : (TT[t >> 1] & 0xFFFFu);
}

// Window starts of the states first .. first + LB-1, one state at a time with an 8-position
// lookahead, completed exactly where the lookahead saturated or reached past the last written
// prefix load (first + LB-1). States past n (demand 0) get valid starts too. In: Sp = start of
// state first - 1.
template <int LB, int H>
__device__ __forceinline__ void lane_starts_careful(LaneLds<H> &L, int lane, int first,
                                                    const uint32_t (&TT)[LB / 2], int Sp,
                                                    int (&sOut)[LB])
{
    const uint32_t lane4 = (uint32_t)lane << 2;
#pragma unroll
    for (int t = 0; t < LB; ++t) {
        const uint32_t T = tt_half<LB>(TT, t);
        const uint32_t off = pp_off<H>(Sp, lane4);
        const uint32_t d0 = pp_at(L, off, 0), d1 = pp_at(L, off, 1);
        const uint32_t d2 = pp_at(L, off, 2), d3 = pp_at(L, off, 3);
        const uint32_t a01 = sign_bytes(pk_sub16(d1, T), pk_sub16(d0, T));
        const uint32_t a23 = sign_bytes(pk_sub16(d3, T), pk_sub16(d2, T));
        const int base = Sp & ~0x80;
        int Sn = base + (int)((__builtin_popcount(a23) + __builtin_popcount(a01)) << 4);
        // A short count (the eighth position expired too) is exact up to its end: every counted
        // position expired, so the walk continues from there. A read past the written prefix
        // loads (first + LB-1) may have counted stale positions: the walk starts over from Sp.
        const bool past = s_of(base) + 7 > first + LB - 1;
        const bool redo = (int32_t)a23 < 0 || past;
        if (redo) Sn = exact_start(L, lane, past ? Sp : Sn, T);
        sOut[t] = Sn;
        Sp = Sn;
    }
}

// Materializes v at this point of the instruction stream (keeps the compiler from sinking a
// computation towards a later use).
__device__ __forceinline__ void pin(int &v) { asm volatile("" : "+v"(v)); }

// The 12 positions a pair reads (6 packed dwords) and the even position they start at.
struct PairData {
    uint32_t d[6];
    int base;
};
template <int H>
__device__ __forceinline__ PairData pair_read(LaneLds<H> &L, uint32_t lane4, int Sp)
{
    PairData p;
    const uint32_t off = pp_off<H>(Sp, lane4);
#pragma unroll
    for (int r = 0; r < 6; ++r) p.d[r] = pp_at(L, off, r);
    p.base = Sp & ~0x80;
    return p;
}
// Start of a state with threshold T counted over the first 2 * D positions of a pair's read;
// last < 0: the last counted position expired too (the count may be short).
template <int D>
__device__ __forceinline__ int pair_count(const PairData &p, uint32_t T, uint32_t &last)
{
    uint32_t cnt = 0;
#pragma unroll
    for (int r = 0; r < D; r += 2) {
        const uint32_t x = sign_bytes(pk_sub16(p.d[r + 1], T), pk_sub16(p.d[r], T));
        cnt = __builtin_popcount(x) + cnt;
        last = x;
    }
    return p.base + (int)(cnt << 4);
}

// Start counted over the first 10 positions of a pair's read; last < 0: position 9 expired.
__device__ __forceinline__ int pair_count10(const PairData &p, uint32_t T, uint32_t &last)
{
    const uint32_t x0 = sign_bytes(pk_sub16(p.d[1], T), pk_sub16(p.d[0], T));
    const uint32_t x1 = sign_bytes(pk_sub16(p.d[3], T), pk_sub16(p.d[2], T));
    const uint32_t x2 = sign_bytes(pk_sub16(p.d[4], T), 0u);
    last = x2;
    uint32_t cnt = __builtin_popcount(x0);
    cnt = __builtin_popcount(x1) + cnt;
    cnt = __builtin_popcount(x2) + cnt;
    return p.base + (int)(cnt << 4);
}

// Window starts of the states first .. first + LB-1 from Sp (start of state first - 1) with the
// pair counts; where a count may be short or a read reached past the written prefix loads
// (first + LB-1), the block is redone state by state.
template <int LB, int H>
__device__ __forceinline__ void lane_starts_pairs(LaneLds<H> &L, int lane, int first,
                                                  const uint32_t (&TT)[LB / 2], int Sp,
                                                  int (&sOut)[LB])
{
    const uint32_t lane4 = (uint32_t)lane << 2;
    const int S_in = Sp;
    uint32_t sat = 0;
#pragma unroll
    for (int u = 0; u < LB / 2; ++u) {
        const PairData p = pair_read(L, lane4, Sp);
        uint32_t x0, x1;
        sOut[2 * u] = pair_count<4>(p, TT[u] & 0xFFFFu, x0);
        sOut[2 * u + 1] = pair_count<6>(p, TT[u] >> 16, x1);
        sat |= x0 | x1;
        Sp = sOut[2 * u + 1];
    }
    if (__any((int32_t)sat < 0 || (s_of(sOut[LB - 3]) & ~1) > first + LB - 12))
        lane_starts_careful<LB, H>(L, lane, first, TT, S_in, sOut);
}

// 16 positions (8 packed dwords) from the even position below Sp.
struct WideData {
    uint32_t d[8];
    int base;
};
template <int H>
__device__ __forceinline__ WideData wide_read(LaneLds<H> &L, uint32_t lane4, int Sp)
{
    WideData p;
    const uint32_t off = pp_off<H>(Sp, lane4);
#pragma unroll
    for (int r = 0; r < 8; ++r) p.d[r] = pp_at(L, off, r);
    p.base = Sp & ~0x80;
    return p;
}
template <int D>
__device__ __forceinline__ int wide_count(const WideData &p, uint32_t T, uint32_t &last)
{
    uint32_t cnt = 0;
#pragma unroll
    for (int r = 0; r < D; r += 2) {
        const uint32_t x = sign_bytes(pk_sub16(p.d[r + 1], T), pk_sub16(p.d[r], T));
        cnt = __builtin_popcount(x) + cnt;
        last = x;
    }
    return p.base + (int)(cnt << 4);
}
// Redo of a block's starts after the fast counts fell short or read past the written prefix
// loads: pairs again, from one 16-position read each, the first state counting 12 positions and
// the second all 16 (half the serial reads of a state-by-state redo, which has no other work
// left to overlap); where those fall short or read past the written prefix loads too, state by
// state. Used for 16-state blocks (an 8-state block's ring rarely holds 16 positions ahead).
template <int LB, int H>
__device__ __forceinline__ void lane_starts_wide(LaneLds<H> &L, int lane, int first,
                                                 const uint32_t (&TT)[LB / 2], int Sp,
                                                 int (&sOut)[LB])
{
    const uint32_t lane4 = (uint32_t)lane << 2;
    const int S_in = Sp;
    uint32_t sat = 0;
#pragma unroll
    for (int u = 0; u < LB / 2; ++u) {
        const WideData p = wide_read(L, lane4, Sp);
        uint32_t x0, x1;
        sOut[2 * u] = wide_count<6>(p, TT[u] & 0xFFFFu, x0);
        sOut[2 * u + 1] = wide_count<8>(p, TT[u] >> 16, x1);
        sat |= x0 | x1;
        Sp = sOut[2 * u + 1];
    }
    if (__any((int32_t)sat < 0 || (s_of(sOut[LB - 3]) & ~1) > first + LB - 16))
        lane_starts_careful<LB, H>(L, lane, first, TT, S_in, sOut);
}

// g of state t of a block (t uniform). Written as explicit selects: the compiler would
// otherwise turn it into an indexed load from a scratch copy of the whole block.
template <int LB>
__device__ __forceinline__ int block_g_at(const int (&gb)[LB], int t)
{
    t = __builtin_amdgcn_readfirstlane(t);
    int g = gb[0];
#pragma unroll
    for (int k = 1; k < LB; ++k) {
        int m = __builtin_amdgcn_readfirstlane(-(int)(t == k));
        asm volatile("" : "+s"(m));  // an opaque 0 / -1 mask
        g = (gb[k] & m) | (g & ~m);
    }
    return g;
}

// Block c complete (R = c mod kRing): suffix minima as 16-bit offsets from the block minimum,
// and the records of the kRecs - 1 newest blocks (bm[j]: minimum of block c - 1 - j).
template <int LB, int H>
__device__ __forceinline__ void lane_block_end(LaneLds<H> &L, int lane, int R,
                                               const int (&gb)[LB],
                                               int (&bm)[LaneCfg<LB, H>::kRecs - 2], int &ovf)
{
    constexpr int NR = LaneCfg<LB, H>::kRecs;
    int sm[LB];
    sm[LB - 1] = gb[LB - 1];
#pragma unroll
    for (int t = LB - 2; t >= 0; --t) sm[t] = min(sm[t + 1], gb[t]);
    const int bmin = sm[0];
    ovf |= (sm[LB - 1] - bmin) & ~0xFFFF;  // the largest offset is the last one
#pragma unroll
    for (int t = 0; t < LB; ++t) L.dl[LB * R + t][lane] = (uint16_t)(sm[t] - bmin);
    auto pack = [](int lo, int hi) {
        return (uint64_t)(uint32_t)lo | ((uint64_t)(uint32_t)hi << 32);
    };
    L.rec[R & (NR - 1)][lane] = pack(bmin, kInf);
    int between = bmin;
#pragma unroll
    for (int j = 1; j < NR - 1; ++j) {
        L.rec[(R + NR - j) & (NR - 1)][lane] = pack(bm[j - 1], between);
        between = min(between, bm[j - 1]);
    }
#pragma unroll
    for (int j = NR - 3; j > 0; --j) bm[j] = bm[j - 1];
    bm[0] = bmin;
}

// DP of block c, state by state, for any window position (inside the block, or empty).
// States past n (demand 0, weight 0) are evaluated too and not used.
template <int LB, int H>
__device__ __forceinline__ void lane_dp_careful(LaneLds<H> &L, int lane, int c,
                                                ci32 *__restrict__ w,
                                                const int (&sCur)[LB], int (&gb)[LB], bool &err)
{
    const int p0 = c * LB;
    const uint32_t lane8 = (uint32_t)lane << 3;
    // every state's older-block lookup, issued up front (in bounds for any start; a lane whose
    // window lies inside the block does not use its result)
    uint32_t qd[LB];
    uint64_t qr[LB];
#pragma unroll
    for (int t = 0; t < LB; ++t) query_issue<LB, H>(L, sCur[t], lane8, qd[t], qr[t]);
    int pre = kInf;
#pragma unroll
    for (int t = 0; t < LB; ++t) {
        const int i = p0 + t;
        int g;
        if (i == 0) {
            g = w[0];
        } else {
            const int s = s_of(sCur[t]);
            int m;
            if (s >= p0) {  // window inside the block, or empty (s == i: q_i > Q)
                err |= (s >= i);
                int mm = kInf;
                if (s == p0) {
                    mm = pre;  // the whole block so far (block 0 of a long-window tour)
                } else {
#pragma unroll
                    for (int j = 0; j < t; ++j)
                        if (p0 + j >= s) mm = min(mm, gb[j]);
                }
                m = mm;
            } else {
                m = query_min(qd[t], qr[t], pre);
            }
            g = w[i] + m;
        }
        gb[t] = g;
        pre = min(pre, g);
    }
}

// Demands of block blk, by buffer loads: the descriptor holds the demand base, the row's byte
// offset is the scalar offset and the lane's scenario offset the vector one. rowoff is padded
// past n with a valid row, so blocks past n load unguarded (their values are not used).
template <int LB>
__device__ __forceinline__ void lane_load_block(__amdgpu_buffer_rsrc_t rsrc,
                                                cu32 *__restrict__ rowoff,
                                                uint32_t lane_off, int blk, uint16_t (&q)[LB])
{
#pragma unroll
    for (int t = 0; t < LB; ++t)
        q[t] = __builtin_amdgcn_raw_buffer_load_b16(rsrc, lane_off, (int)rowoff[blk * LB + t], 0);
}

// The LB weights of block blk by vector loads (every lane the same 16 bytes, LB / 4 times): a
// scalar load here would need a wait that also drains every outstanding LDS operation.
typedef int i32x4 __attribute__((ext_vector_type(4)));
template <int LB>
__device__ __forceinline__ void lane_load_w(__amdgpu_buffer_rsrc_t wrsrc, int blk, int (&wv)[LB])
{
#pragma unroll
    for (int j = 0; j < LB / 4; ++j) {
        const i32x4 v = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                       wrsrc, 0, (blk * LB + 4 * j) * 4, 0));
        wv[4 * j] = v.x;
        wv[4 * j + 1] = v.y;
        wv[4 * j + 2] = v.z;
        wv[4 * j + 3] = v.w;
    }
}

template <int LB, int H>
struct LaneState {
    uint32_t Plast;  // high half: prefix load of the last position written to the ring
    uint32_t qor;    // OR of the demands read
    int bm[LaneCfg<LB, H>::kRecs - 2];  // minima of the last completed blocks
    int gres;        // g_n
    bool err;
    int ovf;         // nonzero: past the history or 16 bits (a lane mask in scalar registers
                     // measured 1% slower over the whole kernel)
    bool past;       // H = 256: a window start fell out of the lane kernel's 64 positions
    int Send;        // half a tour: start of its last state, and Plast as of that state
    uint32_t Pend;
};

// One block step (R = c mod kRing): demands of block c + 3, window starts of block c + 1, DP
// of block c. qUse holds the demands of block c + 1, qLoad receives those of block c + 3. HALF: the
// run ends inside a tour, in the last state of a block or (`fill`) in the one before, so that the
// last block's records are written too, and the tour goes on past it.
template <int LB, int H, bool HALF>
__device__ __forceinline__ void lane_step(LaneLds<H> &L, int lane, int R, int c, int n, bool fill, uint32_t QQ,
                                          __amdgpu_buffer_rsrc_t dem, __amdgpu_buffer_rsrc_t wrsrc,
                                          cu32 *__restrict__ rowoff, uint32_t lane_off,
                                          ci32 *__restrict__ w, const uint16_t (&qUse)[LB],
                                          uint16_t (&qLoad)[LB], const int (&sCur)[LB],
                                          int (&sNext)[LB], const int (&wUse)[LB],
                                          int (&wLoad)[LB], LaneState<LB, H> &st)
{
    using C = LaneCfg<LB, H>;
    // weights of block c + 1 (used by the next step), demands of block c + 3; unconditional,
    // so that every path has the same vector-memory wait counts
    lane_load_w<LB>(wrsrc, c + 1, wLoad);
    lane_load_block<LB>(dem, rowoff, lane_off, c + 3, qLoad);
    const int nb = n >> C::kLog;
    if (c > nb) return;
    const int p0 = c * LB;
    const int first = p0 + LB;  // states of block c + 1
    const uint32_t lane4 = (uint32_t)lane << 2, lane8 = (uint32_t)lane << 3;
    // the ring and the block records must still hold every window start of block c + 1
    // (state LB*c + LB-1 exists whenever block c + 1 does)
    if constexpr (HALF) {
        if (c == nb) {
            st.Send = sCur[LB - 1];
            st.Pend = st.Plast;
        }
    }
    if (HALF || c + 1 <= nb) {
        st.ovf |= (sCur[LB - 1] - ((p0 - (C::kRecs - 2) * LB) << 7)) & INT_MIN;
        if constexpr (H > 64) st.past |= sCur[LB - 1] < ((p0 - 2 * LB) << 7);
    }
    int gb[LB];
    // states past n (demand 0, weight 0) are evaluated like the others and not used
    const bool fast = c >= 1 && !__any(sCur[LB - 1] >= (p0 << 7));
    if (fast) {
        // Software pipeline over the LB/2 pairs of block c + 1 and the LB states of block c.
        // Iteration u: window lookups for the DP of the next pair, DP of states 2u, 2u+1,
        // first state of pair u-1, then second state of pair u (whose read was issued at the
        // end of iteration u-1) and the read of pair u+1. The scheduling barriers keep the
        // independent work between each read and its first use.
        // the block's weights, in vector registers since the previous step
        int wv[LB];
#pragma unroll
        for (int t = 0; t < LB; ++t) wv[t] = wUse[t];
        uint32_t TT[LB / 2];
        lane_prefix<LB, H>(L, lane, (R + 1) % C::kRing, qUse, QQ, st.Plast, st.qor, TT);
        uint32_t qd[LB];
        uint64_t qr[LB];
        query_issue<LB, H>(L, sCur[0], lane8, qd[0], qr[0]);
        query_issue<LB, H>(L, sCur[1], lane8, qd[1], qr[1]);
        PairData pcur = pair_read(L, lane4, sCur[LB - 1]);
        PairData pprev = pcur;
        uint32_t sat = 0;  // sign bit: some count of this lane may be short
        int pre = kInf;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < LB / 2; ++u) {
            if (u + 1 < LB / 2) {
                query_issue<LB, H>(L, sCur[2 * u + 2], lane8, qd[2 * u + 2], qr[2 * u + 2]);
                query_issue<LB, H>(L, sCur[2 * u + 3], lane8, qd[2 * u + 3], qr[2 * u + 3]);
            }
#pragma unroll
            for (int t = 2 * u; t < 2 * u + 2; ++t) {
                const int g = wv[t] + query_min(qd[t], qr[t], pre);
                gb[t] = g;
                pre = min(pre, g);
            }
            if (u > 0) {
                uint32_t x;
                sNext[2 * u - 2] = pair_count<4>(pprev, TT[u - 1] & 0xFFFFu, x);
                sat |= x;
                pin(sNext[2 * u - 2]);
            }
            __builtin_amdgcn_sched_barrier(0);
            uint32_t x1;
            sNext[2 * u + 1] = pair_count10(pcur, TT[u] >> 16, x1);
            sat |= x1;
            pprev = pcur;
            if (u + 1 < LB / 2) pcur = pair_read(L, lane4, sNext[2 * u + 1]);
            __builtin_amdgcn_sched_barrier(0);
        }
        {
            uint32_t x;
            sNext[LB - 2] = pair_count<4>(pprev, TT[LB / 2 - 1] & 0xFFFFu, x);
            sat |= x;
        }
        // no later block reads the last block's records (and its suffix offsets would hold
        // g_n = f_n, which need not fit 16 bits)
        if constexpr (HALF) {
            if (c == nb && fill) gb[LB - 1] = gb[LB - 2];
        }
        if (HALF || c < nb) lane_block_end<LB, H>(L, lane, R, gb, st.bm, st.ovf);
        // the last pair counts positions up to its base + 9; the ring is written up to
        // first + LB-1. Either condition below is rare: redo the block's starts (16-state
        // blocks with wider pair counts first, then state by state where those fall short).
        if (__any((int32_t)sat < 0 || (s_of(sNext[LB - 3]) & ~1) > first + LB - 10)) {
            if constexpr (LB == 16)
                lane_starts_wide<LB, H>(L, lane, first, TT, sCur[LB - 1], sNext);
            else
                lane_starts_careful<LB, H>(L, lane, first, TT, sCur[LB - 1], sNext);
        }
        if (!HALF && c == nb) st.gres = block_g_at<LB>(gb, n & (LB - 1));
        return;
    }
    // careful step (positions past n load demand 0)
    if (HALF || c + 1 <= nb) {
        uint32_t TT[LB / 2];
        lane_prefix<LB, H>(L, lane, (R + 1) % C::kRing, qUse, QQ, st.Plast, st.qor, TT);
        lane_starts_pairs<LB, H>(L, lane, first, TT, sCur[LB - 1], sNext);
    }
    lane_dp_careful<LB, H>(L, lane, c, w, sCur, gb, st.err);
    if constexpr (HALF) {
        if (c == nb && fill) gb[LB - 1] = gb[LB - 2];
    }
    if (HALF || c + 1 <= nb) {
        lane_block_end<LB, H>(L, lane, R, gb, st.bm, st.ovf);
    } else {
        st.gres = block_g_at<LB>(gb, n & (LB - 1));  // block c holds state n
    }
}

// Issue priority by progress through the work item: 3 over the first quarter of its blocks,
// down to 0 over the last. Among waves of equal priority a SIMD issues from the oldest, which
// drives the items of its two wavefronts half an item apart, so that at the end of a launch one
// of them runs alone for about half an item. Favouring the wavefront that is less far along
// keeps the two in step (measured on one tour: the two last items of a SIMD end about 14 us
// apart instead of 57, and the launch takes about 1% less). Used only when every item has the
// same length (one tour, or tours of one length): in a batch of uneven tours the items' ends
// are spread anyway, and this order measured about 0.5-0.9% slower there.
__device__ __forceinline__ void item_priority(int c, int nb)
{
    const int x = 4 * c, m = nb + 1;
    if (x < m)
        __builtin_amdgcn_s_setprio(3);
    else if (x < 2 * m)
        __builtin_amdgcn_s_setprio(2);
    else if (x < 3 * m)
        __builtin_amdgcn_s_setprio(1);
    else
        __builtin_amdgcn_s_setprio(0);
}

// A tour's per-position arrays and the descriptors of its weights and of the demands.
struct LaneTour {
    cu32 *__restrict__ rowoff;
    ci32 *__restrict__ w;
    __amdgpu_buffer_rsrc_t wrsrc;
    int n;
};

__device__ __forceinline__ LaneTour lane_tour(const EvalArgs &a, int t)
{
    // tour values come from memory: state that they are the same on every lane
    ci64 *tptr = (ci64 *)a.tour.tptr;
    const int64_t p0 = tptr[t];
    const int64_t ab = p0 + (int64_t)t * (1 + kRowPad);
    LaneTour r;
    r.n = (int)(tptr[t + 1] - p0);
    r.rowoff = (cu32 *)a.tour.rowoff32 + ab;
    r.w = (ci32 *)a.tour.w + ab;
    r.wrsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(a.tour.w + ab), (short)0,
                                                (int)(sizeof(int32_t) * (r.n + 1 + kRowPad)),
                                                0x00020000);
    return r;
}

// Counts are exact only while 8 * max(q) + Q < 2^15 (qor >= max(q), in either half); bit 15 (a negative
// int16 demand) also lands here, and the general kernel reports it.
__device__ __forceinline__ bool past_bound(uint32_t qor, int Q)
{
    return 8u * ((qor | (qor >> 16)) & 0xFFFFu) + (uint32_t)Q > 32767u;
}

// States 0..n of a tour for the scenarios at byte offset lane_off (one per lane) of its demand
// rows; qA, qB and qC hold the demands of blocks 0, 1 and 2. H = 256: ends where no lane that is
// wanted can be finished any more (one scenario with windows of 500 among 2^20: 1.70 ms a call
// without, 1.64 with).
template <int LB, int H, bool HALF = false>
__device__ __forceinline__ void lane_run(LaneLds<H> &L, const LaneTour &tr, int Q,
                                         __amdgpu_buffer_rsrc_t rsrc, uint32_t lane_off,
                                         uint16_t (&qA)[LB], uint16_t (&qB)[LB],
                                         uint16_t (&qC)[LB], bool by_progress,
                                         LaneState<LB, H> &st, bool fill = false, bool wanted = true)
{
    using C = LaneCfg<LB, H>;
    const int lane = threadIdx.x & 63;
    const int n = tr.n;
    cu32 *__restrict__ rowoff = tr.rowoff;
    ci32 *__restrict__ w = tr.w;
    const __amdgpu_buffer_rsrc_t wrsrc = tr.wrsrc;
    const uint32_t QQ = (uint32_t)Q | ((uint32_t)Q << 16);

    st.Plast = 0;
    st.qor = 0;
#pragma unroll
    for (int j = 0; j < C::kRecs - 2; ++j) st.bm[j] = kInf;
    st.gres = 0;
    st.err = false;
    st.ovf = 0;
    st.past = false;

    const int nb = n >> C::kLog;
    uint16_t qD[LB];
    int sA[LB], sB[LB];
    int wA[LB], wB[LB];  // weights of the block a step evaluates, loaded one step ahead
#pragma unroll
    for (int k = 0; k < LB; ++k) {
        sA[k] = S_of(0, lane);
        sB[k] = S_of(0, lane);
    }
    lane_load_w<LB>(wrsrc, 0, wA);
    {
        // block 0: position 0 has no demand (P_0 = 0, its row offset is absent); start 0
        uint32_t TT[LB / 2];
        lane_prefix<LB, H>(L, lane, 0, qA, QQ, st.Plast, st.qor, TT);
        lane_starts_pairs<LB, H>(L, lane, 0, TT, S_of(0, lane), sA);
    }
    // block b's demands live in q[A, B, C, D][b & 3], its starts and weights in [A, B][b & 1];
    // kSteps steps per iteration keep these roles constant (H = 64: and the LDS rows of a step)
    for (int c = 0; c <= nb; c += C::kSteps) {
        if (by_progress) item_priority(c, nb);
        if (H > 64 && !__any(wanted && st.ovf == 0 && !past_bound(st.qor, Q))) break;
        const int R = H == 64 ? 0 : c & (C::kRing - 1);
        lane_step<LB, H, HALF>(L, lane, R, c, n, fill, QQ, rsrc, wrsrc, rowoff, lane_off, w, qB, qD, sA, sB, wA, wB, st);
        lane_step<LB, H, HALF>(L, lane, R + 1, c + 1, n, fill, QQ, rsrc, wrsrc, rowoff, lane_off, w, qC, qA, sB, sA, wB, wA, st);
        lane_step<LB, H, HALF>(L, lane, R + 2, c + 2, n, fill, QQ, rsrc, wrsrc, rowoff, lane_off, w, qD, qB, sA, sB, wA, wB, st);
        lane_step<LB, H, HALF>(L, lane, R + 3, c + 3, n, fill, QQ, rsrc, wrsrc, rowoff, lane_off, w, qA, qC, sB, sA, wB, wA, st);
        if constexpr (C::kSteps == 8) {
            lane_step<LB, H, HALF>(L, lane, 4, c + 4, n, fill, QQ, rsrc, wrsrc, rowoff, lane_off, w, qB, qD, sA, sB, wA, wB, st);
            lane_step<LB, H, HALF>(L, lane, 5, c + 5, n, fill, QQ, rsrc, wrsrc, rowoff, lane_off, w, qC, qA, sB, sA, wB, wA, st);
            lane_step<LB, H, HALF>(L, lane, 6, c + 6, n, fill, QQ, rsrc, wrsrc, rowoff, lane_off, w, qD, qB, sA, sB, wA, wB, st);
            lane_step<LB, H, HALF>(L, lane, 7, c + 7, n, fill, QQ, rsrc, wrsrc, rowoff, lane_off, w, qA, qC, sB, sA, wB, wA, st);
        }
    }
    st.ovf |= past_bound(st.qor, Q);
}

// The end of a work item: the costs of the scenarios that are done; the others are marked for the
// tail kernel, which also counts them under `recount`.
__device__ __forceinline__ void lane_finish(const EvalArgs &a, int t, long long scen, int ovf,
                                            bool err, int gres, bool recount)
{
    __builtin_amdgcn_s_setprio(0);
    const bool active = scen < a.S;
    const bool left = active && ovf != 0;
    if (active && (left || !err))
        a.cost[(long long)t * a.ldc + scen] = left ? kCostOvf : gres;
    item_costs(a.sums, t, scen >> 6, active && !left && !err ? (uint32_t)gres : 0u);
    const unsigned long long m = __ballot(left);
    if (m != 0 && threadIdx.x == 0) {
        a.ctl->ovf_total = 1;  // whoever writes it, the same value
        if (!recount) atomicAdd(&a.stats[t].ovf_count, (int)__popcll(m));
    }
    if (active && !left && err) atomicOr(&a.stats[t].err_demand, 1);
}

// Sum over the 64 lanes of a wavefront, for all of them. (With shuffles windows_long cost the lane kernel
// 30 spilled scalars an item: 2% of a call over short tours.)
__device__ __forceinline__ float wave_fsum(float v)
{
    auto add = [&v](auto ctrl, auto rows) {
        v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value,
                                                        decltype(rows)::value, 0xf, false));
    };
    using std::integral_constant;
    add(integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{});  // row_shr:1
    add(integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{});  // row_shr:2
    add(integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{});  // row_shr:4
    add(integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{});  // row_shr:8
    add(integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{});  // row_bcast:15
    add(integral_constant<int, 0x143>{}, integral_constant<int, 0xc>{});  // row_bcast:31
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Whether windows are so long that an item of 64 scenarios almost surely has one of more than 47
// predecessors, from the 47 customers of positions 1 .. 47 in every scenario: the load of 48
// customers is about normal, its mean and its spread (per customer, over scenarios and positions,
// or of the whole load over the scenarios where that is wider) are those of the 47. A lane checks
// one window in 16, (n - 48) / 18 of them about independent; the item is expected to have 1.7 past
// the history where the capacity lies z standard deviations under the mean load of 48 with
// z^2 = 1.8 ln(n - 48) - 1.7 (within 0.3 for n of 65 to 5000). One in five such items has none.
// The line: an item left to the long kernel takes 4 times the lane kernel's share of the chip, one
// that the lane kernel marks after all, both. Measured, whole calls, 1000 customers, S = 2^20, mean
// windows of 41, 43, 44 and 60 under Poisson demands: 1.25, 4.34, 3.81 and 3.81 ms;
// 0.95 ms under constant demands and windows of up to 47. A rule by the first 15 customers' share of
// the capacity alone (at most 15 / 40) sent every item of all these to the long kernel.
__device__ __forceinline__ bool windows_long(const uint16_t (&qA)[16], const uint16_t (&qB)[16],
                                             const uint16_t (&qC)[16], int n, int Q)
{
    float load = 0.f, sq = 0.f;
    auto add = [&](const uint16_t (&q)[16]) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const float x = (float)q[j];
            load += x;
            sq += x * x;
        }
    };
    add(qA);  // position 0 has no demand
    add(qB);
    add(qC);
    const float s1 = wave_fsum(load), s2 = wave_fsum(load * load);
    sq = wave_fsum(sq);
    const float m = s1 / 64.f;  // mean load of 47 customers
    if (!(m > 0.f)) return true;
    const float cv2 = fmaxf(47.f * sq / (64.f * m * m) - 1.f, 47.f * (s2 / (64.f * m * m) - 1.f));
    const float room = 48.f - 47.f * (float)Q / m;
    const float z2 = 1.8f * __logf((float)(n - 48)) - 1.7f;
    return room <= 0.f || room * room <= z2 * 48.f * (cv2 - 1e-5f);
}

// The windows of a work item, from the demands of its first positions (loaded anyway):
//  kWindowsLong   see windows_long; looked at only where under half of the scenarios or more the
//                 first 15 customers fill at most 15 / 32 of the capacity;
//  kWindowsShort  the mean window W over the first 47 positions plus 4.6 times its spread (from the
//                 spread of those 47 customers' load over the scenarios) stays within 22, and under
//                 every scenario the first route holds at most 18 customers: 8-state blocks keep
//                 windows of up to 23, and a 16-state block would mostly see windows that start
//                 inside it. A lane whose first 15 customers fill at most 15 / 22 of the capacity
//                 decides against it from block 0 alone, before blocks 1 and 2 have arrived.
// Windows of 14.6 under uniform demands (a coefficient of variation of 0.55) pass 23 a few times in
// 10^5, and redoing their items made a call of 849 scenarios 121 us instead of 93.
// The class only chooses a kernel: what outgrows its history all the same is redone by the long one.
// Measured, whole calls: 200 customers, windows of 13, S = 10^5: 83 us (90 in blocks of 16);
// 1000 customers, windows of 60, S = 10,000: 167 us (249 with blocks of 16 first).
enum { kWindowsMid, kWindowsShort, kWindowsLong };
__device__ __forceinline__ int window_class(const uint16_t (&qA)[16], const uint16_t (&qB)[16],
                                            const uint16_t (&qC)[16], int n, int Q,
                                            bool active)
{
    int load = 0, len = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) load += qA[j];  // position 0 has no demand
    if (__any(22 * load <= 15 * Q)) {
        if (n <= 64 || 2 * __popcll(__ballot(active && 32 * load <= 15 * Q)) <
                           __popcll(__ballot(active)))
            return kWindowsMid;
        return windows_long(qA, qB, qC, n, Q) ? kWindowsLong : kWindowsMid;
    }
    load = 0;
    auto count = [&](const uint16_t (&q)[16]) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            load += q[j];
            len += load <= Q ? 1 : 0;  // counts position 0 too
        }
    };
    count(qA);
    count(qB);
    count(qC);
    if (__any(len > 19)) return kWindowsMid;
    float s1 = (float)load, s2 = s1 * s1;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        s1 += __shfl_xor(s1, off, 64);
        s2 += __shfl_xor(s2, off, 64);
    }
    const float k = (float)min(n, 47), m = s1 / 64.f;
    const float W = k * (float)Q / m;
    const float var = fmaxf(s2 / 64.f - m * m, 0.f) / (m * m) * k * W;
    const float room = 22.f - W;
    return __any(!(room > 0.f && 4.6f * 4.6f * var <= room * room)) ? kWindowsMid : kWindowsShort;
}

// One work item: the 64 scenarios sb*64 .. sb*64+63 of tour t. LB = 0: blocks of 8 or 16 states, or
// the long kernel, by the item's windows.
template <int LB>
__device__ __forceinline__ void lane_item(LaneLds<64> &L, const EvalArgs &a, int t, long long sb,
                                          __amdgpu_buffer_rsrc_t rsrc)
{
    const LaneTour tr = lane_tour(a, t);
    const long long scen = sb * 64 + (int)threadIdx.x;
    const uint32_t lane_off = (uint32_t)min(scen, (long long)a.S - 1) * 2u;
    const bool prio = a.lane_uniform != 0;
    if constexpr (LB == 8) {
        uint16_t qA[8], qB[8], qC[8];
        lane_load_block<8>(rsrc, tr.rowoff, lane_off, 0, qA);
        lane_load_block<8>(rsrc, tr.rowoff, lane_off, 1, qB);
        lane_load_block<8>(rsrc, tr.rowoff, lane_off, 2, qC);
        LaneState<8, 64> st;
        lane_run<8, 64>(L, tr, a.Q, rsrc, lane_off, qA, qB, qC, prio, st);
        lane_finish(a, t, scen, st.ovf, st.err, st.gres, false);
    } else {
        uint16_t qA[16], qB[16], qC[16];
        lane_load_block<16>(rsrc, tr.rowoff, lane_off, 0, qA);
        lane_load_block<16>(rsrc, tr.rowoff, lane_off, 1, qB);
        lane_load_block<16>(rsrc, tr.rowoff, lane_off, 2, qC);
        int cls = kWindowsMid;
        if constexpr (LB == 0) cls = window_class(qA, qB, qC, tr.n, a.Q, scen < a.S);
        int ovf = 1, gres = 0;
        bool err = false;
        if (__builtin_expect(cls == kWindowsMid, 1)) {
            LaneState<16, 64> st;
            lane_run<16, 64>(L, tr, a.Q, rsrc, lane_off, qA, qB, qC, prio, st);
            ovf = st.ovf;
            err = st.err;
            gres = st.gres;
        } else if (cls == kWindowsShort) {
            uint16_t rA[8], rB[8], rC[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                rA[j] = qA[j];
                rB[j] = qA[8 + j];
                rC[j] = qB[j];
            }
            LaneState<8, 64> st;
            lane_run<8, 64>(L, tr, a.Q, rsrc, lane_off, rA, rB, rC, prio, st);
            ovf = st.ovf;
            err = st.err;
            gres = st.gres;
        }
        lane_finish(a, t, scen, ovf, err, gres, true);
    }
}

// Work item k = (tour order[k / nsb], scenario block k % nsb), nsb = ceil(S / 64). Workgroup b
// runs item b, then either items b + gridDim.x, b + 2 gridDim.x, ... (lane_static) or items
// gridDim.x, gridDim.x + 1, ... taken from a queue until none is left (a grid of at least
// T * nsb workgroups runs one item each). A queue index is fetched while the current item runs.
// At the start of a 64 KB page: where its code lies after the kernels before it in this file moves a
// launch by up to 0.5% (in turn, three runs each: 256 tours, S = 65,536: 8,451 us so, 8,479 without;
// 1000 customers, S = 2^20: 930.5 and 934.1).
template <int LB>
__global__ __launch_bounds__(64) __attribute__((aligned(65536))) void split_lane_kernel(EvalArgs a)
{
    __shared__ LaneLds<64> L;
    const int lane = threadIdx.x;
    // raw buffer over the demand bytes the tours can address (gfx9 descriptor word 3:
    // 0x00020000); loads at offsets past lane_bytes (absent positions) return 0
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)a.demand, (short)0, (int)a.lane_bytes, 0x00020000);
    const long long nsb = (a.S + 63) / 64;
    const long long items = nsb * *(ci64 *)a.tour.nt;
    const bool queue = (long long)gridDim.x < items;
    uint32_t k = blockIdx.x;
    while ((long long)k < items) {
        uint32_t knext = 0xFFFFFFFFu;
        if (queue) {
            if (a.lane_static)
                knext = k + gridDim.x;
            else if (lane == 0)
                knext = gridDim.x + atomicAdd(&a.ctl->head, 1u);
        }
        const long long r = (long long)k / nsb;
        const int t = ((ci32 *)a.tour.order)[r];
        lane_item<LB>(L, a, t, (long long)k - r * nsb, rsrc);
        k = __builtin_amdgcn_readfirstlane(knext);
    }
}

// ------------------------------------------------------------------------- pair kernel
//
// A launch of few work items is bound by the serial chain of one wavefront per item, on a fraction
// of the chip. Here two wavefronts share an item: one runs the DP from the depot forward over states
// 0..m, the other from the tour's end backward over states n..m+1 (H_i = w_i + min of H over the
// predecessors' mirror image, the states that a route starting at i can end in), and the best pair
// of a forward and a backward state with one route between them joins them:
//     f_n = D[n] + min { G_p + H_i : p <= m < i, P_i - P_p <= Q }.
// The integers are the same, so is the minimum. The backward half is the same code on mirrored
// arrays (prep kernel): position k holds break n - k + d, and the first d + 1 positions stand for
// break n (no weight and a full vehicle's demand from one to the next: the same value); d makes the states k = 15, 31, ... those with
// n - k + d = 15, 31, ..., whose windows reach over more than 47 positions exactly where a forward
// state 48 positions on sees more than 47 predecessors: every scenario that the one-wavefront
// form would mark is marked here. m + 1 is a multiple of 16; the backward half then ends one state
// short of a full block.
// Measured, this kernel against the lane kernel: 1000 customers, 157 items 72 us against 104, 1024
// items 92 against 122. It is not half: the join takes about 10 us, and two wavefronts of one
// compute unit run each state 10 to 20% slower than one.

// The join, by the forward wavefront: window starts of the next (at most three) blocks of states
// i > m, the forward minimum over their predecessors up to m, and the backward suffix minimum at
// i (the least H from m + 1 to i in its block: a smaller i has an older start, so a minimum no
// larger, and the least sum is the same). Starts left at or before m after three blocks are past
// the history, and flagged by its test.
template <int LB>
__device__ __forceinline__ int pair_join(LaneLds<64> &F, LaneLds<64> &B, const LaneTour &tr, int Q,
                                         __amdgpu_buffer_rsrc_t rsrc, uint32_t lane_off, int m,
                                         LaneState<LB, 64> &st)
{
    using C = LaneCfg<LB, 64>;
    const int lane = threadIdx.x & 63;
    const uint32_t lane8 = (uint32_t)lane << 3;
    const uint32_t QQ = (uint32_t)Q | ((uint32_t)Q << 16);
    const int n = tr.n, k_of_0 = n + pair_shift(n);
    uint16_t q[LB], qn[LB];
    lane_load_block<LB>(rsrc, tr.rowoff, lane_off, (m + 1) / LB, q);
    uint32_t P = st.Pend;
    int Sp = st.Send, best = kInf;
    // one copy of the block's code: run two or three times, unrolled it would cost its fetches
#pragma unroll 1
    for (int e = 0; e < 3; ++e) {
        const int p0 = m + 1 + e * LB;
        if (p0 > n || !__any(Sp < S_of(m + 1, 0))) break;
        lane_load_block<LB>(rsrc, tr.rowoff, lane_off, p0 / LB + 1, qn);
        uint32_t TT[LB / 2];
        int s[LB];
        lane_prefix<LB, 64>(F, lane, (p0 / LB) & (C::kRing - 1), q, QQ, P, st.qor, TT);
        lane_starts_pairs<LB, 64>(F, lane, p0, TT, Sp, s);
#pragma unroll
        for (int t = 0; t < LB; ++t) {
            const int i = p0 + t;
            const int k = k_of_0 - i;  // the backward position of break i
            uint32_t dlv;
            uint64_t recv;
            query_issue<LB, 64>(F, s[t], lane8, dlv, recv);
            const int g = query_min(dlv, recv, kInf);
            const int h = (int)(uint32_t)B.rec[(k >> C::kLog) & 3][lane] + (int)B.dl[k & 63][lane];
            if (s_of(s[t]) <= m && i <= n) best = min(best, g + h);
            if (t == 0) st.err |= e == 0 && s_of(s[t]) > m;  // customer m + 1 does not fit
        }
#pragma unroll
        for (int t = 0; t < LB; ++t) q[t] = qn[t];
        Sp = s[LB - 1];
        st.ovf |= (Sp - ((p0 - 2 * LB) << 7)) & INT_MIN;
    }
    return best;
}

// Half of a work item in blocks of LB states; then, in the forward wavefront, the join: returns its
// scenario's cost.
template <int LB>
__device__ __forceinline__ int pair_item(LaneLds<64> (&L)[2], const EvalArgs &a, const LaneTour &tr,
                                         const LaneTour &half, int total, bool back, uint32_t lane_off,
                                         __amdgpu_buffer_rsrc_t rsrc, uint16_t (&qA)[LB],
                                         uint16_t (&qB)[LB], uint16_t (&qC)[LB], int &ovf,
                                         bool &err)
{
    const int lane = threadIdx.x & 63;
    LaneState<LB, 64> st;
    lane_run<LB, 64, true>(L[back], half, a.Q, rsrc, lane_off, qA, qB, qC, false, st, back);
    // the backward prefix loads are not needed any more: their first row takes its flags
    if (back) L[1].pp[0][lane] = (st.ovf != 0 ? 1u : 0u) | (st.err ? 2u : 0u);
    __syncthreads();
    if (back) return 0;
    const uint32_t flags = L[1].pp[0][lane];
    const int best = pair_join<LB>(L[0], L[1], tr, a.Q, rsrc, lane_off, half.n, st);
    ovf = st.ovf | (int)(flags & 1u) |
          (past_bound(st.qor, a.Q) ? 1 : 0);
    err = st.err || (flags & 2u);
    return total + best;
}

__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(2))) void split_pair_kernel(
    EvalArgs a)
{
    __shared__ LaneLds<64> L[2];
    __shared__ int s_class;
    const bool back = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) != 0;
    const int lane = threadIdx.x & 63;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)a.demand, (short)0, (int)a.lane_bytes, 0x00020000);
    const long long nsb = (a.S + 63) / 64;
    const long long k = blockIdx.x;
    if (k >= nsb * *(ci64 *)a.tour.nt) return;
    const int t = ((ci32 *)a.tour.order)[k / nsb];
    const long long sb = k - k / nsb * nsb;
    const LaneTour tr = lane_tour(a, t);
    const long long scen = sb * 64 + lane;
    const uint32_t lane_off = (uint32_t)min(scen, (long long)a.S - 1) * 2u;
    int cost = 0, ovf = 1;
    bool err = false;
    if (tr.n >= 16) {  // shorter tours go to the tail kernel
        const int m = pair_middle(tr.n);
        const int64_t ab = ((ci64 *)a.tour.tptr)[t] + (int64_t)t * (1 + kRowPad);
        LaneTour half = tr;
        half.n = m;
        ci32 *wb = (ci32 *)a.tour.w_back + ab;
        if (back) {
            half.n = tr.n - m - 1 + pair_shift(tr.n);
            half.rowoff = (cu32 *)a.tour.rowoff32_back + ab;
            half.w = wb;
            half.wrsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(a.tour.w_back + ab), (short)0,
                                                           (int)(sizeof(int32_t) * (tr.n + 1 + kRowPad)),
                                                           0x00020000);
        }
        const int total = tr.w[tr.n] - wb[0];  // the tour's arcs
        uint16_t qA[16], qB[16], qC[16];
        lane_load_block<16>(rsrc, half.rowoff, lane_off, 0, qA);
        lane_load_block<16>(rsrc, half.rowoff, lane_off, 1, qB);
        lane_load_block<16>(rsrc, half.rowoff, lane_off, 2, qC);
        if (back) {
            // positions 1 .. d demand a full vehicle: each sees the one before it, the customers'
            // windows none but the last
            const int d = pair_shift(tr.n);
#pragma unroll
            for (int j = 1; j < 16; ++j) qA[j] = j <= d ? (uint16_t)a.Q : qA[j];
        }
        int cls = kWindowsMid;
        if (a.lane_block == 0) {
            if (!back) {
                cls = window_class(qA, qB, qC, tr.n, a.Q, scen < a.S);
                if (lane == 0) s_class = cls;
            }
            __syncthreads();
            cls = __builtin_amdgcn_readfirstlane(s_class);
        }
        if (cls == kWindowsMid) {
            cost = pair_item<16>(L, a, tr, half, total, back, lane_off, rsrc, qA, qB, qC, ovf, err);
        } else if (cls == kWindowsShort) {
            uint16_t rA[8], rB[8], rC[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                rA[j] = qA[j];
                rB[j] = qA[8 + j];
                rC[j] = qB[j];
            }
            cost = pair_item<8>(L, a, tr, half, total, back, lane_off, rsrc, rA, rB, rC, ovf, err);
        }
    }
    if (!back) lane_finish(a, t, scen, ovf, err, cost, true);
}

// ------------------------------------------------------------------------- wave kernel

// Minimum over the 64 lanes of a wavefront with DPP row shifts and row broadcasts; the
// result is returned to every lane.
__device__ __forceinline__ int wave_min(int v)
{
    v = min(v, __builtin_amdgcn_update_dpp(kInf, v, 0x111, 0xf, 0xf, false));  // row_shr:1
    v = min(v, __builtin_amdgcn_update_dpp(kInf, v, 0x112, 0xf, 0xf, false));  // row_shr:2
    v = min(v, __builtin_amdgcn_update_dpp(kInf, v, 0x114, 0xf, 0xf, false));  // row_shr:4
    v = min(v, __builtin_amdgcn_update_dpp(kInf, v, 0x118, 0xf, 0xf, false));  // row_shr:8
    v = min(v, __builtin_amdgcn_update_dpp(kInf, v, 0x142, 0xa, 0xf, false));  // row_bcast:15
    v = min(v, __builtin_amdgcn_update_dpp(kInf, v, 0x143, 0xc, 0xf, false));  // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}

// Exclusive prefix sum over the 64 lanes.
__device__ __forceinline__ int wave_exclusive_sum(int v)
{
    const int lane = threadIdx.x & 63;
    int inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(inc, d, 64);
        if (lane >= d) inc += o;
    }
    return inc - v;
}

// Orders a wavefront's LDS accesses among its lanes (the others of its workgroup go their own way).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One scenario by one wavefront. First the prefix loads P_0..P_n are built in LDS with all
// lanes loading demands in parallel (chunk per lane + wavefront scan). Then, state by state,
// every lane runs the same two-pointer on the same data (uniform control flow), lane j reads
// g of predecessor s + j (+ 64k for long windows) and the wavefront reduces them.
// Returns the scenario's cost, or 0 where a demand is infeasible (flagged).
__device__ __forceinline__ uint32_t wave_one(const EvalArgs &a, int t, long long scen, int32_t *G,
                                             int32_t *PP)
{
    const int lane = threadIdx.x & 63;
    const int64_t ab = tour_abase(a.tour.tptr, t);
    const int n = (int)(a.tour.tptr[t + 1] - a.tour.tptr[t]);
    const int64_t *rowoff = a.tour.rowoff + ab;
    const int32_t *w = a.tour.w + ab;
    const int Q = a.Q;
    const char *dem = reinterpret_cast<const char *>(a.demand + scen);
    const int chunk = (n + 63) / 64;
    const int lo = lane * chunk + 1;
    const int hi = min(lo + chunk - 1, n);
    int local = 0;
    uint32_t qor = 0;
    for (int i = lo; i <= hi; ++i) {
        const uint32_t q = *(const uint16_t *)(dem + rowoff[i]);
        local += (int)q;
        qor |= q;
    }
    // a negative int16 demand (bit 15) is rejected for any Q, also where Q admits 2^15 and more
    const bool neg = __any((qor & 0x8000u) != 0);
    int run = wave_exclusive_sum(local);
    for (int i = lo; i <= hi; ++i) {
        run += *(const uint16_t *)(dem + rowoff[i]);
        PP[i] = run;
    }
    if (lane == 0) {
        PP[0] = 0;
        G[0] = w[0];
    }
    wave_sync();
    int s = 0;
    bool err = neg;
    for (int i = 1; i <= n && !err; ++i) {
        const int P = PP[i];
        while (P - PP[s] > Q) ++s;
        if (s == i) {
            err = true;
            break;
        }
        int mn = kInf;
        for (int base = s; base < i; base += 64) {
            const int p = base + lane;
            if (p < i) mn = min(mn, G[p]);
        }
        G[i] = wave_min(mn) + w[i];
    }
    const int32_t cost = err ? 0 : G[n];
    if (lane == 0) {
        if (err)
            atomicOr(&a.stats[t].err_demand, 1);
        else
            a.cost[(long long)t * a.ldc + scen] = cost;
    }
    wave_sync();
    return (uint32_t)cost;
}

// Every (tour, scenario) pair, k = t * S + s over k = blockIdx.x, blockIdx.x + gridDim.x, ...
__global__ __launch_bounds__(64) void split_wave_kernel(EvalArgs a)
{
    extern __shared__ int32_t lds[];
    int32_t *G = lds;
    int32_t *PP = lds + (a.maxn + 1);
    const long long T = *a.tour.nt;
    for (long long k = blockIdx.x; k < T * a.S; k += gridDim.x) {
        const int t = (int)(k / a.S);
        const long long scen = k - (long long)t * a.S;
        const uint32_t c = wave_one(a, t, scen, G, PP);
        if (threadIdx.x == 0) {
            const unsigned long long q = (unsigned long long)c * c;
            add_sums(sums_at(a.sums, t, scen & (a.sums.slots - 1)),
                     CostSums{c, q & 0xFFFFFFFFull, q >> 32});
        }
    }
}

// ------------------------------------------------------------------------- tail kernel

// Tour t's result from its slots, by one wavefront. The slots were added to at the device's scope,
// by earlier launches or (once every workgroup is counted in) by this one: read there too.
__device__ __forceinline__ void report_tour(const EvalArgs &a, int t)
{
    const int lane = threadIdx.x & 63;
    auto load = [](const auto *p) {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    unsigned long long v[3] = {0, 0, 0};
#pragma unroll 8
    for (long long k = lane; k < a.sums.slots; k += 64) {
        const CostSums *s = sums_at(a.sums, t, k);
        v[0] += load(&s->sum);
        v[1] += load(&s->sq_l32);
        v[2] += load(&s->sq_h32);
    }
    for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
        for (int j = 0; j < 3; ++j) v[j] += __shfl_xor(v[j], off, 64);
    }
    if (lane == 0)
        a.out[t] = TourResult{v[0], v[1], v[2], load(&a.stats[t].err_demand),
                              load(&a.stats[t].ovf_count)};
}

// The scenarios that the DP kernels marked, 64 at a time through the lane kernel's blocks of 16 over a
// history of 256 positions (windows of up to 239), by the first wavefront. Those that outgrow this
// history too, or whose suffix offsets or demands pass 16 bits, are then finished one by one, a
// scenario by each of the four wavefronts, in the same LDS. With a.recount the kernel counts the
// scenarios past the lane kernel's history (n_fallback): an item is left here whole.
//
// Bound by the latency of one wavefront's serial chain: 80 KB of LDS leave two workgroups a compute
// unit. For the blocks that is still one state of 64 scenarios per step, where one scenario per
// wavefront leaves most lanes idle: 701 customers, windows of about 60, S = 20,011 took 14.76 ms as
// a call; with this kernel 0.13 ms. One by one, four wavefronts a workgroup take as many scenarios
// at once as a kernel of their own with 8 bytes of LDS a position did: 200 customers, coordinates up
// to 10^5, S = 2^17: 4.3 ms a call (19.0 with one wavefront, 4.5 in the separate kernel); 1000
// customers, windows of 300, S = 2^17: 32.7 (149.5 and 35.1). wave_one has to be inlined: as a call
// it reads LDS through generic pointers, and keeps the blocks' registers in scratch memory (1000
// customers, windows of 60, S = 2^20: 6.1 ms a call against 3.8).
// Counts go to memory once per item: one atomic per scenario took 240 us of this launch there.
//
// Where something is marked, workgroups take chunks of items from a queue: marks are mostly few and
// may come at any stride (the same scenarios of every tour, say). Up to kTailChunk items a chunk, so
// that the queue's counter is no bottleneck, and about 16 chunks a workgroup.
// 256 tours over 65,536 scenarios, four of them with windows of 500: 10.0 ms a call (8.9 without
// them; 228 with items at a fixed stride and the last workgroup reporting every tour, 51 with 2,048
// workgroups at a fixed stride); 1000 customers, S = 2^20, windows of 42, 3,279 marks: 1.9 ms (3.9
// and 3.4).
//
// The tours' results go straight to the caller's (pinned host) memory. Where nothing was marked, each
// wavefront reports its share at once; otherwise whoever finishes the last of a tour's items reports
// the tour.
constexpr int kTailWaves = 4;
constexpr int kTailChunk = 32;
constexpr int kTailWords = (80 * 1024 - 16 * kTailChunk - 64) / 4;  // two workgroups fill a compute unit's LDS

__global__ __launch_bounds__(64 * kTailWaves) __attribute__((amdgpu_waves_per_eu(2)))
void split_tail_kernel(EvalArgs a)
{
    __shared__ union {
        LaneLds<256> L;
        int32_t words[kTailWords];
    } lds;
    // the scenarios of a chunk's items that are left, at first and after the history
    __shared__ unsigned long long s_todo[kTailChunk], s_wide[kTailChunk];
    __shared__ uint32_t s_chunk, s_marks;
    static_assert(sizeof lds == 4 * kTailWords && kTailWords >= 2 * (SPLIT_MAX_N + 1),
                  "the history fits, and a wavefront's prefix loads and g values of a maximal tour");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const long long T = *(ci64 *)a.tour.nt;
    if (*(cu32 *)&a.ctl->ovf_total == 0) {
        for (long long t = (long long)blockIdx.x * kTailWaves + wave; t < T;
             t += (long long)gridDim.x * kTailWaves)
            report_tour(a, (int)t);
        return;
    }
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)a.demand, (short)0, (int)a.lane_bytes, 0x00020000);
    const long long nsb = (a.S + 63) / 64, items = T * nsb;
    const int per = (int)min((long long)kTailChunk, max(1ll, items / (16ll * gridDim.x)));
    // the wavefronts that have room for a tour's arrays of their own
    const int room = 2 * (a.maxn + 1);
    const int nw = min(kTailWaves, kTailWords / room);
    int32_t *G = lds.words + wave * room;
    for (;;) {
        __syncthreads();  // the last chunk's LDS is free
        if (threadIdx.x == 0) {
            s_chunk = atomicAdd(&a.ctl->tail_head, 1u);
            s_marks = 0;
        }
        __syncthreads();
        const long long k0 = (long long)s_chunk * per;
        if (k0 >= items) return;
        const int cnt = (int)min((long long)per, items - k0);
        const int t0 = (int)(k0 / nsb);
        const long long sb0 = k0 - (long long)t0 * nsb;
        // tour, scenario block and sums of the chunk's item i
        auto item = [&](int i, int &t, long long &sb) {
            const long long past = sb0 + i;  // within the tour, or past its end
            const int dt = past < nsb ? 0 : (int)((uint32_t)past / (uint32_t)nsb);
            t = t0 + dt;
            sb = past - dt * nsb;
        };
        auto sums = [&](int t, long long sb) {
            return sums_at(a.sums, t, a.sums.by_item ? sb : sb & (a.sums.slots - 1));
        };
        for (int i = wave; i < cnt; i += kTailWaves) {
            int t;
            long long sb;
            item(i, t, sb);
            const long long scen = sb * 64 + lane;
            const int32_t mark = scen < a.S ? a.cost[(long long)t * a.ldc + scen] : 0;
            const unsigned long long todo = __ballot(mark == kCostOvf);
            if (lane == 0) {
                s_todo[i] = todo;
                s_wide[i] = 0;
                if (todo) s_marks = 1;  // whoever writes it, the same value
            }
        }
        __syncthreads();
        const bool marks = s_marks != 0;
        if (marks && wave == 0) {
            for (int i = 0; i < cnt; ++i) {
                const unsigned long long todo = s_todo[i];
                if (todo == 0) continue;
                int t;
                long long sb;
                item(i, t, sb);
                const bool mine = (todo >> lane) & 1;
                const long long scen = min(sb * 64 + lane, (long long)a.S - 1);
                LaneState<16, 256> st;
                st.ovf = 1;
                st.past = false;
                st.err = false;
                st.gres = 0;
                // the demands lie within a buffer descriptor's reach, and a longer history can help (20
                // customers, coordinates up to 10^5, S = 2^20: 0.90 ms a call, 1.23 with the blocks first)
                const LaneTour tr = lane_tour(a, t);
                if (a.lane_bytes != 0 && tr.n >= a.history_min_n) {
                    const uint32_t lane_off = (uint32_t)scen * 2u;
                    uint16_t qA[16], qB[16], qC[16];
                    lane_load_block<16>(rsrc, tr.rowoff, lane_off, 0, qA);
                    lane_load_block<16>(rsrc, tr.rowoff, lane_off, 1, qB);
                    lane_load_block<16>(rsrc, tr.rowoff, lane_off, 2, qC);
                    lane_run<16, 256>(lds.L, tr, a.Q, rsrc, lane_off, qA, qB, qC, false, st, false, mine);
                }
                const int past = (int)__popcll(__ballot(mine && (st.past || st.ovf)));
                const unsigned long long wide = __ballot(mine && st.ovf);
                uint32_t c = 0;
                if (mine && st.ovf == 0) {
                    if (st.err) {
                        atomicOr(&a.stats[t].err_demand, 1);
                    } else {
                        c = (uint32_t)st.gres;
                        a.cost[(long long)t * a.ldc + scen] = st.gres;
                    }
                }
                const CostSums v = wave_costs(c);
                if (lane == 63) add_sums(sums(t, sb), v);
                if (lane == 0) {
                    if (a.recount && past) atomicAdd(&a.stats[t].ovf_count, past);
                    s_wide[i] = wide;
                }
            }
        }
        if (marks) __syncthreads();
        if (marks && wave < nw) {
            int turn = 0;
            for (int i = 0; i < cnt; ++i) {
                int t;
                long long sb;
                item(i, t, sb);
                for (unsigned long long m = s_wide[i]; m; m &= m - 1) {
                    const int j = __builtin_ctzll(m);
                    const bool mine = turn == wave;
                    turn = turn + 1 < nw ? turn + 1 : 0;
                    if (!mine) continue;
                    const unsigned long long c = wave_one(a, t, sb * 64 + j, G, G + a.maxn + 1);
                    const unsigned long long q = c * c;
                    if (lane == 0) add_sums(sums(t, sb), CostSums{c, q & 0xFFFFFFFFull, q >> 32});
                }
            }
        }
        // Every wavefront's additions are complete before the chunk's items count as done. They are
        // atomic at the device's scope, as the count and the reads of a report are, so their
        // completion is all that is waited for: a fence would write a whole L2 back (153 customers,
        // windows of 56, S = 56,771: 105 us a call, 152 with a fence a chunk).
        if (marks) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
        }
        for (int t = t0 + wave; (t - t0) * nsb < sb0 + cnt; t += kTailWaves) {
            const long long lo = max(0ll, sb0 - (t - t0) * nsb);
            const long long hi = min(nsb, sb0 + cnt - (t - t0) * nsb);
            const uint32_t mine = (uint32_t)(hi - lo);
            uint32_t before = 0;
            if (lane == 0) before = atomicAdd(&a.stats[t].done, mine);
            if ((uint32_t)__builtin_amdgcn_readfirstlane((int)before) + mine != (uint32_t)nsb) continue;
            asm volatile("" ::: "memory");
            report_tour(a, t);
        }
    }
}

// ------------------------------------------------------------------------- small evaluations

// One tour of at most kSmallN customers, one scenario per thread, in one launch: the tour comes with
// the arguments, every workgroup computes the weights for itself, prefix loads and g stay in
// registers, each state takes the minimum over its predecessors one by one (496 of them at most),
// and every workgroup reports its part to pinned host memory, where the host adds up at most 128 of
// them: with atomic sums, a count of the finished workgroups and the window scan in LDS the kernel
// took 30 us. Bound by launch and memory latency: 20 customers, S = 1000 takes 7.6 us here.
__global__ __launch_bounds__(kSmallPer) void split_small_kernel(SmallArgs a)
{
    __shared__ int32_t w[kSmallN + 1];
    __shared__ CostSums part[kSmallPer / 64];
    __shared__ int32_t flags[kSmallPer / 64][2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = a.n;
    const long long scen = (long long)blockIdx.x * kSmallPer + tid;
    const bool active = scen < a.S;
    const int s32 = (int)min(scen, (long long)a.S - 1);
    uint32_t q[kSmallN];
#pragma unroll
    for (int i = 0; i < kSmallN; ++i) {  // past the tour: its last customer again, not used
        const uint16_t *row = a.demand + (long long)(a.tour[i] - 1) * a.ld;
        q[i] = row[s32];
    }
    if (wave == 0) {
        // lane k's customer, from scalar registers (an indexed read of the arguments is a round trip
        // to memory)
        int after = 0;
#pragma unroll
        for (int i = 0; i < kSmallN; ++i) after = lane == i ? a.tour[i] : after;
        const int up = __shfl_up(after, 1, 64);
        const int before = lane > 0 ? up : 0;
        after = lane < n ? after : 0;
        int link = 0;
        if (lane <= n) {
            const int in = lane > 0 ? arc_cost(a, before, 0) : 0;
            const int out = lane < n ? arc_cost(a, 0, after) : 0;
            if (lane > 0 && lane < n) link = arc_cost(a, before, after);
            w[lane] = in + out - link;
        }
        for (int off = 32; off > 0; off >>= 1) link += __shfl_xor(link, off, 64);
        if (lane == n) w[n] += link;  // the arcs of the tour: turns g back into f
    }
    __syncthreads();
    uint32_t qor = 0;
    bool err = false;
    int P[kSmallN + 1], G[kSmallN + 1];
    P[0] = 0;
    G[0] = w[0];
    int cost = 0;
#pragma unroll
    for (int i = 1; i <= kSmallN; ++i) {
        if (i <= n) {
            P[i] = P[i - 1] + (int)q[i - 1];
            qor |= q[i - 1];
            err |= (int)q[i - 1] > a.Q;
            const int over = P[i] - a.Q;  // predecessors with a smaller prefix load are out
            int m = kInf;
#pragma unroll
            for (int p = i - 1; p >= 0; --p) m = min(m, P[p] >= over ? G[p] : kInf);
            G[i] = w[i] + m;
            cost = G[i];
        } else {
            P[i] = 0;
            G[i] = 0;
        }
    }
    err |= (qor & 0x8000u) != 0;  // a negative int16 demand, for any Q
    const bool ok = active && !err;
    if (ok) a.cost[scen] = cost;
    const CostSums v = wave_costs(ok ? (uint32_t)cost : 0u);
    const unsigned long long bad = __ballot(active && err);
    const unsigned long long past =
        __ballot(active && a.count_bound && 8u * qor + (uint32_t)a.Q > 32767u);
    if (lane == 63) {
        part[wave] = v;
        flags[wave][0] = bad != 0;
        flags[wave][1] = (int)__popcll(past);
    }
    __syncthreads();
    if (tid == 0) {
        TourResult r = {0, 0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < kSmallPer / 64; ++k) {
            r.sum += part[k].sum;
            r.sq_l32 += part[k].sq_l32;
            r.sq_h32 += part[k].sq_h32;
            r.err_demand |= flags[k][0];
            r.ovf_count += flags[k][1];
        }
        a.out[blockIdx.x] = r;
    }
}

// ------------------------------------------------------------------------- two-kernel form

// The paper's literal two-kernel form, kept as an ablation of the fused lane kernel: first the
// Eq. (2) window starts of every (state, scenario) are written to an int16 matrix in HBM
// (row abase(t) + i, scenario fastest), then a second kernel reads them back and takes each
// window's minimum by scanning it.

// One lane per scenario of work item (tour, 64-scenario block): prefix loads with a two-pointer;
// mask = smallest p with P_i - P_p <= Q (p == i when q_i > Q: the window is empty).
__global__ __launch_bounds__(64) void split_mask_kernel(EvalArgs a, int16_t *mask,
                                                        long long mask_ld)
{
    const long long nsb = (a.S + 63) / 64;
    const long long k = blockIdx.x;
    const long long T = *a.tour.nt;
    if (k >= nsb * T) return;
    const int t = (int)(k / nsb);
    const long long scen = (k - (long long)t * nsb) * 64 + threadIdx.x;
    if (scen >= a.S) return;
    const int64_t ab = tour_abase(a.tour.tptr, t);
    const int n = (int)(a.tour.tptr[t + 1] - a.tour.tptr[t]);
    const int64_t *rowoff = a.tour.rowoff + ab;
    const char *dem = reinterpret_cast<const char *>(a.demand + scen);
    int P = 0, Ps = 0, s = 0;
    for (int i = 1; i <= n; ++i) {
        const uint32_t q = *(const uint16_t *)(dem + rowoff[i]);
        P += (int)q;
        while (s < i && P - Ps > a.Q) {
            ++s;
            Ps += *(const uint16_t *)(dem + rowoff[s]);
        }
        // a negative int16 demand (bit 15) gets an empty window: reported as infeasible
        mask[(ab + i) * mask_ld + scen] = (int16_t)((q & 0x8000u) ? i : s);
    }
}

// One lane per scenario: g_i = w_i + min of g over [mask_i, i - 1], scanning the window in a
// 64-entry history of g per lane in LDS. A window longer than 63 states sends the scenario to
// the general kernel (cost marked kCostOvf); an empty window reports an infeasible demand.
__global__ __launch_bounds__(64) void split_masked_dp_kernel(EvalArgs a, const int16_t *mask,
                                                             long long mask_ld)
{
    __shared__ int ring[64][64];
    const int lane = threadIdx.x;
    const long long nsb = (a.S + 63) / 64;
    const long long k = blockIdx.x;
    const long long T = *a.tour.nt;
    if (k >= nsb * T) return;
    const int t = (int)(k / nsb);
    const long long scen_raw = (k - (long long)t * nsb) * 64 + lane;
    const bool active = scen_raw < a.S;
    const long long scen = active ? scen_raw : a.S - 1;
    const int64_t ab = tour_abase(a.tour.tptr, t);
    const int n = (int)(a.tour.tptr[t + 1] - a.tour.tptr[t]);
    const int32_t *w = a.tour.w + ab;
    bool err = false, ovf = false;
    int g = w[0];
    ring[0][lane] = g;
    for (int i = 1; i <= n; ++i) {
        int s = mask[(ab + i) * mask_ld + scen];
        err |= s >= i;
        ovf |= i - s > 63;
        if (s < i - 63) s = i - 63;
        // uniform trip count: the longest window of the wavefront (at most 63)
        int len = i - s;
        for (int off = 32; off > 0; off >>= 1) len = max(len, __shfl_xor(len, off, 64));
        int m = kInf;
        for (int d = 1; d <= len; ++d) {
            const int p = i - d;
            if (p >= s) m = min(m, ring[p & 63][lane]);
        }
        g = w[i] + m;
        ring[i & 63][lane] = g;
    }
    item_costs(a.sums, t, scen_raw >> 6, active && !ovf && !err ? (uint32_t)g : 0u);
    if (!active) return;
    if (ovf) {
        a.cost[(long long)t * a.ldc + scen] = kCostOvf;
        atomicAdd(&a.stats[t].ovf_count, 1);
        a.ctl->ovf_total = 1;
    } else if (err) {
        atomicOr(&a.stats[t].err_demand, 1);
    } else {
        a.cost[(long long)t * a.ldc + scen] = g;
    }
}

// ------------------------------------------------------------------------- scratch

// Fixed device scratch of the allocation-free evaluation (split_eval_noalloc): every per-call
// device buffer of a one-tour evaluation (staged tour, per-position arrays, result block,
// counters, cost sums) is carved from it. Each GPU holds its own copy for the life of the
// process; its device address is looked up once per device, with that device current.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

hipError_t scratch_address(int device, void **out)
{
    static std::mutex mu;
    static void *addr[kMaxScratchDevices] = {};
    *out = nullptr;
    if (device < 0 || device >= kMaxScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device) return hipErrorInvalidDevice;  // the caller makes `device` current
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = p;
    }
    *out = addr[device];
    return hipSuccess;
}

// ------------------------------------------------------------------------- launchers

hipError_t launch_prep(const PrepArgs &a, hipStream_t stream)
{
    hipLaunchKernelGGL(split_prep_kernel, dim3(a.tour.T_grid), dim3(a.threads), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_lane(const EvalArgs &a, hipStream_t stream)
{
    if (a.lane_block == 0)
        hipLaunchKernelGGL(split_lane_kernel<0>, dim3((unsigned)a.lane_grid), dim3(64), 0, stream,
                           a);
    else if (a.lane_block == 8)
        hipLaunchKernelGGL(split_lane_kernel<8>, dim3((unsigned)a.lane_grid), dim3(64), 0, stream,
                           a);
    else
        hipLaunchKernelGGL(split_lane_kernel<16>, dim3((unsigned)a.lane_grid), dim3(64), 0,
                           stream, a);
    return hipGetLastError();
}

static size_t wave_lds_bytes(int maxn) { return sizeof(int32_t) * 2 * ((size_t)maxn + 1); }

// Dynamic LDS beyond the default 64 KiB (tours near the maximum length) must be opted into.
static hipError_t wave_lds_allow(size_t bytes)
{
    if (bytes <= 65536) return hipSuccess;
    return hipFuncSetAttribute((const void *)split_wave_kernel,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

hipError_t launch_small(const SmallArgs &a, hipStream_t stream)
{
    hipLaunchKernelGGL(split_small_kernel, dim3((unsigned)((a.S + kSmallPer - 1) / kSmallPer)),
                       dim3(kSmallPer), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_pair(const EvalArgs &a, hipStream_t stream)
{
    const long long items = (a.S + 63) / 64 * a.tour.T_grid;
    hipLaunchKernelGGL(split_pair_kernel, dim3((unsigned)items), dim3(128), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_wave_all(const EvalArgs &a, hipStream_t stream)
{
    hipError_t e = wave_lds_allow(wave_lds_bytes(a.maxn));
    if (e != hipSuccess) return e;
    const long long work = a.S * a.tour.T_grid;
    const long long nb = work < a.wave_grid ? work : a.wave_grid;
    hipLaunchKernelGGL(split_wave_kernel, dim3((unsigned)nb), dim3(64), wave_lds_bytes(a.maxn), stream,
                       a);
    return hipGetLastError();
}

hipError_t launch_tail(const EvalArgs &a, hipStream_t stream)
{
    const long long work = (a.S + 63) / 64 * a.tour.T_grid;
    const long long nb = work < a.tail_grid ? work : a.tail_grid;
    hipLaunchKernelGGL(split_tail_kernel, dim3((unsigned)nb), dim3(64 * kTailWaves), 0,
                       stream, a);
    return hipGetLastError();
}

hipError_t launch_mask(const EvalArgs &a, int16_t *mask, long long mask_ld, hipStream_t stream)
{
    const long long items = (a.S + 63) / 64 * a.tour.T_grid;
    hipLaunchKernelGGL(split_mask_kernel, dim3((unsigned)items), dim3(64), 0, stream, a, mask,
                       mask_ld);
    return hipGetLastError();
}

hipError_t launch_masked_dp(const EvalArgs &a, const int16_t *mask, long long mask_ld,
                            hipStream_t stream)
{
    const long long items = (a.S + 63) / 64 * a.tour.T_grid;
    hipLaunchKernelGGL(split_masked_dp_kernel, dim3((unsigned)items), dim3(64), 0, stream, a,
                       mask, mask_ld);
    return hipGetLastError();
}

const char *mask_kernel_name() { return "split_mask_kernel+split_masked_dp_kernel"; }

const char *lane_kernel_name() { return "split_lane_kernel"; }
const char *pair_kernel_name() { return "split_pair_kernel"; }
const char *tail_kernel_name() { return "split_tail_kernel"; }
const char *wave_kernel_name() { return "split_wave_kernel"; }

}  // namespace splitgpu
