// fcfs.hip -- the per-request variant of the plan score: first come, first
// served inside each group, every request with its own SLO.  Interface:
// qlm_fcfs_* in include/qlm.h.
//
// Request r (r = 0 the first to arrive) of the group i at position j of queue
// g has ahead of it the groups before j and the r earlier requests of group i
// (Sec. 4 request groups are served first come, first served; Sec. 6, Eq.
// output_token_dist counts every request ahead), and carries its own TTFT SLO
// (Sec. 3, Definition "SLO"):
//
//   E[W_r]  = A / Theta_g + K + r (mu_i / Theta_g)
//   SD[W_r] = sqrt(V + r sigma_i^2) / Theta_g
//   P_r     = Q((slo_r - E[W_r]) / SD[W_r]),  [E[W_r] > slo_r] at SD = 0
//   score_p = sum of P_r over every request of the plan
//
// A, V are the tokens and the token variance of the groups ahead of position
// j, K the swap and eviction seconds up to and including it.  At 8192 groups
// of 128 requests a plan holds 1,048,576 requests, each with its own tail: the
// work is arithmetic, one tail per request, and the kernels are laid out for
// that, not for memory traffic.
//
// Screen.  The running sums are per position (one walk of each plan), the
// tails are per request.  Most requests need no tail: a spread is tens of
// seconds, waits and SLOs are hundreds or thousands apart, and where a margin is
// beyond six spreads the tail table holds exactly 0 or 1.  The walk forms, at
// every position, the group's start E[W] = A/Theta + K (double) and its variance
// ahead (single, scaled for the tail table), and compares them with the group's
// earliest and latest SLO: a group whose requests all lie on one side adds 0 or
// its request count.  The others are listed; another kernel takes 64 of them at a
// time, one per lane, and looks at their blocks of 32 requests in the same way; the
// blocks that remain are listed again, and 64 of those are evaluated at
// a time, a block per lane: per request a margin in double, a variance in single
// and one read of the normal-tail table.  (8192 groups of 128 requests, random
// plans: 14% of the groups and 41% of their blocks remain.)
//
// The walk reads the plans slot-major with every lane (plan) of a wavefront at
// the same slot, so its reads are coalesced.  It is cut into segments of 128
// slots (32 or 64 for few plans): k_fseg sums each segment's trailing queue piece, k_fstart chains the
// pieces into each segment's starting sums, and k_fwalk walks each segment again
// from them.
//
// Sums.  A block's terms but the first are added in single precision (31 terms at
// most), then the first in double; the sum joins the plan's over the segment as a
// 64-bit fixed-point number, rounded to the nearest, so that the order in which
// blocks are evaluated changes no bit.  The point lies as low as the number of
// requests allows (a million: 2^-41, the last bit of a double-precision sum of
// 4096); the segments' sums are added in order, in double.
//
// Screening bound, per request: table error below 2.2e-6; single-precision
// rounding of the cell coordinate, of the line's evaluation, of the margin and
// of the variance below 1.7e-6; the sum of at most 32 terms in single
// precision below 1.9e-6 per term; the rounding of a sum to fixed point below 1e-10
// (2^-34, with 2^28 requests or more); so |screened - exact| <= 8e-6 per request.
// The margin is formed in double from the start E[W], whose rounding stays
// below 2^-50 E[W_r]: negligible while E[W_r] <= 2^30 SD[W_r] (true of any
// plan whose variances are not zero or vanishingly small).  A request with
// SD = 0 at r = 0 (a queue's first group, or one behind groups without
// variance) is decided by the sign of its margin, the exact comparison with the
// oracle's E[W] (formed in the oracle's order: where a segment starts with
// nothing varying ahead, its sums are formed again from the queue's first slot);
// a group without variance there is compared exactly throughout.
//
// Exact argmin.  Plans whose screened score is within twice the bound of the
// lowest are re-scored exactly (k_fexact: one workgroup per queue, the running
// sums rippled from lane to lane in position order, each request's term in
// double with erfc, its 16 wavefronts over slices of every group's requests),
// and the lowest exact score, the lowest index on ties, wins.
//
// Kernels
//   k_fprep     per group: clamped count, request offset, statistics; the
//               request total; per instance: Theta, the variance scale, class
//               and first model; k_fblocks: each group's and block's first and
//               last SLO
//   k_fseg      one lane per plan, one wavefront per (64 plans, segment):
//               each segment's trailing queue piece
//   k_fstart    one lane per plan: the sums at each segment's first slot
//   k_fwalk     as k_fseg: the walk, and the list of the groups that are not sure
//   k_ftails    one workgroup per (64 plans, segment): the listed groups' blocks
//               and tails
//   k_fsum      the segments' sums -> screened plan scores, and the per-block
//               minimum
//   k_fselect   the plans within the bound of the lowest -> candidates
//   k_fexact    one workgroup per (candidate, queue): exact queue scores
//   k_fpick / k_fplan   exact plan scores; the lowest (score, index)
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "internal.h"
#include "qlm.h"
#include "ripple.h"
#include "tail.h"

namespace {

using qlm_internal::check_plans;
using qlm_internal::check_problem;
using qlm_internal::fail;
using qlm_internal::hip_fail;
using qlm_ripple::from_left;
using qlm_ripple::from_left0;
using qlm_ripple::lane_value;
using qlm_ripple::wave_id;

constexpr int kWave = 64;
constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kSeg = 128;                   // most slots per segment of the queue walks
constexpr int kMinSeg = 32;                 // and fewest (segment_of)
constexpr int kSegThreads = 1024;           // k_fseg, k_fwalk: at most 16 wavefronts a workgroup
constexpr int kSegWaves = kSegThreads / kWave;
constexpr int kSegBlocks = 230;             // workgroups that (nearly) every CU has one of
constexpr size_t kSegLdsLimit = 160 * 1024; // LDS of one workgroup
constexpr int kPrepThreads = 256;
constexpr int kReqBlk = 32;                 // most requests of a block of a group
constexpr int kHalf = 16;                   // of which so many SLOs are staged at a time
constexpr int kEval = 4;                    // and so many evaluated at least
constexpr int kSub = 8;                     // slots of a k_fwalk batch
constexpr int kTailWaves = 4;               // wavefronts of a k_ftails workgroup
constexpr int kBounds = 2;                  // blocks whose bounds are read at a time
constexpr int kShare = 2048;                // groups of one, while the list is that long
constexpr int kBlockList = 2 * kWave;       // blocks a wavefront's list holds
constexpr int kMaxFcfsGroups = 1 << 16;
constexpr int kMaxFcfsInstances = 4096;
constexpr int kSumBlocks = 1024;            // k_fsum blocks (per-block minima)
constexpr int kExactBlocks = 256;
constexpr int kPickThreads = 256;
constexpr uint32_t kCountMask = (1u << 21) - 1u;
constexpr double kEpsP = 8e-6;              // screening bound per request
constexpr int64_t kMaxRequests = (int64_t)1 << 31;
constexpr size_t kChunkBudget = (size_t)1 << 30;  // bytes of lists and segment sums per chunk
// Tail cells beyond which a tail is surely in an end cell (exactly 0 or 1): the
// table's half width, 512, and room for the rounding of margin and spread.
constexpr float kSureCells = 516.0f;
constexpr int kFixBits = 62;                // bits of a segment's score below its sign

// Per group, built once per call: for the walks (the count clamped to 21 bits,
// the model clamped to [0, M), the bounds of the group's SLOs) in 16 bytes, so
// that a table of 8192 groups fits LDS.  The bounds are the upper halves of
// floats, rounded outwards (a sure side may be missed for it, never mistaken) ...
struct FGrp {
    float mu, var;
    uint32_t cm;                // count | model << 21
    uint32_t bounds;            // upper half of the lowest SLO | of the highest << 16
};
__device__ inline uint32_t grp_count(const FGrp &g) { return g.cm & kCountMask; }
__device__ inline int grp_model(const FGrp &g) { return (int)(g.cm >> 21); }
__device__ inline float grp_smin(const FGrp &g) { return __uint_as_float(g.bounds << 16); }
__device__ inline float grp_smax(const FGrp &g) { return __uint_as_float(g.bounds & 0xFFFF0000u); }

// ... and for the requests: where their SLOs start, how many are scored (clamped to
// n_requests) with how many a block holds (blocks_of) above, and the group's
// statistics again: k_ftails reads 64 groups' at a time, in one read of 16 bytes.
struct alignas(16) FReq {
    uint32_t first, np;
    float mu, var;
};
__device__ inline int req_count(const FReq &r) { return (int)(r.np & kCountMask); }
__device__ inline int req_block(const FReq &r) { return (int)(r.np >> 21); }

// The blocks of n requests: as few as hold them in 32 each, and of one size (the
// last may be smaller).  A wavefront evaluates 64 blocks in as many steps as the
// largest has requests, so 33 requests are two blocks of 17, not one of 32 and one
// of 1.
__device__ inline int blocks_of(int n) { return (n + kReqBlk - 1) / kReqBlk; }

// Per instance, for the walks: Theta, its reciprocal (for what need not be exact),
// the table scale over Theta^2, the class
// clamped to [0, C), the model loaded at the start (-1: none).
struct FInst {
    double theta, inv, vscale;
    int32_t cls, m0;
};

// A listed group of a plan: the start E[W] of its first request, its variance
// ahead V / Theta^2 times the table's scale, group | lane of the plan << 16.
// Its queue is in a list beside.
struct FEntry {
    double c0;
    float v0;
    uint32_t id;
};

// Sums over the slots of one segment of a plan that belong to the queue open
// at the segment's end (tokens, variance, fixed costs), whether that queue
// starts inside the segment, and the queue open at the segment's start.
struct Piece {
    double A, V, K;
    int32_t head, q0;
};

// The running sums at a segment's first slot (those of its queue so far).
struct Start {
    double A, V, K;
    int32_t pad[2];
};

struct FArgs {
    int32_t G, I, M, C;
    const int32_t *grp_count;
    const float *grp_mu, *grp_var;
    const int32_t *grp_model;
    const float *inst_tput;
    const int32_t *inst_class, *inst_model0;
    const float *swap_cost;
    float evict_cost;
    int64_t P, ld;
    const int32_t *perm, *qoff;
    const uint32_t *evict_bits;
    const float *req_slo;
    int64_t n_req;
    // workspace
    FGrp *grp;                // [G]
    FReq *req;                // [G]
    FInst *inst;              // [I]
    float2 *blk;              // lowest and highest SLO of each block (block_of)
    float *slo;               // [kReqBlk] SLOs of each block, +inf past its last
    double *nreq;             // [1] requests scored
    FEntry *list;             // [tiles][nseg][kSeg * 64] the listed groups
    uint16_t *listq;          // and their queues
    int32_t *listn;           // [tiles][nseg] how many
    Piece *piece;             // [nseg][chunk]
    Start *start;             // [nseg][chunk]
    int64_t *part;            // [nseg][chunk] the segments' screened scores, in fixed point
    double *F;                // [P] screened scores
    double *bmin;             // [kSumBlocks]
    int32_t *ncand;           // [1]
    int64_t *cand;            // [P]
    double *Q;                // [P][I] exact queue scores
    double *parts;            // [2 kExactBlocks] their sums of sixteen slices, when tasks are shared
    int64_t chunk;
    int32_t seg, nseg;        // slots per segment, segments of a plan
    int32_t fix_bits;         // bits after the point of a segment's score
    double fix, unfix;        // 2^fix_bits and 2^-fix_bits
};

__device__ inline int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Block b of a group whose requests start at `first`, group i, in FArgs::blk: a
// group of n requests from `first` on has at most floor(n / 32) + 1 blocks, so
// the groups' ranges do not overlap.
__device__ inline int64_t block_of(uint32_t first, int i, int b)
{
    return (int64_t)(first / kReqBlk) + i + b;
}

__device__ inline double wave_min(double v)
{
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, kWave));
    return v;
}

// (score, index) is better than (s2, i2): lower score, then lower index; a NaN
// score is never better.
__device__ inline bool better(double s, int64_t i, double s2, int64_t i2)
{
    return s < s2 || (s == s2 && i < i2);
}

#pragma clang fp contract(off)

// ---------------------------------------------------------------------------
// Per-call tables

// Clamped counts, request offsets, group statistics, the request total, the
// instance table.  A workgroup takes 256 groups and adds up every count before
// them itself, coalesced and all in flight: 8192 groups take 6.7 us on 32
// workgroups, and took 48 in one workgroup that scanned them.
__global__ __launch_bounds__(kPrepThreads) void k_fprep(FArgs a)
{
    __shared__ int64_t part[kPrepThreads / kWave], mine[kPrepThreads / kWave];
    const int t = threadIdx.x, lane = t & (kWave - 1), w = wave_id();
    const int b0 = (int)blockIdx.x * kPrepThreads;
    int64_t before = 0;
#pragma unroll 8
    for (int k = t; k < b0; k += kPrepThreads)
        before += (int64_t)((uint32_t)a.grp_count[k] & kCountMask);
    const int i = b0 + t;
    const int64_t want = i < a.G ? (int64_t)((uint32_t)a.grp_count[i] & kCountMask) : 0;
    int64_t off = want;                        // inclusive scan over the wavefront
    for (int o = 1; o < kWave; o <<= 1) {
        const int64_t y = __shfl_up(off, o, kWave);
        if (lane >= o) off += y;
    }
    for (int o = kWave / 2; o > 0; o >>= 1) before += __shfl_xor(before, o, kWave);
    if (lane == kWave - 1) mine[w] = off;
    if (lane == 0) part[w] = before;
    __syncthreads();
    off -= want;
    for (int k = 0; k < kPrepThreads / kWave; ++k) off += part[k] + (k < w ? mine[k] : 0);
    if (i < a.G) {
        const int64_t lo = off < a.n_req ? off : a.n_req;
        const int64_t hi = off + want < a.n_req ? off + want : a.n_req;
        FGrp g;
        g.mu = a.grp_mu[i];
        g.var = a.grp_var[i];
        g.cm = (uint32_t)want | ((uint32_t)clampi(a.grp_model[i], 0, a.M - 1) << 21);
        g.bounds = 0x7F80FF80u;                // none sure, before k_fblocks (-inf, inf)
        a.grp[i] = g;
        FReq r;
        r.first = (uint32_t)lo;
        const uint32_t n = (uint32_t)(hi - lo);
        const uint32_t nb = (uint32_t)max(blocks_of((int)n), 1);
        r.np = n | ((n + nb - 1u) / nb << 21);
        r.mu = g.mu;
        r.var = g.var;
        a.req[i] = r;
        if (i == a.G - 1) {
            a.nreq[0] = (double)hi;
            a.ncand[0] = 0;
        }
    }
    for (int q = i; q < a.I; q += (int)gridDim.x * kPrepThreads) {
        FInst v;
        v.theta = (double)a.inst_tput[q];
        v.inv = 1.0 / v.theta;
        v.vscale = qlm_tail::kVarScale / (v.theta * v.theta);
        v.cls = clampi(a.inst_class[q], 0, a.C - 1);
        v.m0 = a.inst_model0 ? clampi(a.inst_model0[q], -1, a.M - 1) : -1;
        a.inst[q] = v;
    }
}

// The lowest and highest SLO of every block of a group's requests and of the
// group, and the blocks' SLOs, each block in a line of its own (128 bytes), with
// +inf after its last: a request that is never late.  One wavefront per group, half
// of it per block.
__global__ __launch_bounds__(kThreads) void k_fblocks(FArgs a)
{
    const int i = (int)blockIdx.x * kWaves + wave_id();
    if (i >= a.G) return;
    const int lane = threadIdx.x & (kWave - 1);
    const FReq q = a.req[i];
    const int n = req_count(q), per = req_block(q), nb = blocks_of(n);
    const int j = lane & (kReqBlk - 1);
    float gmin = INFINITY, gmax = -INFINITY;
    for (int b0 = 0; b0 < nb; b0 += kWave / kReqBlk) {
        const int b = b0 + lane / kReqBlk;
        const int r = b * per + j;
        float lo = INFINITY, hi = -INFINITY, v = INFINITY;
        if (j < per && r < n) {
            v = a.req_slo[q.first + r];
            lo = v == v ? v : -INFINITY;
            hi = v == v ? v : INFINITY;
        }
        const int64_t at = block_of(q.first, i, b);
        if (b < nb) a.slo[at * kReqBlk + j] = v;
        for (int o = kReqBlk / 2; o > 0; o >>= 1) {
            lo = fminf(lo, __shfl_xor(lo, o, kWave));
            hi = fmaxf(hi, __shfl_xor(hi, o, kWave));
        }
        if (j == 0 && b < nb) a.blk[at] = make_float2(lo, hi);
        gmin = fminf(gmin, fminf(lo, __shfl_xor(lo, kReqBlk, kWave)));
        gmax = fmaxf(gmax, fmaxf(hi, __shfl_xor(hi, kReqBlk, kWave)));
    }
    if (lane == 0) {
        if (!(a.grp[i].mu >= 0.0f)) {
            gmin = -INFINITY;
            gmax = INFINITY;
        }
        // outwards: the upper half as it is rounds towards zero
        uint32_t lo = __float_as_uint(gmin), hi = __float_as_uint(gmax);
        if ((lo & 0x80000000u) && (lo & 0xFFFFu)) lo += 0x10000u;
        if (!(hi & 0x80000000u) && (hi & 0xFFFFu)) hi += 0x10000u;
        a.grp[i].bounds = (lo >> 16) | (hi & 0xFFFF0000u);
    }
}

// ---------------------------------------------------------------------------
// Screen

// The walk of one plan's slots in order, one lane per plan, every lane of a
// wavefront at the same slot (so the reads of the plan rows are coalesced).
// Queues are contiguous slot ranges; at a queue's first slot the running sums
// restart.  The sums and costs are formed with the oracle's operations in the
// oracle's order.
constexpr int kAhead = 3;      // queue boundaries a walk holds beyond the open queue's
static_assert(kAhead == 3, "open_queue settles nh and three boundaries");

// x / y, y's reciprocal r correctly rounded: a product and two corrections by its
// exact remainder give the correctly rounded quotient (Markstein's theorem; x and
// y are products and copies of single-precision numbers, far from overflow and
// underflow).  Half of a division's instructions.
__device__ inline double quotient(double x, double y, double r)
{
    double q = x * r;
    q = fma(fma(-q, y, x), r, q);
    return fma(fma(-q, y, x), r, q);
}

struct Walk {
    int q, nh;                 // open queue, first slot of the next queue
    int nx[kAhead];            // qoff[q + 2 + j] (j < kAhead), -1 where not read
    double theta, inv, vscale;
    int cls, prev;
    double A, V, K;
};

__device__ inline void set_queue(const FInst *inst, int q, Walk &w)
{
    const FInst v = inst[q];
    w.q = q;
    w.theta = v.theta;
    w.inv = v.inv;
    w.vscale = v.vscale;
    w.cls = v.cls;
    w.prev = v.m0;
    w.A = w.V = w.K = 0.0;
}

// Open queue q: its end boundary and the next kAhead ones are read together
// and waited for at once, so that no later read of the walk waits behind
// them (memory reads complete in order), and the switches to the next
// queues read nothing.  inst: the per-instance table (in LDS or global
// memory).
__device__ inline void open_queue(const FArgs &a, const FInst *inst, int64_t p, int q, Walk &w)
{
    w.nh = a.qoff[(int64_t)(q + 1) * a.ld + p];
#pragma unroll
    for (int j = 0; j < kAhead; ++j)
        w.nx[j] = q + 2 + j <= a.I ? a.qoff[(int64_t)(q + 2 + j) * a.ld + p] : -1;
    asm volatile("" ::"v"(w.nh), "v"(w.nx[0]), "v"(w.nx[1]), "v"(w.nx[2]));
    set_queue(inst, q, w);
}

// Slot s lies past the open queue: open the queue that holds it.
__device__ inline void next_queue(const FArgs &a, const FInst *inst, int64_t p, int s, Walk &w)
{
    if (w.q + 1 < a.I && w.nx[0] >= 0 && (w.q + 2 >= a.I || w.nx[0] > s)) {
        // the next queue (qoff[q+1] <= s < qoff[q+2]), from the boundaries held
        // (a negative one is taken as not held)
        w.nh = w.nx[0];
#pragma unroll
        for (int j = 0; j + 1 < kAhead; ++j) w.nx[j] = w.nx[j + 1];
        w.nx[kAhead - 1] = -1;
        set_queue(inst, w.q + 1, w);
    } else {
        int q = w.q;
        while (q + 1 < a.I && a.qoff[(int64_t)(q + 1) * a.ld + p] <= s) ++q;
        open_queue(a, inst, p, q, w);
    }
}

// The queue holding slot s: the largest q with qoff[q] <= s.
__device__ inline int queue_at(const FArgs &a, int64_t p, int s)
{
    int lo = 0, hi = a.I - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.qoff[(int64_t)mid * a.ld + p] <= s)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Slots [s0, s1) of the walk, B at a time: a batch's reads (group ids, one
// eviction word, the group records) are issued together, and with kPipe the
// next batch's reads are issued while a batch is walked.  Batches start at
// multiples of B (so one eviction word covers a batch); slots before s0 are
// passed over.  At a queue's first slot (the next queue's first slot reached,
// empty queues skipped) the sums restart; then the slot's model-change and
// eviction costs; then the group's tokens and variance join the sums.  Ids
// out of range (a malformed plan) are skipped.  The group records and swap
// costs are read from grp and swc: the problem's own arrays, or copies in LDS.
template <int B>
struct Batch {
    int ids[B];
    uint32_t ev;
};

template <int B>
__device__ inline void batch_ids(const FArgs &a, int64_t p, int sb, int s1, Batch<B> &b)
{
    // (rows past s1 clamp to its last one: the walk stops at s1, and no read
    // waits behind a conditional one)
#pragma unroll
    for (int u = 0; u < B; ++u) b.ids[u] = a.perm[(int64_t)min(sb + u, s1 - 1) * a.ld + p];
    b.ev = a.evict_bits ? a.evict_bits[(int64_t)(sb >> 5) * a.ld + p] : 0u;
}

// (every gather is issued, at a clamped id, so that all of a batch's are in
// flight together; the walk does not use the record of an id out of range)
template <int B>
__device__ inline void batch_groups(const FArgs &a, const FGrp *grp, const Batch<B> &b, FGrp *gr)
{
#pragma unroll
    for (int u = 0; u < B; ++u) gr[u] = grp[clampi(b.ids[u], 0, a.G - 1)];
}

template <int B, bool kPipe>
__device__ inline void walk(const FArgs &a, const FGrp *grp, const float *swc, const FInst *inst,
                            int64_t p, int s0, int s1, Walk &w, bool *fresh)
{
    static_assert(B <= 32 && (B & (B - 1)) == 0, "a batch lies in one eviction word");
    if (s0 >= s1) return;
    int sb = s0 & ~(B - 1);
    Batch<B> cur;
    FGrp gr[B];
    batch_ids<B>(a, p, sb, s1, cur);
    batch_groups<B>(a, grp, cur, gr);
    for (; sb < s1; sb += B) {
        Batch<B> nxt;
        const bool more = sb + B < s1;
        if (kPipe && more) batch_ids<B>(a, p, sb + B, s1, nxt);
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int s = sb + u;
            if (s < s0) continue;
            if (s >= s1) break;
            if (s >= w.nh) {
                next_queue(a, inst, p, s, w);
                *fresh = true;
            }
            const int i = cur.ids[u];
            if (i < 0 || i >= a.G) continue;
            const int m = grp_model(gr[u]);
            if (w.prev >= 0 && w.prev != m && a.swap_cost)
                w.K += (double)swc[((int64_t)w.cls * a.M + w.prev) * a.M + m];
            if ((cur.ev >> (s & 31)) & 1u) w.K += (double)a.evict_cost;
            const double n = (double)grp_count(gr[u]);
            w.A += n * (double)gr[u].mu;
            w.V += n * (double)gr[u].var;
            w.prev = m;
        }
        if (more) {
            if (kPipe)
                cur = nxt;
            else
                batch_ids<B>(a, p, sb + B, s1, cur);
            batch_groups<B>(a, grp, cur, gr);
        }
    }
}

// Bytes of the swap-cost table, rounded up to 16.
__device__ __host__ inline size_t swap_bytes(const FArgs &a)
{
    return a.swap_cost ? ((sizeof(float) * (size_t)a.C * a.M * a.M + 15) & ~(size_t)15) : 0;
}

// Copies of the swap costs and the instance table in LDS at t (swap_bytes(a)
// then I FInst); every thread of the workgroup takes part.
__device__ inline void stage_tables(const FArgs &a, unsigned char *t, int nthreads,
                                    const float **swc, const FInst **inst)
{
    float *sc = reinterpret_cast<float *>(t);
    FInst *si = reinterpret_cast<FInst *>(t + swap_bytes(a));
    if (a.swap_cost)
        for (int k = threadIdx.x; k < a.C * a.M * a.M; k += nthreads) sc[k] = a.swap_cost[k];
    for (int q = threadIdx.x; q < a.I; q += nthreads) si[q] = a.inst[q];
    *swc = a.swap_cost ? sc : nullptr;
    *inst = si;
}

// The group records, the swap costs and the instance table in LDS at t; every
// thread of a workgroup takes part.
__device__ inline void stage_groups(const FArgs &a, unsigned char *t, const FGrp **grp,
                                    const float **swc, const FInst **inst)
{
    FGrp *sg = reinterpret_cast<FGrp *>(t);
    const int nthreads = (int)blockDim.x;
    for (int i = threadIdx.x; i < a.G; i += nthreads) sg[i] = a.grp[i];
    stage_tables(a, t + sizeof(FGrp) * (size_t)a.G, nthreads, swc, inst);
    __syncthreads();
    *grp = sg;
}

// Grid: ceil(chunk/64) tiles x ceil(nseg/wavefronts); wavefront = (tile, segment).
// Pass 1: each segment's trailing piece (the sums of its last queue over the
// segment's slots).  With kLds the group records, the swap costs and the
// instance table are first copied into LDS (dynamic: 16 G bytes, the costs,
// 32 I bytes), so that every slot's gather is an LDS read, not a random L2
// access.
template <bool kLds>
__global__ __launch_bounds__(kSegThreads) void k_fseg(FArgs a, int64_t p0, int64_t pc)
{
    extern __shared__ __align__(16) unsigned char fseg_lds[];
    const FGrp *grp = a.grp;
    const float *swc = a.swap_cost;
    const FInst *inst = a.inst;
    if (kLds) stage_groups(a, fseg_lds, &grp, &swc, &inst);
    const int nseg = a.nseg;
    const int waves = (int)(blockDim.x / kWave);
    const int sq = (nseg + waves - 1) / waves;
    const int64_t tile = blockIdx.x / sq;
    const int k = (int)(blockIdx.x % sq) * waves + wave_id();
    if (k >= nseg) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t col = tile * kWave + lane;
    const bool on = col < pc;
    const int64_t p = p0 + (on ? col : pc - 1);
    const int s0 = k * a.seg, s1 = min(a.G, s0 + a.seg);
    Walk w;
    const int q0 = queue_at(a, p, s0);
    open_queue(a, inst, p, q0, w);
    bool fresh = s0 == 0 || a.qoff[(int64_t)q0 * a.ld + p] >= s0;
    if (!fresh) {
        const int i = a.perm[(int64_t)(s0 - 1) * a.ld + p];
        if (i >= 0 && i < a.G) w.prev = grp_model(grp[i]);
    }
    walk<8, true>(a, grp, swc, inst, p, s0, s1, w, &fresh);
    if (on) {
        Piece t;
        t.A = w.A;
        t.V = w.V;
        t.K = w.K;
        t.head = fresh ? 1 : 0;
        t.q0 = q0;
        a.piece[(int64_t)k * a.chunk + col] = t;
    }
}

// Pass 2: one lane per plan, the segments in order: the sums at each
// segment's first slot.  (Eight segments' pieces are read together; one at a
// time, 64 segments took 26 us.)
__global__ __launch_bounds__(kWave) void k_fstart(FArgs a, int64_t pc)
{
    const int64_t col = (int64_t)blockIdx.x * kWave + threadIdx.x;
    if (col >= pc) return;
    const int nseg = a.nseg;
    double A = 0.0, V = 0.0, K = 0.0;
    for (int k0 = 0; k0 < nseg; k0 += 8) {
        Piece t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = a.piece[(int64_t)min(k0 + u, nseg - 1) * a.chunk + col];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (k0 + u >= nseg) break;
            Start st;
            st.A = A;
            st.V = V;
            st.K = K;
            st.pad[0] = st.pad[1] = 0;
            a.start[(int64_t)(k0 + u) * a.chunk + col] = st;
            A = t[u].head ? t[u].A : A + t[u].A;
            V = t[u].head ? t[u].V : V + t[u].V;
            K = t[u].head ? t[u].K : K + t[u].K;
        }
    }
}

__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// This lane's place among the lanes of a ballot.
__device__ inline int lane_rank(uint64_t mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Requests whose SLOs lie in [smin, smax], whose mean waits lie in [lo, hi] and
// whose scaled variances are at most vmax: whether every tail is exactly 0 or
// every one exactly 1 (a NaN is never sure), and which.
struct Side {
    bool sure, one;
};
__device__ inline Side side_of(float smin, float smax, double lo, double hi, float vmax)
{
    const double early = (double)smin - hi, late = lo - (double)smax;   // (one at most is > 0)
    Side r;
    r.one = late > early;
    r.sure = (float)(r.one ? late : early) * __builtin_amdgcn_rsqf(vmax) >= kSureCells;
    return r;
}

// Pass 3: the walk of one segment of 64 plans, one wavefront.  A queue open at
// the segment's start continues from the sums of pass 2; where nothing varies
// ahead (V = 0) those sums are formed again slot by slot from the queue's
// first slot, so that E[W] is the oracle's bit for bit wherever an exact
// comparison uses it.  Groups whose side is sure add their requests to the
// plan's count here; the others go to the (tile, segment)'s list, one after
// another.  kLds as for k_fseg.
template <bool kLds>
__global__ __launch_bounds__(kSegThreads) void k_fwalk(FArgs a, int64_t p0, int64_t pc)
{
    extern __shared__ __align__(16) unsigned char fseg_lds[];
    const FGrp *grp = a.grp;
    const float *swc = a.swap_cost;
    const FInst *inst = a.inst;
    if (kLds) stage_groups(a, fseg_lds, &grp, &swc, &inst);
    const int nseg = a.nseg;
    const int waves = (int)(blockDim.x / kWave);
    const int sq = (nseg + waves - 1) / waves;
    const int64_t tile = blockIdx.x / sq;
    const int k = (int)(blockIdx.x % sq) * waves + wave_id();
    if (k >= nseg) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t col = tile * kWave + lane;
    const bool on = col < pc;
    const int64_t c = on ? col : pc - 1;
    const int64_t p = p0 + c;
    const int s0 = k * a.seg, s1 = min(a.G, s0 + a.seg);
    Walk w;
    const int q0 = a.piece[(int64_t)k * a.chunk + c].q0;
    open_queue(a, inst, p, q0, w);
    const int b = a.qoff[(int64_t)q0 * a.ld + p];
    if (s0 > 0 && b < s0) {
        const Start st = a.start[(int64_t)k * a.chunk + c];
        if (st.V == 0.0) {
            // nothing varies ahead: form the sums again in the oracle's order
            bool f = false;
            walk<8, true>(a, grp, swc, inst, p, max(b, 0), s0, w, &f);
        } else {
            w.A = st.A;
            w.V = st.V;
            w.K = st.K;
            const int i = a.perm[(int64_t)(s0 - 1) * a.ld + p];
            if (i >= 0 && i < a.G) w.prev = grp_model(grp[i]);
        }
    }
    int sure = 0;                              // requests whose tail is exactly 1 (below 2^29)
    int ng = 0;                                // entries of the list
    FEntry *list = a.list + (tile * nseg + k) * (int64_t)(a.seg * kWave);
    uint16_t *listq = a.listq + (tile * nseg + k) * (int64_t)(a.seg * kWave);
    Batch<kSub> cur, nxt;
    FGrp gr[kSub];
    batch_ids<kSub>(a, p, s0, s1, cur);
    batch_groups<kSub>(a, grp, cur, gr);
    // batches of kSub slots (s0 is a multiple of kSub), the next batch's group
    // ids in flight while one is walked
    for (int sb = s0; sb < s1; sb += kSub) {
        const bool more = sb + kSub < s1;
        if (more) batch_ids<kSub>(a, p, sb + kSub, s1, nxt);
#pragma unroll
        for (int u = 0; u < kSub; ++u) {
            const int s = sb + u;
            if (s >= s1) break;
            if (s >= w.nh) next_queue(a, inst, p, s, w);
            const int i = cur.ids[u];
            bool put = false;
            FEntry e{0.0, 0.0f, 0u};
            if (i >= 0 && i < a.G) {
                const int m = grp_model(gr[u]);
                if (w.prev >= 0 && w.prev != m && a.swap_cost)
                    w.K += (double)swc[((int64_t)w.cls * a.M + w.prev) * a.M + m];
                if ((cur.ev >> (s & 31)) & 1u) w.K += (double)a.evict_cost;
                const double n = (double)grp_count(gr[u]);
                const double mu = (double)gr[u].mu, var = (double)gr[u].var;
                e.c0 = quotient(w.A, w.theta, w.inv) + w.K;
                e.v0 = (float)(w.V * w.vscale);
                e.id = (uint32_t)i | ((uint32_t)lane << 16);
                // (up to where the group after it starts, to within rounding, and
                // the variance ahead there; a group with mu < 0 has no sure side)
                const double tok = n * mu, tvar = n * var;
                w.A += tok;
                w.V += tvar;
                const Side d = side_of(grp_smin(gr[u]), grp_smax(gr[u]), e.c0,
                                       fma(tok, w.inv, e.c0), (float)(w.V * w.vscale));
                put = on && !d.sure && n > 0.0;
                sure += d.sure && d.one ? (int)grp_count(gr[u]) : 0;
                w.prev = m;
            }
            const uint64_t mask = __builtin_amdgcn_ballot_w64(put);
            if (put) {
                const int at = ng + lane_rank(mask);
                list[at] = e;
                listq[at] = (uint16_t)w.q;
            }
            ng += __builtin_popcountll(mask);
        }
        if (more) {
            cur = nxt;
            batch_groups<kSub>(a, grp, cur, gr);
        }
    }
    if (lane == 0) a.listn[tile * nseg + k] = ng;
    if (on) a.part[(int64_t)k * a.chunk + col] = (int64_t)((uint64_t)sure << a.fix_bits);
}

// A wavefront's list of blocks to be evaluated, and the room for their SLOs.  An
// entry, in two halves: the mean wait E[W] of the block's first request and the
// step from one request to the next (double each); the variance ahead of the block
// and its step (single), the block's number, and requests | lane of the plan << 6
// | nothing varies << 12.  Where nothing varies the wait is the group's first
// request's, and the block's first request r of the group stands in place of the
// variance: E[W_r] is formed from them as the oracle forms it.
// The SLOs come 16 of every block at a time, four reads of 16 bytes a lane, four
// neighbouring lanes to a block, and are stored as they come: lane l's read i, of
// block 16 i + l / 4, in place l of row i.  Which of the block's four pieces a lane
// takes turns with l / 16, so that 16 lanes that read one piece of their own blocks
// meet on no bank.  Two rows lie in the list's upper half, which is free once 64
// entries have been read.
struct BlockList {
    uint4 half[2][kBlockList];
    uint4 more[2][kWave];
};
__device__ inline uint4 *slo_row(BlockList &bl, int i)
{
    return i < 2 ? &bl.half[i][kWave] : bl.more[i - 2];
}
__device__ inline uint4 block_half(double x, double y)
{
    return make_uint4((uint32_t)__double2loint(x), (uint32_t)__double2hiint(x),
                      (uint32_t)__double2loint(y), (uint32_t)__double2hiint(y));
}

// A sum as a 64-bit fixed-point number, to the nearest.
__device__ inline unsigned long long fixed_point(const FArgs &a, double x)
{
    return (unsigned long long)__double2ll_rn(x * a.fix);
}

// kN requests of a block, from request h + k0 on (the staging holds those from h):
// their tails added to S, that of the block's first request put into S0.  kFlat:
// blocks where nothing varies are among the lanes'.
template <int kN, bool kFlat>
__device__ __attribute__((always_inline)) inline void eval_step(const float2 *tab, BlockList &bl,
                                                                double eb, double c1, float v0,
                                                                float v1, bool flat, int r0, int h,
                                                                int k0, float &S0, float &S)
{
    const int lane = threadIdx.x & (kWave - 1);
    const uint4 *mine = slo_row(bl, lane >> 4) + 4 * (lane & 15);
    float slo[kN];
#pragma unroll
    for (int c = 0; c < kN / 4; ++c) {
        const uint4 w = mine[(k0 / 4 + c) ^ ((lane >> 2) & 3)];
        slo[4 * c] = __uint_as_float(w.x);
        slo[4 * c + 1] = __uint_as_float(w.y);
        slo[4 * c + 2] = __uint_as_float(w.z);
        slo[4 * c + 3] = __uint_as_float(w.w);
    }
#pragma unroll
    for (int u = 0; u < kN; ++u) {
        const int k = h + k0 + u;
        const float m = (float)fma(-(double)k, c1, (double)slo[u] - eb);
        float q = qlm_tail::q_of(tab, m, fmaf((float)k, v1, v0));
        if (kFlat) {
            const float late = eb + (double)(r0 + k) * c1 > (double)slo[u] ? 1.0f : 0.0f;
            q = flat ? late : q;
        }
        if (k == 0)
            S0 = q;
        else
            S += q;
    }
}

// The list's entries [from, from + n), n <= 64 and from <= 64, one per lane,
// evaluated and added to their plans' sums.  A block's requests are padded with ones
// that are never late, so no lane is masked but those without an entry.
__device__ __attribute__((always_inline)) inline void eval_blocks(const FArgs &a, const float2 *tab,
                                                                  BlockList &bl,
                                                                  unsigned long long *sum, int from,
                                                                  int n)
{
    const int lane = threadIdx.x & (kWave - 1);
    const bool on = lane < n;
    // (with n < 64 the list ends there, from = 0: what the other lanes read is an
    // entry evaluated before or the empty one)
    const uint4 x = bl.half[0][from + lane], y = bl.half[1][from + lane];
    const int piece = (lane ^ (lane >> 4)) & 3, b0 = lane >> 2;
    const float4 *src[kWave / 16];
#pragma unroll
    for (int i = 0; i < kWave / 16; ++i)
        src[i] = reinterpret_cast<const float4 *>(
                     a.slo + (int64_t)bl.half[1][from + 16 * i + b0].z * kReqBlk) + piece;
    const uint32_t what = y.w;
    // the steps of the largest block, in units of kEval
    const int cnt = on ? (int)(what & 63u) : 0;
    int trip = kEval;
#pragma unroll
    for (int b = kReqBlk / 2; b >= kEval; b /= 2)
        trip += __builtin_amdgcn_ballot_w64(cnt > trip - kEval + b) != 0 ? b : 0;
    const double eb = __hiloint2double((int)x.y, (int)x.x), c1 = __hiloint2double((int)x.w, (int)x.z);
    const float v0 = __uint_as_float(y.x), v1 = __uint_as_float(y.y);
    const bool flat = (what >> 12) & 1u;
    const bool any_flat = __builtin_amdgcn_ballot_w64(flat) != 0;
    float4 s[kWave / 16];
#pragma unroll
    for (int i = 0; i < kWave / 16; ++i) s[i] = src[i][0];
    float S0 = 0.0f, S = 0.0f;
#pragma unroll
    for (int h = 0; h < kReqBlk; h += kHalf) {
        if (h >= trip) break;
        wave_sync();
#pragma unroll
        for (int i = 0; i < kWave / 16; ++i)
            slo_row(bl, i)[lane] = make_uint4(__float_as_uint(s[i].x), __float_as_uint(s[i].y),
                                              __float_as_uint(s[i].z), __float_as_uint(s[i].w));
        // (the second half is on its way while the first is evaluated)
        if (h == 0 && trip > kHalf)
#pragma unroll
            for (int i = 0; i < kWave / 16; ++i) s[i] = src[i][kHalf / 4];
        wave_sync();
        const int r0 = (int)y.x, rest = trip - h;
        if (any_flat) {
            for (int k0 = 0; k0 < min(kHalf, rest); k0 += kEval)
                eval_step<kEval, true>(tab, bl, eb, c1, v0, v1, flat, r0, h, k0, S0, S);
        } else if (rest >= kHalf) {
            eval_step<kHalf, false>(tab, bl, eb, c1, v0, v1, flat, r0, h, 0, S0, S);
        } else {
            if (rest >= 8) eval_step<8, false>(tab, bl, eb, c1, v0, v1, flat, r0, h, 0, S0, S);
            if (rest == 12) eval_step<4, false>(tab, bl, eb, c1, v0, v1, flat, r0, h, 8, S0, S);
            if (rest == 4) eval_step<4, false>(tab, bl, eb, c1, v0, v1, flat, r0, h, 0, S0, S);
        }
    }
    if (on) atomicAdd(&sum[(what >> 6) & 63u], fixed_point(a, (double)S0 + (double)S));
}

// Pass 4: the listed groups of one (tile, segment), one workgroup: its wavefronts
// take 64 of them at a time, one per lane, look at their blocks of 32 requests
// and evaluate the blocks that are not sure, 64 at a time.
//
// What the walk, the lists and this replaced: the records of every (group, plan)
// sorted by group in two passes through LDS and memory, so that a wavefront
// could take one group of 64 plans and evaluate all of its requests with the SLOs
// in scalar registers (0.31 + 1.45 ms for 4096 plans of 8192 groups of 128
// requests, however many are sure; the call 2.0).  Here few requests are evaluated:
// 0.10 + 0.16 ms on random plans, the call 0.40.  With spreads as wide as the waits
// nearly all are, and the L1's misses count: a line per lane for the SLOs, one per
// block for its bounds and two per group took the kernel to 3.0 ms; 64 blocks' SLOs
// read as whole lines and passed through LDS, two blocks' bounds and all of a
// group's numbers read at a time leave 1.85 (arithmetic busy 88% of it), the call
// 2.11 to 2.16.  So the sorted form would still be the faster one for groups of 128
// requests that all need their tails, by 4 to 14% (2048 groups), and this is for
// smaller groups (33 requests 0.93 ms for 1.02, 32 3.68 for 4.30 on 16384 plans) and
// wherever a third of the requests are sure.  With the lists in LDS and both passes
// in one kernel its registers left two wavefronts a SIMD: 1.40 ms on random plans.
// Four wavefronts a workgroup: with two or three fewer lists wait for room (6000
// plans of 1000 groups 87 and 91 us, 93 with four, 110 with eight) and the tables
// are copied more often (8192 groups 439 and 431, 417 with four).
__global__ __launch_bounds__(kTailWaves * kWave) __attribute__((amdgpu_waves_per_eu(4))) void k_ftails(
    FArgs a, int64_t pc, uint32_t lists_n)
{
    __shared__ __align__(16) float2 tab[qlm_tail::kCells];
    __shared__ BlockList lists[kTailWaves];
    __shared__ unsigned long long sum[kWave];  // per plan, in fixed point
    const int nseg = a.nseg;
    const int64_t which = blockIdx.x % lists_n;
    const int64_t tile = which / nseg;
    const int k = (int)(which % nseg);
    const int total = min(a.listn[which], a.seg * kWave);
    // of a long list, every share-th workgroup's groups (2048 of them: half as many
    // cost more in tables staged and in last evaluations of a few blocks)
    const int part = (int)(blockIdx.x / lists_n);
    const int share = (total + kShare - 1) / kShare;
    if (part >= share) return;                 // (the same in the whole workgroup)
    const int lane = threadIdx.x & (kWave - 1);
    const FEntry *list = a.list + which * (a.seg * kWave);
    const uint16_t *listq = a.listq + which * (a.seg * kWave);
    int g0 = (part * kTailWaves + wave_id()) * kWave;   // the next groups, their entries read ahead
    FEntry ahead = list[min(g0 + lane, total - 1)];
    uint32_t aheadq = listq[min(g0 + lane, total - 1)];
    qlm_tail::stage(tab, (int)threadIdx.x, kTailWaves * kWave);
    if (threadIdx.x < kWave) sum[threadIdx.x] = 0ull;
    __syncthreads();
    BlockList &bl = lists[wave_id()];
    bl.half[0][lane] = bl.half[1][lane] = make_uint4(0u, 0u, 0u, 0u);
    int nb = 0;                                // entries of the list of blocks
    bool have = false;                         // the groups in hand have blocks left
    int n = 0, bb = 0;                         // this lane's requests; the block in hand
    FEntry e{0.0, 0.0f, 0u};
    uint32_t q = 0u;
    int64_t block = 0;                         // the group's first block
    int per = 1;
    const float2 *blk = a.blk;
    float2 mm[kBounds];                        // the bounds of its next blocks, read ahead
#pragma unroll
    for (int u = 0; u < kBounds; ++u) mm[u] = make_float2(0.0f, 0.0f);
    double c1 = 0.0;
    float v1 = 0.0f;
    bool flat = false;
    unsigned long long ones = 0ull;            // its sure blocks
    for (;;) {
        while (nb < kWave) {
            if (!have) {
                if (g0 >= total) break;
                const bool mine = g0 + lane < total;
                e = ahead;
                q = aheadq;
                g0 += share * kTailWaves * kWave;
                ahead = list[min(g0 + lane, total - 1)];
                aheadq = listq[min(g0 + lane, total - 1)];
                const int i = (int)(e.id & 0xFFFFu);
                const FReq r = a.req[i];
                const FInst in = a.inst[q];
                per = req_block(r);
                c1 = (double)r.mu / in.theta;
                v1 = (float)((double)r.var * in.vscale);
                flat = r.var == 0.0f && e.v0 == 0.0f;
                n = mine ? req_count(r) : 0;
                block = block_of(r.first, i, 0);
                blk = a.blk + block;
#pragma unroll
                for (int u = 0; u < kBounds; ++u) mm[u] = blk[u];
                ones = 0ull;
                bb = 0;
                have = true;
            }
            const int rb = bb * per;
            const float vb = fmaf((float)rb, v1, e.v0);
            const int cb = min(per, n - rb);
            const double ea = e.c0 + (double)rb * c1;
            bool put = false;
            if (rb < n) {
                const double ez = e.c0 + (double)(rb + cb - 1) * c1;
                const Side d = side_of(mm[0].x, mm[0].y, fmin(ea, ez), fmax(ea, ez),
                                       fmaf((float)cb, v1, vb));
                put = !d.sure;
                ones += d.sure && d.one ? (unsigned long long)cb << a.fix_bits : 0ull;
            }
            const uint64_t mask = __builtin_amdgcn_ballot_w64(put);
            if (put) {
                const int to = nb + lane_rank(mask);
                bl.half[0][to] = block_half(flat ? e.c0 : ea, c1);
                bl.half[1][to] = make_uint4(flat ? (uint32_t)rb : __float_as_uint(vb),
                                            __float_as_uint(v1), (uint32_t)(block + bb),
                                            (uint32_t)cb | ((e.id >> 16) << 6) |
                                                (flat ? 1u << 12 : 0u));
            }
            nb += __builtin_popcountll(mask);
            ++bb;
            const bool more = bb * per < n;
#pragma unroll
            for (int u = 0; u + 1 < kBounds; ++u) mm[u] = mm[u + 1];
            if (bb % kBounds == 0 && more)
#pragma unroll
                for (int u = 0; u < kBounds; ++u) mm[u] = blk[bb + u];
            if (__builtin_amdgcn_ballot_w64(more) == 0) {
                if (ones) atomicAdd(&sum[e.id >> 16], ones);
                have = false;
            }
        }
        if (nb == 0) break;
        const int m = min(nb, kWave);
        nb -= m;
        wave_sync();
        eval_blocks(a, tab, bl, sum, nb, m);
        wave_sync();
    }
    __syncthreads();
    const int64_t col = tile * kWave + threadIdx.x;
    if (threadIdx.x < kWave && col < pc) {
        int64_t *score = &a.part[(int64_t)k * a.chunk + col];
        if (share == 1)
            *score += (int64_t)sum[threadIdx.x];
        else
            atomicAdd((unsigned long long *)score, sum[threadIdx.x]);
    }
}

// Screened plan scores of the chunk (the segments' sums in order) and the
// running minimum per block (grid-stride over plans, fixed grid).
__global__ __launch_bounds__(kThreads) void k_fsum(FArgs a, int64_t p0, int64_t pc, int first_chunk)
{
    __shared__ double lmin[kWaves];
    const int nb = a.nseg;
    double mn = first_chunk ? INFINITY : a.bmin[blockIdx.x];
    for (int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x; c < pc;
         c += (int64_t)gridDim.x * kThreads) {
        double s = 0.0;
        // (eight reads in flight: one after another they took 21 us for 64 segments)
        for (int b0 = 0; b0 < nb; b0 += 8) {
            int64_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                v[u] = a.part[(int64_t)min(b0 + u, nb - 1) * a.chunk + c];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += b0 + u < nb ? (double)v[u] * a.unfix : 0.0;
        }
        a.F[p0 + c] = s;
        mn = fmin(mn, s);
    }
    mn = wave_min(mn);
    if ((threadIdx.x & (kWave - 1)) == 0) lmin[threadIdx.x / kWave] = mn;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kWaves; ++w) mn = fmin(mn, lmin[w]);
        a.bmin[blockIdx.x] = mn;
    }
}

// Candidates: plans whose screened score lies within twice the bound of the
// lowest (their exact score can be the lowest), and plans with a NaN score.
// (k_fprep clears the counter; k_fzero does when there is no plan.)
__global__ void k_fzero(FArgs a) { if (threadIdx.x == 0) a.ncand[0] = 0; }

__global__ __launch_bounds__(kThreads) void k_fselect(FArgs a, int nbmin)
{
    __shared__ double smin;
    if (threadIdx.x < kWave) {
        double m = INFINITY;
        for (int b = threadIdx.x; b < nbmin; b += kWave) m = fmin(m, a.bmin[b]);
        m = wave_min(m);
        if (threadIdx.x == 0) smin = m;
    }
    __syncthreads();
    const double lim = smin + 2.0 * kEpsP * a.nreq[0] + 1e-9 * fabs(smin);
    for (int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x; p < a.P;
         p += (int64_t)gridDim.x * kThreads) {
        const double f = a.F[p];
        if (f <= lim || f != f) {
            const int k = atomicAdd(a.ncand, 1);
            a.cand[k] = p;
        }
    }
}

// ---------------------------------------------------------------------------
// Exact scores

// Workgroups over a fixed grid take (candidate k, queue g) tasks; every group's
// requests are cut into 64 slices (consecutive arrivals), four next to each other for
// each of a workgroup's 16 wavefronts (so that groups of a few requests keep as many
// wavefronts busy).  A wavefront walks the queue's positions 64 at a time, one per
// lane; the running sums ripple from lane to lane in position order, then each
// lane forms its slices of its group's requests' terms, and a lane per slice adds
// them in position order.  (Rippled like the running sums, slice after slice, the
// terms took longer than their erfc where many plans are re-scored: 64 plans of 64
// queues 1.00 ms, 0.77 so.)  The queue score is the sum over the wavefronts' first
// slices, second, third and fourth ones, each in order, then of the four (the
// oracle's sum reassociated: equal to within the rounding of a sum of that many
// terms).
// When few tasks are there (one candidate of 64 queues is the usual case) two or
// four workgroups share a task, each with half or a quarter of every wavefront's
// slices, and the sums of sixteen go to `parts` (task_score adds them); the
// additions are the same.  One candidate of 64 queues and 1,048,576 requests: 58
// us on 64 workgroups, 36 on 256.
constexpr int kExactThreads = 1024;
constexpr int kExactWaves = kExactThreads / kWave;
constexpr int kExactSubs = 4;                      // slices per wavefront
constexpr int kExactSlices = kExactWaves * kExactSubs;

// The oracle's terms for one group in double: its requests, their mean wait EW and
// the step from one to the next, the variance ahead and its step.  slice: the sum of
// slice j of the requests (consecutive arrivals), which starts at 0 and adds its P_r
// in arrival order.
struct ExactGroup {
    const float *slo;
    int n;
    double EW, step, V, var;
    __device__ inline double slice(double theta, int j) const
    {
        double slot = 0.0;
        const int r0 = n * j / kExactSlices, r1 = n * (j + 1) / kExactSlices;  // (n < 2^21)
        for (int r = r0; r < r1; ++r) {
            const double sl = (double)slo[r];
            const double Er = EW + (double)r * step;
            const double SDr = sqrt(V + (double)r * var) / theta;
            double P;
            if (SDr > 0.0)
                P = 0.5 * erfc((sl - Er) / (SDr * 1.4142135623730951));
            else
                P = (Er > sl) ? 1.0 : 0.0;
            slot += P;
        }
        return slot;
    }
};

// Workgroups that share a task.
__device__ inline int task_split(int64_t tasks)
{
    return tasks * 4 <= kExactBlocks ? 4 : (tasks * 2 <= kExactBlocks ? 2 : 1);
}

// The exact score of queue g of candidate k of n, after k_fexact.
__device__ inline double task_score(const FArgs &a, int64_t n, int64_t k, int g)
{
    const int64_t t = k * a.I + g;
    if (task_split(n * a.I) == 1) return a.Q[t];
    double q = 0.0;
    for (int s = 0; s < kExactSubs; ++s) q += a.parts[t * kExactSubs + s];
    return q;
}

__global__ __launch_bounds__(kExactThreads) void k_fexact(FArgs a, const int64_t *plan_index,
                                                           const int32_t *count_dev, int64_t count)
{
    __shared__ double part[kExactSubs][kExactWaves];
    __shared__ double terms[kExactWaves][kExactSubs][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int js = wave_id();
    const int64_t n = count_dev ? (int64_t)__builtin_amdgcn_readfirstlane(count_dev[0]) : count;
    const int64_t tasks = n * a.I;
    const int split = task_split(tasks);
    const int subs = kExactSubs / split;            // of this workgroup, from sub0 on
    const double ecost = (double)a.evict_cost;
    for (int64_t ts = blockIdx.x; ts < tasks * split; ts += gridDim.x) {
        const int64_t t = ts / split;
        const int sub0 = (int)(ts % split) * subs;
        const int64_t k = t / a.I;
        const int g = (int)(t % a.I);
        int64_t p = plan_index[k];
        p = p < 0 ? 0 : (p >= a.P ? a.P - 1 : p);
        const int G = a.G;
        const int bq = clampi(a.qoff[(int64_t)g * a.ld + p], 0, G);
        const int eq = clampi(a.qoff[(int64_t)(g + 1) * a.ld + p], bq, G);
        const double theta = (double)a.inst_tput[g];
        const int cls = clampi(a.inst_class[g], 0, a.C - 1);
        int prev = a.inst_model0 ? clampi(a.inst_model0[g], -1, a.M - 1) : -1;
        double rA = 0.0, rV = 0.0, rK = 0.0;
        double rC = 0.0;                       // lane s < subs: the sum of its slice sub0 + s
        for (int v0 = bq; v0 < eq; v0 += kWave) {
            const int cnt = min(kWave, eq - v0);
            const bool on = lane < cnt;
            int i = -1;
            if (on) {
                i = a.perm[(int64_t)(v0 + lane) * a.ld + p];
                if (i < 0 || i >= G) i = -1;
            }
            const int m = i >= 0 ? grp_model(a.grp[i]) : -1;
            // an invalid id (malformed plan) keeps the model before it
            int pm = __shfl_up(m, 1, kWave);
            if (lane == 0) pm = prev;
            const int mm = m >= 0 ? m : pm;
            double xa = 0.0, xb = 0.0, c1 = 0.0, c2 = 0.0;
            if (i >= 0) {
                const double nn = (double)grp_count(a.grp[i]);
                xa = nn * (double)a.grp[i].mu;
                xb = nn * (double)a.grp[i].var;
                if (pm >= 0 && pm != m && a.swap_cost)
                    c1 = (double)a.swap_cost[((int64_t)cls * a.M + pm) * a.M + m];
                const int s = v0 + lane;
                if (a.evict_bits && ((a.evict_bits[(int64_t)(s >> 5) * a.ld + p] >> (s & 31)) & 1u))
                    c2 = ecost;
            }
            const double la = from_left0(xa), lb = from_left0(xb);
            const double l1 = from_left0(c1), l2 = from_left0(c2);
            double A = rA, V = rV, K0 = rK;
            // cnt - 1 steps, rounded up to blocks of 8 (a step past the last
            // position leaves every position's sums unchanged), the count in
            // a scalar register so that only a block ends in a branch
            const int steps = __builtin_amdgcn_readfirstlane(cnt - 1);
            for (int j = 0; j < steps; j += 8) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    A = from_left(A) + la;
                    V = from_left(V) + lb;
                    K0 = (from_left(K0) + l1) + l2;
                }
            }
            double K = K0 + c1;
            K = K + c2;
            const int last = cnt - 1;
            // the slices' terms, a position per lane, change places in LDS: a lane per
            // slice then adds its positions one after another
            double (*mine)[kWave] = terms[js];
            ExactGroup x{nullptr, 0, 0.0, 0.0, V, 0.0};
            if (i >= 0) {
                const FReq q = a.req[i];
                x.slo = a.req_slo + q.first;
                x.n = req_count(q);
                x.EW = A / theta + K;
                x.step = (double)q.mu / theta;
                x.var = (double)q.var;
            }
            bool some = false;
            for (int s = 0; s < subs; ++s) {
                const double t = x.slice(theta, js * kExactSubs + sub0 + s);
                some = some || t != 0.0;
                mine[s][lane] = t;
            }
            wave_sync();
            // (zeros leave the sums as they are: slices without requests, tails of none)
            if (__builtin_amdgcn_ballot_w64(some) != 0 && lane < subs) {
                const double *t = mine[lane];
                int j = 0;
                for (; j + 8 <= cnt; j += 8) {
                    double x[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) x[u] = t[j + u];
#pragma unroll
                    for (int u = 0; u < 8; ++u) rC += x[u];
                }
                for (; j < cnt; ++j) rC += t[j];
            }
            wave_sync();
            rA = lane_value(A, last) + lane_value(xa, last);
            rV = lane_value(V, last) + lane_value(xb, last);
            rK = lane_value(K, last);
            // the model the next round starts from: the last valid one
            int carry = __builtin_amdgcn_readlane(mm, last);
            prev = carry;
        }
        if (lane < subs) part[lane][js] = rC;
        __syncthreads();
        if (threadIdx.x == 0) {
            double q = 0.0;
            for (int s = 0; s < subs; ++s) {
                double x = 0.0;
                for (int j = 0; j < kExactWaves; ++j) x += part[s][j];
                if (split > 1) a.parts[t * kExactSubs + sub0 + s] = x;
                q += x;
            }
            if (split == 1) a.Q[t] = q;
        }
        __syncthreads();
    }
}

// Exact plan scores of the listed plans (queue scores summed in order).
__global__ __launch_bounds__(kThreads) void k_fplan(FArgs a, int64_t n, double *score)
{
    for (int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * kThreads) {
        double s = 0.0;
        for (int g = 0; g < a.I; ++g) s += task_score(a, n, k, g);
        score[k] = s;
    }
}

// The lowest (exact score, plan index) over the candidates.
__global__ __launch_bounds__(kPickThreads) void k_fpick(FArgs a, int64_t *best_index,
                                                        double *best_score)
{
    __shared__ double ls[kPickThreads / kWave];
    __shared__ int64_t li[kPickThreads / kWave];
    const int n = a.ncand[0];
    double bs = INFINITY;
    int64_t bi = -1;
    const int lane = threadIdx.x & (kWave - 1);
    auto take = [&](double s, int64_t p) {
        if (s == s && (bi < 0 || better(s, p, bs, bi))) {   // a NaN score never wins
            bs = s;
            bi = p;
        }
    };
    if (n <= 2 * a.I) {
        // one wavefront per candidate: the lanes load its queue scores, which are
        // added in queue order
        for (int k = wave_id(); k < n; k += kPickThreads / kWave) {
            double s = 0.0;
            for (int g0 = 0; g0 < a.I; g0 += kWave) {
                const double q = g0 + lane < a.I ? task_score(a, n, k, g0 + lane) : 0.0;
                const int c = min(kWave, a.I - g0);
                for (int j = 0; j < c; ++j) s += lane_value(q, j);
            }
            if (lane == 0) take(s, a.cand[k]);
        }
    } else {
        // many (every plan, where none misses an SLO): a lane per candidate; 4096 of
        // 16 queues took 1.3 ms a wavefront each
        for (int k = threadIdx.x; k < n; k += kPickThreads) {
            double s = 0.0;
            for (int g = 0; g < a.I; ++g) s += task_score(a, n, k, g);
            take(s, a.cand[k]);
        }
    }
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const double s2 = __shfl_xor(bs, o, kWave);
        const int64_t i2 = __shfl_xor(bi, o, kWave);
        if (i2 >= 0 && (bi < 0 || better(s2, i2, bs, bi))) {
            bs = s2;
            bi = i2;
        }
    }
    const int w = threadIdx.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        ls[w] = bs;
        li[w] = bi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < kPickThreads / kWave; ++k)
            if (li[k] >= 0 && (bi < 0 || better(ls[k], li[k], bs, bi))) {
                bs = ls[k];
                bi = li[k];
            }
        best_index[0] = bi;
        best_score[0] = bi < 0 ? INFINITY : bs;
    }
}

#pragma clang fp contract(on)

// ---------------------------------------------------------------------------
// Host side

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

// Slots per segment: 128, or 64 or 32 while that leaves fewer than 2048 wavefronts
// (a wavefront walks a segment one slot after another).  6000 plans of 1000
// groups, k_fseg and k_fwalk: 49 and 65 us with 128 slots in workgroups of 16
// wavefronts (94 of them), 23 and 31 us with 32 in workgroups of 8.  All the
// plans of a call count, not those of a chunk: chunks change no bit.
int segment_of(int32_t G, int64_t P)
{
    const int64_t tiles = (P + kWave - 1) / kWave;
    int seg = kSeg;
    while (seg > kMinSeg && tiles * ((G + seg - 1) / seg) < 2048) seg /= 2;
    return seg;
}

// Plans per chunk: as many as `want` asks for (0 = up to kChunkBudget bytes of
// lists, which hold every group at most, and segment sums), a multiple of 64, no more than the plans rounded up.
int64_t chunk_of(int32_t G, int64_t P, int64_t want)
{
    const size_t nseg = (size_t)((G > 0 ? G : 1) + kSeg - 1) / kSeg;
    int64_t c = (int64_t)(kChunkBudget / ((kSeg / kMinSeg * (sizeof(Piece) + sizeof(Start) + 8) +
                                         kSeg * (sizeof(FEntry) + sizeof(uint16_t))) * nseg));
    if (want > 0) c = want;
    c = (c + kWave - 1) / kWave * kWave;
    const int64_t all = (P + kWave - 1) / kWave * kWave;
    if (all < c) c = all;
    return c < kWave ? kWave : c;
}

struct FLayout {
    size_t grp, req, inst, blk, slo, nreq, list, listq, listn, piece, start, part, F, bmin, ncand, cand, Q, parts, total;
    int64_t chunk;
    int seg;
};

FLayout flayout(const qlm_problem *pr, int64_t P, int64_t n_req, int64_t chunk)
{
    FLayout L{};
    const int32_t G = pr->n_groups, I = pr->n_instances;
    L.chunk = chunk_of(G, P, chunk);
    const int64_t Pn = P > 0 ? P : 1;
    size_t o = 0;
    auto put = [&](size_t &field, size_t bytes) {
        field = o;
        o += align256(bytes);
    };
    put(L.grp, sizeof(FGrp) * (size_t)G);
    put(L.req, sizeof(FReq) * (size_t)G);
    put(L.inst, sizeof(FInst) * (size_t)I);
    put(L.blk, sizeof(float2) * ((size_t)n_req / kReqBlk + (size_t)G + kBounds));
    put(L.slo, sizeof(float) * kReqBlk * ((size_t)n_req / kReqBlk + (size_t)G + 1));
    put(L.nreq, 8);
    L.seg = segment_of(G, P);
    // (room for the longest and the most segments whatever P asks for: the size
    // may not grow as P falls, or a workspace taken for a large batch in small
    // chunks would be refused for a smaller one)
    const size_t slots = (size_t)((G + kSeg - 1) / kSeg) * kSeg;
    const size_t nseg = (size_t)((G + kMinSeg - 1) / kMinSeg);
    const size_t tiles = (size_t)(L.chunk / kWave);
    put(L.list, sizeof(FEntry) * tiles * slots * kWave);
    put(L.listq, sizeof(uint16_t) * tiles * slots * kWave);
    put(L.listn, 4 * tiles * nseg);
    put(L.piece, sizeof(Piece) * nseg * (size_t)L.chunk);
    put(L.start, sizeof(Start) * nseg * (size_t)L.chunk);
    put(L.part, 8 * nseg * (size_t)L.chunk);
    put(L.F, 8 * (size_t)Pn);
    put(L.bmin, 8 * (size_t)kSumBlocks);
    put(L.ncand, 256);
    put(L.cand, 8 * (size_t)Pn);
    put(L.Q, 8 * (size_t)Pn * (size_t)I);
    put(L.parts, 8 * 2 * (size_t)kExactBlocks);
    L.total = o;
    return L;
}

int check_requests(const qlm_problem *pr, const float *req_slo, int64_t n_req)
{
    (void)pr;
    if (n_req < 0 || n_req >= kMaxRequests)
        return fail(QLM_ERR_ARG, "n_requests must be in [0, 2^31)");
    if (n_req > 0 && !req_slo) return fail(QLM_ERR_ARG, "req_slo is NULL");
    return QLM_OK;
}

FArgs fargs(const qlm_problem *pr, const qlm_plans *pl, const float *req_slo, int64_t n_req,
            void *ws, const FLayout &L)
{
    FArgs a{};
    a.G = pr->n_groups;
    a.I = pr->n_instances;
    a.M = pr->n_models;
    a.C = pr->n_classes;
    a.grp_count = pr->grp_count;
    a.grp_mu = pr->grp_mu;
    a.grp_var = pr->grp_var;
    a.grp_model = pr->grp_model;
    a.inst_tput = pr->inst_tput;
    a.inst_class = pr->inst_class;
    a.inst_model0 = pr->inst_model0;
    a.swap_cost = pr->swap_cost;
    a.evict_cost = pr->evict_cost;
    a.P = pl->n_plans;
    a.ld = pl->plan_stride;
    a.perm = pl->perm;
    a.qoff = pl->qoff;
    a.evict_bits = pl->evict_bits;
    a.req_slo = req_slo;
    a.n_req = n_req;
    unsigned char *w = (unsigned char *)ws;
    a.grp = (FGrp *)(w + L.grp);
    a.req = (FReq *)(w + L.req);
    a.inst = (FInst *)(w + L.inst);
    a.blk = (float2 *)(w + L.blk);
    a.slo = (float *)(w + L.slo);
    a.nreq = (double *)(w + L.nreq);
    a.list = (FEntry *)(w + L.list);
    a.listq = (uint16_t *)(w + L.listq);
    a.listn = (int32_t *)(w + L.listn);
    a.piece = (Piece *)(w + L.piece);
    a.start = (Start *)(w + L.start);
    a.part = (int64_t *)(w + L.part);
    a.F = (double *)(w + L.F);
    a.bmin = (double *)(w + L.bmin);
    a.ncand = (int32_t *)(w + L.ncand);
    a.cand = (int64_t *)(w + L.cand);
    a.Q = (double *)(w + L.Q);
    a.parts = (double *)(w + L.parts);
    a.chunk = L.chunk;
    a.seg = L.seg;
    a.nseg = (a.G + L.seg - 1) / L.seg;
    // a segment of a plan holds at most every request, and 2^28 (128 groups of 2^21)
    const int64_t most = n_req < ((int64_t)1 << 28) ? n_req : (int64_t)1 << 28;
    a.fix_bits = kFixBits;
    while (most >> (kFixBits - a.fix_bits)) --a.fix_bits;
    a.fix = ldexp(1.0, a.fix_bits);
    a.unfix = ldexp(1.0, -a.fix_bits);
    return a;
}

int launched(const char *what)
{
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? QLM_OK : hip_fail(e, what);
}

// Common start of every call: argument checks, the workspace, the per-call
// tables.
int fbegin(const qlm_problem *problem, const qlm_plans *plans, const float *req_slo,
           int64_t n_req, void *ws, size_t ws_bytes, FArgs *out, FLayout *lay, bool screen,
           bool prep, hipStream_t stream)
{
    int rc = check_problem(problem);
    if (rc) return rc;
    rc = check_plans(problem, plans);
    if (rc) return rc;
    rc = check_requests(problem, req_slo, n_req);
    if (rc) return rc;
    if (problem->n_groups > kMaxFcfsGroups || problem->n_instances > kMaxFcfsInstances)
        return fail(QLM_ERR_CAPACITY, "the per-request calls take at most 65536 groups and 4096 "
                                      "instances");
    if (!ws || ((uintptr_t)ws & 255u))
        return fail(QLM_ERR_WORKSPACE, "workspace must be non-NULL and 256-byte aligned");
    // the largest chunk the workspace holds, from the default down to 64 plans
    FLayout L = flayout(problem, plans->n_plans, n_req, 0);
    if (ws_bytes < L.total) {
        const FLayout L64 = flayout(problem, plans->n_plans, n_req, kWave);
        if (ws_bytes < L64.total) return fail(QLM_ERR_WORKSPACE, "workspace too small");
        const size_t per = (L.total - L64.total) / (size_t)(L.chunk - kWave);
        int64_t c = kWave + (int64_t)((ws_bytes - L64.total) / (per > 0 ? per : 1));
        c = c / kWave * kWave;
        L = flayout(problem, plans->n_plans, n_req, c);
        while (L.total > ws_bytes && c > kWave) L = flayout(problem, plans->n_plans, n_req, c -= kWave);
    }
    *out = fargs(problem, plans, req_slo, n_req, ws, L);
    *lay = L;
    if (plans->n_plans == 0 || !prep) return QLM_OK;
    hipLaunchKernelGGL(k_fprep, dim3((unsigned)((out->G + kPrepThreads - 1) / kPrepThreads)),
                       dim3(kPrepThreads), 0, stream, *out);
    if ((rc = launched("k_fprep launch"))) return rc;
    if (screen) {
        hipLaunchKernelGGL(k_fblocks, dim3((unsigned)((out->G + kWaves - 1) / kWaves)),
                           dim3(kThreads), 0, stream, *out);
        if ((rc = launched("k_fblocks launch"))) return rc;
    }
    return QLM_OK;
}

// The screen over every plan, chunk by chunk: F and the per-block minima.
int screen_all(const FArgs &a, hipStream_t stream)
{
    int rc;
    for (int64_t p0 = 0; p0 < a.P; p0 += a.chunk) {
        const int64_t pc = a.P - p0 < a.chunk ? a.P - p0 : a.chunk;
        const int64_t tiles = (pc + kWave - 1) / kWave;
        // workgroups of 16 wavefronts, or of 8 or 4 where that leaves CUs without
        // one (the tables in LDS are then copied by more workgroups)
        int waves = kSegWaves;
        while (waves > 4 && tiles * ((a.nseg + waves - 1) / waves) < kSegBlocks) waves /= 2;
        const dim3 wgrid((unsigned)(tiles * ((a.nseg + waves - 1) / waves)));
        const dim3 wblock((unsigned)(waves * kWave));
        const size_t tab_bytes = swap_bytes(a) + sizeof(FInst) * (size_t)a.I;
        const size_t seg_lds = sizeof(FGrp) * (size_t)a.G + tab_bytes;
        if (seg_lds <= kSegLdsLimit) {
            const hipError_t e = hipFuncSetAttribute((const void *)k_fseg<true>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)seg_lds);
            if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute");
            hipLaunchKernelGGL(k_fseg<true>, wgrid, wblock, seg_lds, stream, a, p0, pc);
        } else {
            hipLaunchKernelGGL(k_fseg<false>, wgrid, wblock, 0, stream, a, p0, pc);
        }
        if ((rc = launched("k_fseg launch"))) return rc;
        hipLaunchKernelGGL(k_fstart, dim3((unsigned)tiles), dim3(kWave), 0, stream, a, pc);
        if ((rc = launched("k_fstart launch"))) return rc;
        if (seg_lds <= kSegLdsLimit) {
            const hipError_t e = hipFuncSetAttribute((const void *)k_fwalk<true>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                                     (int)seg_lds);
            if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute");
            hipLaunchKernelGGL(k_fwalk<true>, wgrid, wblock, seg_lds, stream, a, p0, pc);
        } else {
            hipLaunchKernelGGL(k_fwalk<false>, wgrid, wblock, 0, stream, a, p0, pc);
        }
        if ((rc = launched("k_fwalk launch"))) return rc;
        qlm_internal::TimedLaunch tl;
        if ((rc = qlm_internal::timing_begin(stream, &tl))) return rc;
        // (as many workgroups as the longest list has shares; those without one end at
        // once, after every list's first)
        const unsigned nlists = (unsigned)(tiles * a.nseg);
        const unsigned shares = (unsigned)((a.seg * kWave + kShare - 1) / kShare);
        hipLaunchKernelGGL(k_ftails, dim3(nlists * shares), dim3(kTailWaves * kWave), 0, stream, a,
                           pc, nlists);
        if ((rc = launched("k_ftails launch"))) return rc;
        qlm_internal::timing_end(stream, &tl);
        hipLaunchKernelGGL(k_fsum, dim3(kSumBlocks), dim3(kThreads), 0, stream, a, p0, pc,
                           p0 == 0 ? 1 : 0);
        if ((rc = launched("k_fsum launch"))) return rc;
    }
    return QLM_OK;
}

}  // namespace

// ---------------------------------------------------------------------------
// C interface

extern "C" {

size_t qlm_fcfs_workspace_bytes(const qlm_problem *problem, int64_t n_plans, int64_t n_requests,
                                int64_t chunk_plans)
{
    if (!problem || problem->n_groups < 1 || problem->n_instances < 1) return 0;
    if (n_plans < 0) n_plans = 0;
    if (n_requests < 0) n_requests = 0;
    return flayout(problem, n_plans, n_requests, chunk_plans > 0 ? chunk_plans : 0).total;
}

int qlm_fcfs_score(const qlm_problem *problem, const qlm_plans *plans, const float *req_slo,
                   int64_t n_requests, void *ws, size_t ws_bytes, double *score,
                   qlm_stream stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    FArgs a;
    FLayout L;
    if (plans && plans->n_plans > 0 && !score) return fail(QLM_ERR_ARG, "score is NULL");
    int rc = fbegin(problem, plans, req_slo, n_requests, ws, ws_bytes, &a, &L, true, true, stream);
    if (rc) return rc;
    if (plans->n_plans == 0) return QLM_OK;
    a.F = score;
    return screen_all(a, stream);
}

int qlm_fcfs_score_exact(const qlm_problem *problem, const qlm_plans *plans, const float *req_slo,
                         int64_t n_requests, const int64_t *plan_index, int64_t n, void *ws,
                         size_t ws_bytes, double *score, qlm_stream stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (n < 0) return fail(QLM_ERR_ARG, "n must be >= 0");
    FArgs a;
    FLayout L;
    if (n > 0 && (!plan_index || !score))
        return fail(QLM_ERR_ARG, "plan_index and score are required");
    if (plans && n > plans->n_plans) return fail(QLM_ERR_ARG, "n must be <= n_plans");
    int rc = fbegin(problem, plans, req_slo, n_requests, ws, ws_bytes, &a, &L, false, n > 0,
                    stream);
    if (rc) return rc;
    if (n == 0) return QLM_OK;
    hipLaunchKernelGGL(k_fexact, dim3(kExactBlocks), dim3(kExactThreads), 0, stream, a,
                       plan_index, (const int32_t *)nullptr, n);
    if ((rc = launched("k_fexact launch"))) return rc;
    int64_t blocks = (n + kThreads - 1) / kThreads;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(k_fplan, dim3((unsigned)blocks), dim3(kThreads), 0, stream, a, n, score);
    return launched("k_fplan launch");
}

int qlm_fcfs_best_plan(const qlm_problem *problem, const qlm_plans *plans, const float *req_slo,
                       int64_t n_requests, void *ws, size_t ws_bytes, int64_t *best_index,
                       double *best_score, qlm_stream stream_)
{
    hipStream_t stream = (hipStream_t)stream_;
    if (!best_index || !best_score)
        return fail(QLM_ERR_ARG, "best_index and best_score are required");
    FArgs a;
    FLayout L;
    int rc = fbegin(problem, plans, req_slo, n_requests, ws, ws_bytes, &a, &L, true, true, stream);
    if (rc) return rc;
    if (plans->n_plans == 0) {
        hipLaunchKernelGGL(k_fzero, dim3(1), dim3(kWave), 0, stream, a);
        if ((rc = launched("k_fzero launch"))) return rc;
    } else {
        if ((rc = screen_all(a, stream))) return rc;
        hipLaunchKernelGGL(k_fselect, dim3(kSumBlocks), dim3(kThreads), 0, stream, a, kSumBlocks);
        if ((rc = launched("k_fselect launch"))) return rc;
        hipLaunchKernelGGL(k_fexact, dim3(kExactBlocks), dim3(kExactThreads), 0, stream, a,
                           (const int64_t *)a.cand, (const int32_t *)a.ncand, (int64_t)0);
        if ((rc = launched("k_fexact launch"))) return rc;
    }
    hipLaunchKernelGGL(k_fpick, dim3(1), dim3(kPickThreads), 0, stream, a, best_index, best_score);
    return launched("k_fpick launch");
}

}  // extern "C"
