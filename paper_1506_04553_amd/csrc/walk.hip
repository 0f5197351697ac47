// walk.hip -- grouped tree walk (Section 2.2: Barnes-Hut with opening angle
// theta, walked once per group).  One wavefront walks the tree for one group
// and emits three lists:
//   C_g  accepted cells (multipole interactions),
//   F_g  particles of opened leaves whose box is at least h* = max(h, r_out)
//        away from the group box: for them K = W = 1 and j != i,
//   N_g  particles of the other opened leaves: the only candidates for
//        neighbours of the group's particles and for K, W < 1.
// The particle list P_g of the method is F_g + N_g.
// A cell c is accepted iff theta^2 * D^2(com_c, box_g) > side_c^2 and
// B^2(box_c, box_g) >= h^2, with D the point-to-box and B the box-to-box gap
// distance, each summed as (tx*tx + ty*ty) + tz*tz over per-axis gaps
// t = max(max(lo - p, 0), p - hi).  This file is compiled with
// -ffp-contract=off so these decisions are reproducible bit for bit.
//
// The walk is wavefront-cooperative: up to 64 pending nodes are popped from a
// stack, classified in parallel, and the children of opened internal nodes are
// pushed back.  Node levels never decrease towards the top of the stack and at
// most 8*64 entries of one level are pending at once, so 22*512 entries bound
// the stack; the walk runs with a small stack in LDS and falls back to a
// per-block stack of that bound in global memory if a group overflows it.
//
// Two ways to lay out the lists, both as one (begin, end) segment per group and
// list, with no two groups ever updating the same memory word:
//   fixed stride (when an earlier build gives the group count and the longest
//     lists): group g writes list k at g * cap_k in a single walk; a group
//     beyond the estimated count or a list longer than cap_k raises a flag and
//     the build falls back to
//   two passes: count, prefix-sum, then walk again writing at the exact
//     offsets (segments tile the arrays).
// The statistics (list totals, interaction counts, longest lists) are
// reductions over the per-group counts.
#include "device_util.h"
#include "internal.h"

namespace p3t {

constexpr int kWalkThreads = 64;        // one wavefront per block
constexpr int kWalkGrid = 8192;         // 32 resident wavefronts on each of 256 CUs
constexpr int kLdsStack = 1536;
constexpr int kMaxChild = 8;
constexpr int kGlobalStack = kLevels * kMaxChild * kWave + kWave + kMaxChild;

enum WalkMode { kCount = 0, kEmit = 1, kFixed = 2 };

struct WalkParams {
    double th2, h2, hn2;   // theta^2, h^2, max(h, r_out)^2
    double far2;           // see walk_far2 (0: no cell is far enough)
};

// Device outputs of one walk launch.
struct WalkOut {
    int64_t *cnt;            // [3][stride] per-group counts (count and fixed passes)
    int64_t *beg, *end;      // [3][stride] segments (emit and fixed passes)
    int32_t *idx[3];         // lists
    int64_t cap[3];          // fixed: entries reserved per group and list
    int64_t gcap;            // fixed: groups the lists have room for
    int32_t *stack_ovf;      // set if a group overflowed even the global stack
    int32_t *spilled;        // groups that walked on the global stack
    int32_t *cap_ovf;        // fixed: set if some group did not fit
    int64_t stride;
};

// the c consecutive indices first .. first + c - 1 at d, four to a store (the
// stores need only 4-byte alignment)
typedef int32_t int4u __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ void write_range(int32_t *d, int32_t first, int c) {
    int t = 0;
    for (; t + 4 <= c; t += 4) {
        const int32_t f = first + t;
        *reinterpret_cast<int4u *>(d + t) = int4u{f, f + 1, f + 2, f + 3};
    }
    for (; t < c; ++t) d[t] = first + t;
}

// max(max(u, 0), v); nothing here is NaN, and the sign of a zero is squared away
__device__ __forceinline__ double gap(double u, double v) { return fmax(fmax(u, 0.0), v); }

// Walks the tree for one group on the stack `stk` of `cap` entries (and room for
// kMaxChild more): list k's entries to dst[k] (kEmit, and up to wo.cap[k] of them
// for kFixed), their numbers to run[k].  False if the stack overflows.  Inlined
// for each memory the stack lies in: through a pointer to either, every pop would
// wait for the list stores before it.  (Each iteration is a chain of latencies,
// which bounds the walk of few groups: with that, and branches around what no lane
// needs, 74 us instead of 98 at 65536 particles, 40 instead of 50 at 15001.)
template <int MODE, bool LAZY>
__device__ __forceinline__ bool walk_group(const GroupInfo &gi, const NodeWalk *__restrict__ nodes,
                                           const WalkParams &wp, const WalkOut &wo,
                                           int32_t *const dst[3], int64_t run[3], int32_t *stk,
                                           int cap) {
    const int lane = threadIdx.x;
    run[0] = run[1] = run[2] = 0;
    int sp = 1;
    if (lane == 0) stk[0] = 0;
    wave_order();
    while (sp > 0) {
        const int k = sp < kWave ? sp : kWave;
        const int base = sp - k;
        const int32_t node = lane < k ? stk[base + lane] : -1;
        sp = base;
        wave_order();
        bool acc = false, leaf = false, near = false;
        int32_t first = 0, count = 0, cf = 0, ncld = 0;
        if (node >= 0) {
            const NodeWalk &nd = nodes[node];
            const double l2 = nd.l2;
            const double t0 = gap(gi.lo[0] - nd.cx, nd.cx - gi.hi[0]);
            const double t1 = gap(gi.lo[1] - nd.cy, nd.cy - gi.hi[1]);
            const double t2 = gap(gi.lo[2] - nd.cz, nd.cz - gi.hi[2]);
            const double D2 = t0 * t0 + t1 * t1 + t2 * t2;
            acc = wp.th2 * D2 > fabs(l2);
            if (!(LAZY && acc && l2 > 0.0 && D2 * wp.far2 >= wp.h2)) {
                const double b0 = gap(nd.lo[0] - gi.hi[0], gi.lo[0] - nd.hi[0]);
                const double b1 = gap(nd.lo[1] - gi.hi[1], gi.lo[1] - nd.hi[1]);
                const double b2 = gap(nd.lo[2] - gi.hi[2], gi.lo[2] - nd.hi[2]);
                const double B2 = b0 * b0 + b1 * b1 + b2 * b2;
                acc = acc && (B2 >= wp.h2);
                leaf = nd.n_child == 0;
                near = B2 < wp.hn2;
                first = nd.first;
                count = nd.count;
                cf = nd.child_first;
                ncld = nd.n_child;
            }
        }
        const bool isC = node >= 0 && acc;
        const bool isO = node >= 0 && !acc && !leaf;
        const bool isF = node >= 0 && !acc && leaf && !near;
        const bool isN = node >= 0 && !acc && leaf && near;
        // accepted cells
        const uint64_t mC = ballot(isC);
        if (MODE != kCount && isC) {
            const int64_t pos = run[0] + count_below(mC);
            if (MODE == kEmit || pos < wo.cap[0]) dst[0][pos] = node;
        }
        run[0] += __popcll(mC);
        // particles of far, then near, opened leaves
#pragma unroll
        for (int kk = 1; kk < 3; ++kk) {
            const bool mine = kk == 1 ? isF : isN;
            if (!ballot(mine)) continue;
            const int c = mine ? count : 0;
            int tot;
            const int excl = wave_excl_count(c, tot);
            if (MODE == kEmit && mine) write_range(dst[kk] + run[kk] + excl, first, c);
            if (MODE == kFixed && mine) {
                const int64_t pos = run[kk] + excl;
                const int64_t lim = wo.cap[kk] - pos;
                const int cc = lim < c ? (lim > 0 ? (int)lim : 0) : c;
                write_range(dst[kk] + pos, first, cc);
            }
            run[kk] += tot;
        }
        // children of opened internal nodes
        if (!ballot(isO)) continue;
        const int ocnt = isO ? ncld : 0;
        int otot;
        const int oexcl = wave_excl_small<4>(ocnt, otot);
        if (sp + otot > cap) return false;
        // Every lane writes kMaxChild entries, the last ones first: what goes past
        // its children is then overwritten by the lanes they belong to.
        if (isO) {
            int32_t *d = stk + sp + oexcl;
#pragma unroll
            for (int t = kMaxChild - 1; t >= 0; --t) {
                d[t] = cf + t;
                wave_order();
            }
        }
        sp += otot;
        wave_order();
    }
    return true;
}

template <int MODE, bool LAZY>
__global__ __launch_bounds__(kWalkThreads) void k_walk(const GroupInfo *__restrict__ grp,
                                                        const int32_t *__restrict__ n_groups_dev,
                                                        const NodeWalk *__restrict__ nodes,
                                                        WalkParams wp, WalkOut wo,
                                                        int32_t *__restrict__ gstack, int lds_cap) {
    __shared__ int32_t lstack[kLdsStack + kMaxChild];
    int32_t *const gstk = gstack + (int64_t)blockIdx.x * kGlobalStack;
    const int lane = threadIdx.x;
    const int G = *n_groups_dev;
    const int64_t S = wo.stride;
    for (int g = blockIdx.x; g < G; g += gridDim.x) {
        const GroupInfo gi = grp[g];
        int64_t run[3];
        int32_t *dst[3] = {nullptr, nullptr, nullptr};
        if (MODE == kFixed && g >= wo.gcap) {
            if (lane == 0) atomicOr(wo.cap_ovf, 1);
            continue;
        }
        if (MODE == kEmit)
            for (int k = 0; k < 3; ++k) dst[k] = wo.idx[k] + wo.beg[k * S + g];
        if (MODE == kFixed)
            for (int k = 0; k < 3; ++k) dst[k] = wo.idx[k] + (int64_t)g * wo.cap[k];
        // the walk runs on the LDS stack; a group whose pending nodes outgrow
        // it walks again from the root on this block's stack in global memory
        if (!walk_group<MODE, LAZY>(gi, nodes, wp, wo, dst, run, lstack, lds_cap)) {
            if (lane == 0) atomicAdd(wo.spilled, 1);
            if (!walk_group<MODE, LAZY>(gi, nodes, wp, wo, dst, run, gstk, kGlobalStack - kMaxChild)) {
                if (lane == 0) atomicAdd(wo.stack_ovf, 1);
                continue;   // cannot happen: the global stack holds the bound
            }
        }
        if (lane == 0) {
            bool over = false;
            for (int k = 0; k < 3; ++k) {
                if (MODE == kCount) wo.cnt[k * S + g] = run[k];
                if (MODE == kEmit) wo.end[k * S + g] = wo.beg[k * S + g] + run[k];
                if (MODE == kFixed) {
                    const int64_t b = (int64_t)g * wo.cap[k];
                    over = over || run[k] > wo.cap[k];
                    wo.cnt[k * S + g] = run[k];
                    wo.beg[k * S + g] = b;
                    wo.end[k * S + g] = b + (run[k] < wo.cap[k] ? run[k] : wo.cap[k]);
                }
            }
            if (over) atomicOr(wo.cap_ovf, 1);
        }
    }
}

// Walk results read back by the host (int64 slots).
struct WalkStats {
    unsigned long long total[3];   // sum over groups of |C_g|, |F_g|, |N_g|
    unsigned long long n_groups;
    unsigned long long pc, pp;     // sum_g n_g |C_g|, sum_g n_g (|F_g| + |N_g|)
    unsigned long long pp_near;    // sum_g n_g |N_g|
    unsigned long long n_leaves;
    unsigned long long maxlen[3];  // longest list of each kind
    int32_t stack_ovf, cap_ovf;    // flags written by the walk
    int32_t spilled, n_items;      // groups that needed the global stack; items of split groups
    unsigned long long part_used;  // partial sums handed out to split groups
    unsigned long long blocks_done, pad;   // blocks of the statistics kernel
    // per launch-order bucket (see below): groups, their cost, and what their
    // partial sums would take if they were split (FP32: exactly; FP64: members
    // times cost over rounds, which the share of a part still divides)
    unsigned long long bin[kOrderBins], bin_cost[kOrderBins], bin_room[kOrderBins];
    unsigned long long bin_rounds[kOrderBins];   // rounds of the interaction kernel
};

static_assert(sizeof(WalkStats) == kRbWalkWords * 8, "walk statistics slots");

// ---------------------------------------------------------------------------
// Launch order of the per-group kernels: groups in buckets of estimated work
// (quarter octaves of n_g (35 |C_g| + 15 |P_g|), the interaction kernel's
// instruction count), largest first; the order inside a bucket is arbitrary
// (it decides only which block runs which group).
// ---------------------------------------------------------------------------
__host__ __device__ __forceinline__ int cost_bin(float cost) {
    int b = (int)(4.0f * log2f(cost + 1.0f));
    b = b < 0 ? 0 : (b > kOrderBins - 1 ? kOrderBins - 1 : b);
    return kOrderBins - 1 - b;
}

__device__ __forceinline__ float group_cost(int ng, int64_t c, int64_t p) {
    return (float)ng * (35.0f * (float)c + 15.0f * (float)p);
}

// a group's 256-entry tiles per list in units of `tiles` tiles
__device__ __forceinline__ int64_t units_of(int64_t entries, int tiles) {
    return (entries + 256 * tiles - 1) / (256 * tiles);
}

// FP32: the partial sums of a split group, one per unit, virtual wavefront and lane
__device__ __forceinline__ int64_t fp32_room(int ng, int64_t c, int64_t f, int64_t n) {
    const int ls = choose_log2_slices(ng, 8), nw = kWave >> ls, t = fold_tiles(ls);
    return (units_of(c, t) + units_of(f, t) + units_of(n, t)) * ((ng + nw - 1) / nw) * kWave;
}

// Statistics from the per-group counts, the leaf count of the tree, and the
// launch-order buckets: each group's bucket and rank in it (rank[g], packed in
// 8 + 24 bits; not written when G does not fit), the bucket counts gathered in
// LDS first, so that a bucket sees one global update per block.
__global__ __launch_bounds__(1024) void k_walk_stats(const GroupInfo *__restrict__ grp,
                                                    const int32_t *__restrict__ n_groups_dev,
                                                    const int64_t *__restrict__ cnt, int64_t S,
                                                    const int32_t *__restrict__ nchild,
                                                    int64_t n_nodes, bool wide,
                                                    WalkStats *__restrict__ out,
                                                    int32_t *__restrict__ rank,
                                                    unsigned long long *__restrict__ host) {
    __shared__ unsigned long long s_cost[kOrderBins], s_room[kOrderBins], s_rounds[kOrderBins];
    __shared__ uint32_t s_bin[kOrderBins];
    const int G = *n_groups_dev;
    const bool ranks = G < (1 << 24);
    if (threadIdx.x < kOrderBins) {
        s_bin[threadIdx.x] = 0;
        s_cost[threadIdx.x] = s_room[threadIdx.x] = s_rounds[threadIdx.x] = 0;
    }
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nt = (int64_t)gridDim.x * blockDim.x;
    unsigned long long tot[3] = {0, 0, 0}, mx[3] = {0, 0, 0}, pc = 0, pp = 0, ppn = 0, lv = 0;
    int32_t first_rank = 0;   // of the thread's first group
    for (int64_t g = t0; g < G; g += nt) {
        const int ng = grp[g].count;
        const unsigned long long n = (unsigned long long)ng;
        int64_t c[3];
        for (int k = 0; k < 3; ++k) {
            c[k] = cnt[k * S + g];
            tot[k] += c[k];
            mx[k] = (unsigned long long)c[k] > mx[k] ? c[k] : mx[k];
        }
        pc += n * c[0];
        pp += n * (c[1] + c[2]);
        ppn += n * c[2];
        if (ranks) {
            const float cost = group_cost(ng, c[0], c[1] + c[2]);
            const int b = cost_bin(cost);
            atomicAdd(&s_cost[b], (unsigned long long)cost);
            const int rounds = rounds_of(ng, wide);
            atomicAdd(&s_room[b],
                      wide ? (unsigned long long)((float)ng * (cost + 1.0f) / (float)rounds) + 1
                           : (unsigned long long)fp32_room(ng, c[0], c[1], c[2]));
            atomicAdd(&s_rounds[b], (unsigned long long)rounds);
            const int32_t r = (b << 24) | (int32_t)atomicAdd(&s_bin[b], 1u);
            if (g == t0) first_rank = r; else rank[g] = r;
        }
    }
    __syncthreads();
    if (threadIdx.x < kOrderBins && s_bin[threadIdx.x]) {
        s_bin[threadIdx.x] =
            (uint32_t)atomicAdd(&out->bin[threadIdx.x], (unsigned long long)s_bin[threadIdx.x]);
        atomicAdd(&out->bin_cost[threadIdx.x], s_cost[threadIdx.x]);
        atomicAdd(&out->bin_room[threadIdx.x], s_room[threadIdx.x]);
        atomicAdd(&out->bin_rounds[threadIdx.x], s_rounds[threadIdx.x]);
    }
    __syncthreads();
    if (ranks)   // this block's groups come after those already counted
        for (int64_t g = t0; g < G; g += nt) {
            const int32_t r = g == t0 ? first_rank : rank[g];
            rank[g] = r + (int32_t)s_bin[r >> 24];
        }
    for (int64_t i = t0; i < n_nodes; i += nt) lv += nchild[i] == 0;
    // wave reductions, then one set of updates per block
    __shared__ unsigned long long s_red[16][10];
    unsigned long long v[10] = {pc, pp, ppn, lv, tot[0], tot[1], tot[2], mx[0], mx[1], mx[2]};
    const int w = threadIdx.x / kWave;
    for (int k = 0; k < 10; ++k) {
        v[k] = k < 7 ? wave_total_u64<false>(v[k]) : wave_total_u64<true>(v[k]);
        if (lane_id() == kWave - 1) s_red[w][k] = v[k];
    }
    __syncthreads();
    if (threadIdx.x < 10) {
        const int k = threadIdx.x;
        unsigned long long r = 0;
        for (int q = 0; q < (int)(blockDim.x / kWave); ++q) {
            const unsigned long long x = s_red[q][k];
            r = k < 7 ? r + x : x > r ? x : r;
        }
        unsigned long long *const to[10] = {&out->pc, &out->pp, &out->pp_near, &out->n_leaves,
                                            &out->total[0], &out->total[1], &out->total[2],
                                            &out->maxlen[0], &out->maxlen[1], &out->maxlen[2]};
        if (k < 7) atomicAdd(to[k], r);
        else atomicMax(to[k], r);
    }
    if (t0 == 0) out->n_groups = (unsigned long long)G;
    // the last block hands the sums to the host's readback area
    __shared__ bool s_last;
    if (threadIdx.x < kOrderBins) __threadfence();   // the threads that added to it
    __syncthreads();
    if (threadIdx.x == 0) {
        s_last = atomicAdd(&out->blocks_done, 1ull) + 1 == gridDim.x;
        __threadfence();
    }
    __syncthreads();
    if (!s_last) return;
    const unsigned long long *from = reinterpret_cast<const unsigned long long *>(out);
    for (int k = threadIdx.x; k < kRbWalkWords; k += blockDim.x)
        host[k] = __hip_atomic_load(&from[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A cell's members lie in a cube of side l, and where its l2 says so their centre of
// mass in the members' box, up to 1e-4 l: then the box is at most sqrt(3) (l + 1e-4 l)
// nearer to a group than the centre.  So a cell with theta D > l has a gap of at
// least D (1 - sqrt(3) theta), less 2e-4 D, and where that exceeds h by more than
// any rounding, the test of the gap passes without the box.
static double walk_far2(double theta) {
    const double c = 1.0 - 1.7321 * theta - 1e-3;
    return c > 0.0 ? c * c / 1.002 : 0.0;
}

// With many nodes the walk is bound by the gathers of their records: a lane that
// can tell from the first 32 bytes of 96 that its cell is accepted (four in five)
// reads no more.  That takes the others a second gather, and with few nodes the
// walk is bound by the latency of one after the other: 271 us instead of 300 at
// 2^20 particles (250 thousand nodes), 135 instead of 141 at 2^18 (62 thousand),
// but 83 instead of 74 at 2^16 (15 thousand).
constexpr int64_t kLazyNodes = 50000;

template <int MODE>
static auto walk_kernel(const p3t_ctx *ctx) {
    return ctx->n_nodes > kLazyNodes && walk_far2(ctx->prm.theta) > 0.0 ? k_walk<MODE, true>
                                                                       : k_walk<MODE, false>;
}

static unsigned walk_grid(p3t_ctx *ctx) {
    int64_t g = ctx->n_nodes < kWalkGrid ? ctx->n_nodes : kWalkGrid;
    return (unsigned)(g > 0 ? g : 1);
}

ListsDev lists_dev(const p3t_ctx *ctx) {
    ListsDev L;
    L.order = ptr<int32_t>(ctx->gorder);
    const int64_t stride = ctx->n_nodes + 1;
    const int64_t *beg = ptr<int64_t>(ctx->off), *end = ptr<int64_t>(ctx->seg_end);
    const DevBuf *bufs[3] = {&ctx->c_idx, &ctx->p_idx, &ctx->n_idx};
    for (int k = 0; k < 3; ++k) {
        L.beg[k] = beg + k * stride;
        L.end[k] = end + k * stride;
        L.idx[k] = ptr<int32_t>(*bufs[k]);
    }
    return L;
}

// What splits: the groups of the first buckets, into rounds, and those of the first
// of these, whose partial sums have room, into parts of about `share`.
struct SplitPlan {
    int last_bin;          // groups of buckets 0 .. last_bin are split (-1: none)
    int last_cut;          // ... and of buckets 0 .. last_cut cut into parts
    int first_whole;       // work items kept for them
    bool wide;             // FP64
    float share;
    int32_t *n_items;      // device counters, zero before the launch
    unsigned long long *used;
    SplitGroup *group;     // [G], written for the groups of the split buckets
    WorkItem *work;
};
constexpr int kMaxParts = 256;

// Group order from the ranks, and the work items: each block takes the bucket
// starts (exclusive scan of the counts) itself.  A group of the split buckets
// becomes one item per round and part, with up to one part per unit of its
// lists.
__global__ __launch_bounds__(256) void k_order_place(int64_t G, const int32_t *__restrict__ rank,
                                                     const unsigned long long *__restrict__ bins,
                                                     int32_t *__restrict__ order,
                                                     const GroupInfo *__restrict__ grp,
                                                     const int64_t *__restrict__ cnt, int64_t S,
                                                     SplitPlan sp) {
    static_assert(kOrderBins == 2 * kWave, "two buckets per lane");
    __shared__ uint32_t s_start[kOrderBins + 1];
    const int t = threadIdx.x;
    if (t < kWave) {
        const uint32_t a = (uint32_t)bins[2 * t], b = (uint32_t)bins[2 * t + 1];
        const uint32_t incl = wave_incl_scan(a + b);
        s_start[2 * t] = incl - a - b;
        s_start[2 * t + 1] = incl - b;
        if (t == kWave - 1) s_start[kOrderBins] = incl;
    }
    __syncthreads();
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + t;
    const int32_t r = g < G ? rank[g] : 0;
    const int bin = r >> 24;
    const uint32_t pos = s_start[bin] + (r & 0xffffff);
    const bool split = g < G && bin <= sp.last_bin;
    if (g < G) {
        order[pos] = (int32_t)g;
        if (!split)
            sp.work[sp.first_whole + pos - s_start[sp.last_bin + 1]] = WorkItem{(int32_t)g, 0, 1, -1};
    }
    if (!ballot(split)) return;
    int parts = 0, rounds = 0;
    int64_t room = 0;
    if (split) {
        const int ng = grp[g].count;
        const int64_t c = cnt[g], f = cnt[S + g], n = cnt[2 * S + g];
        const int tiles = sp.wide ? 1 : fold_tiles(choose_log2_slices(ng, 8));
        const int64_t units = units_of(c, tiles) + units_of(f, tiles) + units_of(n, tiles);
        rounds = rounds_of(ng, sp.wide);
        const int64_t want = (int64_t)ceilf(group_cost(ng, c, f + n) / (sp.share * (float)rounds));
        parts = bin > sp.last_cut ? 1 : (int)min<int64_t>(min<int64_t>(want, units), kMaxParts);
        if (parts < 1) parts = 1;
        room = parts == 1 ? 0 : sp.wide ? (int64_t)parts * ng : fp32_room(ng, c, f, n);
    }
    const int64_t rincl = wave_incl_scan(room);
    int64_t rbase = 0;
    if (lane_id() == kWave - 1) rbase = (int64_t)atomicAdd(sp.used, (unsigned long long)rincl);
    rbase = __shfl(rbase, kWave - 1, kWave) + rincl - room;
    const int incl = wave_incl_scan(parts * rounds);
    int32_t base = 0;
    if (lane_id() == kWave - 1) base = atomicAdd(sp.n_items, incl);
    base = __shfl(base, kWave - 1, kWave) + incl - parts * rounds;
    if (split) sp.group[g] = SplitGroup{(int32_t)rbase, parts};
    WorkItem *const out = sp.work + base;
    for (int k = 0; k < rounds; ++k)
        for (int q = 0; q < parts; ++q) out[k * parts + q] = WorkItem{(int32_t)g, q, parts, k};
}

__global__ void k_order_identity(int64_t G, int32_t *__restrict__ order,
                                 WorkItem *__restrict__ work) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= G) return;
    order[g] = (int32_t)g;
    work[g] = WorkItem{(int32_t)g, 0, 1, -1};
}

static WalkStats *walk_stats_dev(const p3t_ctx *ctx) {
    return reinterpret_cast<WalkStats *>(ptr<int64_t>(ctx->readback) + kRbWalk);
}
static const WalkStats *walk_stats_host(const p3t_ctx *ctx) {
    return reinterpret_cast<const WalkStats *>(ctx->hpin + kRbWalk);
}
SplitGroup *split_groups(const p3t_ctx *ctx) {
    return reinterpret_cast<SplitGroup *>(ptr<WorkItem>(ctx->work) + work_blocks(ctx));
}

WorkDev work_dev(const p3t_ctx *ctx) {
    return WorkDev{ptr<WorkItem>(ctx->work), &walk_stats_dev(ctx)->n_items, (int32_t)ctx->n_items};
}

// Which groups are split, from the bucket totals in the host's copy of the
// statistics.  A launch of one block per group ends when its largest group
// does: few particles make few groups, and a group at the cluster's edge has a
// wide box that opens almost every cell.  In FP64, groups above a share of the
// work of the blocks that run at once are cut into parts of that size, in the
// same launch: a quarter of an even share where the groups are few (Plummer
// 65536, Salpeter, 1734 groups: 0.90 ms unsplit, 0.56 at half a share, 0.51 at
// a quarter; Plummer 4096: 155 and 29 us), a whole one where they are many and
// only the largest stand out (King 500009, 6818 groups: 2.55 ms unsplit, 2.61
// at a quarter).  The line is coarse: a whole share and a quarter take 178 and 165 us
// at 1643 groups, 260 and 252 at 2671, 2118 and 2149 at 5517 of up to 256 members,
// 1021 and 985 at 5620 of up to 128.  FP32 has a launch of its own for the parts, before the whole
// groups', which costs more than it gains unless every group goes there, where
// they are too few to fill the GPU (Plummer 1000: 86 us unsplit, 44 split;
// Plummer 2^18, n_crit 128: 0.80 ms unsplit, 0.99 with the groups above half
// a share split).  Nor does it where there is a group for every compute unit and
// none takes much longer than the others (20000 particles in 400 places, the largest
// at most 1.7 times the mean: 36 us unsplit, 43 split, the VJP's two passes 96
// and 108; 20000 on a line, 497 groups, 1.9: 117 and 136; but 20000 in a cube, 512
// groups, 2.4: 71 and 60).
constexpr int kBlocks64 = 256 * 4, kBlocks32 = 256 * 5;   // blocks in flight on 256 CUs
constexpr int kFewGroups64 = 2 * kBlocks64;
constexpr int kEvenGroups32 = 256;         // one for every CU
constexpr double kEven32 = 2.0;            // the largest over the mean
// Bound on the partial sums' bytes.  FP64 stays below it: a group in p > 1 parts, the
// next whole number to c = cost / (share rounds), takes less than 2 c sums of a member,
// and the members of a round are at most 512, so that all groups together take at most
// 2 x 512 x 4 x 1024 of 32 bytes.  FP32 reaches it with the longest lists, and cuts the
// costliest groups.
constexpr int64_t kSplitScratch = (int64_t)256 << 20;
static int plan_split(p3t_ctx *ctx, SplitPlan &sp) {
    int rc;
    const WalkStats *hs = walk_stats_host(ctx);
    const bool wide = ctx->prm.precision == P3T_PREC_FP64;
    sp = SplitPlan{-1, -1, 0, wide, 1.0f, nullptr, nullptr, nullptr, nullptr};
    const double cost = 35.0 * (double)hs->pc + 15.0 * (double)hs->pp;
    const double share =
        cost / (wide ? (ctx->n_groups <= kFewGroups64 ? 4.0 : 1.0) * kBlocks64 : 2.0 * kBlocks32) + 1.0;
    int top = 0;   // the costliest groups' bucket: up to 2^((kOrderBins - top) / 4)
    while (top < kOrderBins - 1 && !hs->bin[top]) ++top;
    const bool even = ctx->n_groups >= kEvenGroups32 &&
                      exp2((kOrderBins - top) / 4.0) * (double)ctx->n_groups < kEven32 * cost;
    const int last = wide ? cost_bin((float)share)
                          : ctx->n_groups <= kBlocks32 && !even ? kOrderBins - 1 : -1;
    int64_t groups = 0, rounds = 0;
    double work = 0.0, sums = 0.0, room = 0.0;   // sums: FP32 partial sums, FP64 without rounding up
    const size_t one = 4 * (wide ? sizeof(double) : sizeof(float));
    for (int b = 0; b <= last; ++b) {
        groups += (int64_t)hs->bin[b];
        work += (double)hs->bin_cost[b];
        rounds += (int64_t)hs->bin_rounds[b];
        sums += (double)hs->bin_room[b] / (wide ? share : 1.0);
        // (rounding parts up adds at most as many sums again, or one of each particle)
        const double most = wide ? 1.0001 * (sums + fmin(sums, (double)ctx->n)) : sums;
        if (most * (double)one > (double)kSplitScratch || sp.last_cut < b - 1) continue;
        sp.last_cut = b;
        room = most;
    }
    // each group: at most cost / share + rounds (and rounding of the sums)
    const int64_t items = groups ? (int64_t)(work / share * 1.0001) + groups + rounds : 0;
    if (groups) {
        sp.last_bin = last;
        sp.first_whole = (int)items;
        sp.share = (float)share;
        if ((rc = ensure(ctx, ctx->fpart, ((size_t)room + 1) * one))) return rc;
        sp.n_items = &walk_stats_dev(ctx)->n_items;
        sp.used = &walk_stats_dev(ctx)->part_used;
    }
    ctx->n_split = groups;
    ctx->n_items = items;
    // the items, then each group's first partial sum and parts
    const int64_t blocks = work_blocks(ctx);
    if ((rc = ensure(ctx, ctx->work,
                     (size_t)blocks * sizeof(WorkItem) + (size_t)ctx->n_groups * sizeof(SplitGroup))))
        return rc;
    sp.work = ptr<WorkItem>(ctx->work);
    sp.group = split_groups(ctx);
    return P3T_OK;
}

static int build_order(p3t_ctx *ctx, int64_t stride) {
    int rc;
    const int64_t G = ctx->n_groups;
    if ((rc = ensure(ctx, ctx->gorder, (G + 1) * sizeof(int32_t)))) return rc;
    ctx->n_split = ctx->n_items = 0;
    if (G <= 0) return P3T_OK;
    // ranks are packed in 24 bits: beyond, keep the group order, every group whole
    if (G >= (1 << 24) || ctx->groups_generic) {
        if ((rc = ensure(ctx, ctx->work, (size_t)G * sizeof(WorkItem)))) return rc;
        k_order_identity<<<blocks_for(G, 256), 256, 0, ctx->stream>>>(G, ptr<int32_t>(ctx->gorder),
                                                                     ptr<WorkItem>(ctx->work));
        return check_hip(ctx, hipGetLastError(), "group order");
    }
    SplitPlan sp;
    if ((rc = plan_split(ctx, sp))) return rc;
    k_order_place<<<blocks_for(G, 256), 256, 0, ctx->stream>>>(
        G, ptr<int32_t>(ctx->grank), walk_stats_dev(ctx)->bin, ptr<int32_t>(ctx->gorder),
        ptr<GroupInfo>(ctx->grp), ptr<int64_t>(ctx->cnt), stride, sp);
    return check_hip(ctx, hipGetLastError(), "group order");
}

static int run_walk_stats(p3t_ctx *ctx, const int32_t *G_dev, int64_t stride, WalkStats *ws) {
    // few large blocks: the block results meet in same-address atomics
    const int64_t fit = (ctx->n_nodes + 1023) / 1024;
    k_walk_stats<<<(unsigned)(fit < 32 ? fit : 32), 1024, 0, ctx->stream>>>(
        ptr<GroupInfo>(ctx->grp), G_dev, ptr<int64_t>(ctx->cnt), stride,
        ptr<int32_t>(ctx->node_nchild), ctx->n_nodes, ctx->prm.precision == P3T_PREC_FP64, ws,
        ptr<int32_t>(ctx->grank), reinterpret_cast<unsigned long long *>(ctx->hpin + kRbWalk));
    int rc = check_hip(ctx, hipGetLastError(), "walk stats");
    if (rc) return rc;
    return check_hip(ctx, hipStreamSynchronize(ctx->stream), "sync");
}

// the lists and their launch order are complete at this point of the
// context's stream: work on other streams that reads them waits for ev_lists
static int lists_done(p3t_ctx *ctx, int rc) {
    if (rc) return rc;
    ctx->rows_queued = false;
    return check_hip(ctx, hipEventRecord(ctx->ev_lists, ctx->stream), "event record");
}

int build_lists(p3t_ctx *ctx, bool stats_cleared) {
    int rc;
    const int64_t nn = ctx->n_nodes;   // bound on the number of groups
    const int64_t stride = nn + 1;
    if ((rc = ensure(ctx, ctx->cnt, 3 * stride * sizeof(int64_t)))) return rc;
    if ((rc = ensure(ctx, ctx->off, 3 * stride * sizeof(int64_t)))) return rc;
    if ((rc = ensure(ctx, ctx->seg_end, 3 * stride * sizeof(int64_t)))) return rc;
    if ((rc = ensure(ctx, ctx->grank, stride * sizeof(int32_t)))) return rc;
    int64_t *cnt = ptr<int64_t>(ctx->cnt), *off = ptr<int64_t>(ctx->off);
    int64_t *end = ptr<int64_t>(ctx->seg_end);
    WalkStats *ws = walk_stats_dev(ctx);
    const WalkStats *hs = walk_stats_host(ctx);
    const int32_t *G_dev = ptr<int32_t>(ctx->gscan) + ctx->n;
    const double hn = ctx->prm.r_search > ctx->prm.r_out ? ctx->prm.r_search : ctx->prm.r_out;
    const WalkParams wp{ctx->prm.theta * ctx->prm.theta, ctx->prm.r_search * ctx->prm.r_search,
                        hn * hn, walk_far2(ctx->prm.theta)};
    const unsigned grid = walk_grid(ctx);
    hipStream_t st = ctx->stream;
    DevBuf *lbuf[3] = {&ctx->c_idx, &ctx->p_idx, &ctx->n_idx};
    WalkOut wo{};
    wo.cnt = cnt;
    wo.beg = off;
    wo.end = end;
    wo.stack_ovf = &ws->stack_ovf;
    wo.cap_ovf = &ws->cap_ovf;
    wo.spilled = &ws->spilled;
    wo.stride = stride;
    // every block has a global-memory stack for groups that outgrow the LDS one
    if ((rc = ensure(ctx, ctx->wstack, (size_t)grid * kGlobalStack * sizeof(int32_t)))) return rc;
    int32_t *gstack = ptr<int32_t>(ctx->wstack);
    const int lds_cap = (ctx->walk_lds_cap >= 64 && ctx->walk_lds_cap < kLdsStack) ? ctx->walk_lds_cap
                                                                              : kLdsStack;

    auto reset = [&]() {
        return check_hip(ctx, hipMemsetAsync(ws, 0, sizeof(WalkStats), st), "memset");
    };
    auto finish = [&](bool fixed) {
        ctx->n_groups = (int64_t)hs->n_groups;
        for (int k = 0; k < 3; ++k) {
            ctx->list_total[k] = (int64_t)hs->total[k];
            ctx->list_extent[k] = fixed ? ctx->n_groups * wo.cap[k] : ctx->list_total[k];
            ctx->hint_max[k] = (int64_t)hs->maxlen[k];
        }
        ctx->hint_groups = ctx->n_groups;
        ctx->n_pc = (int64_t)hs->pc;
        ctx->n_pp = (int64_t)hs->pp;
        ctx->n_pp_near = (int64_t)hs->pp_near;
        ctx->n_leaves = (int64_t)hs->n_leaves;
        ctx->walk_fixed = fixed ? 1 : 0;
        ctx->walk_global = hs->spilled > 0 ? 1 : 0;
    };
    auto stack_error = [&]() {
        return set_error(ctx, P3T_EINVAL, "tree walk stack overflow");
    };

    // ---- single walk into fixed-stride segments, sized from the last build ----
    if (ctx->hint_groups > 0 && ctx->prm.n_crit == ctx->hint_n_crit) {
        const int64_t gcap = ctx->hint_groups + ctx->hint_groups / 8 + 64;
        bool ok = gcap <= stride;
        for (int k = 0; k < 3 && ok; ++k) {
            const int64_t m = ctx->hint_max[k];
            wo.cap[k] = (m + m / 4 + 64 + 63) / 64 * 64;
            // keep the reserved room within a few times the last build's lists
            ok = gcap * wo.cap[k] <= 8 * ctx->list_total[k] + (1 << 22);
        }
        if (ok) {
            wo.gcap = gcap;
            for (int k = 0; k < 3; ++k) {
                if ((rc = ensure(ctx, *lbuf[k], (gcap * wo.cap[k] + 1) * sizeof(int32_t)))) return rc;
                wo.idx[k] = ptr<int32_t>(*lbuf[k]);
            }
            if (!stats_cleared && (rc = reset())) return rc;
            walk_kernel<kFixed>(ctx)<<<grid, kWalkThreads, 0, st>>>(ptr<GroupInfo>(ctx->grp), G_dev,
                                                           ptr<NodeWalk>(ctx->node_walk), wp, wo,
                                                           gstack, lds_cap);
            if ((rc = check_hip(ctx, hipGetLastError(), "walk"))) return rc;
            if ((rc = run_walk_stats(ctx, G_dev, stride, ws))) return rc;
            if (hs->stack_ovf) return stack_error();
            if (!hs->cap_ovf) {
                finish(true);
                return lists_done(ctx, build_order(ctx, stride));
            }
        }
    }

    // ---- two passes: count, prefix sums, emit at exact offsets ----
    if ((rc = reset())) return rc;
    // entries past the last group take part in the scans as zeros
    if ((rc = check_hip(ctx, hipMemsetAsync(cnt, 0, 3 * stride * sizeof(int64_t), st), "memset")))
        return rc;
    walk_kernel<kCount>(ctx)<<<grid, kWalkThreads, 0, st>>>(ptr<GroupInfo>(ctx->grp), G_dev,
                                                   ptr<NodeWalk>(ctx->node_walk), wp, wo, gstack,
                                                   lds_cap);
    if ((rc = check_hip(ctx, hipGetLastError(), "walk count"))) return rc;
    for (int k = 0; k < 3; ++k)
        if ((rc = scan_exclusive_i64(ctx, cnt + k * stride, off + k * stride, stride, nullptr)))
            return rc;
    if ((rc = run_walk_stats(ctx, G_dev, stride, ws))) return rc;
    if (hs->stack_ovf) return stack_error();
    for (int k = 0; k < 3; ++k) {
        if ((rc = ensure(ctx, *lbuf[k], ((int64_t)hs->total[k] + 1) * sizeof(int32_t)))) return rc;
        wo.idx[k] = ptr<int32_t>(*lbuf[k]);
        wo.cap[k] = 0;
    }
    finish(false);
    ctx->hint_n_crit = ctx->prm.n_crit;
    walk_kernel<kEmit>(ctx)<<<grid, kWalkThreads, 0, st>>>(ptr<GroupInfo>(ctx->grp), G_dev,
                                                  ptr<NodeWalk>(ctx->node_walk), wp, wo, gstack,
                                                  lds_cap);
    if ((rc = check_hip(ctx, hipGetLastError(), "walk emit"))) return rc;
    return lists_done(ctx, build_order(ctx, stride));
}

}  // namespace p3t
