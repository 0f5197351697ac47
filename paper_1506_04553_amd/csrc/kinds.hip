// kinds.hip -- particle kinds for the SMBH runs (Section 3.2.2): the last
// n_special particles of the arrays are special; a pair of a normal and a
// special particle takes its own cutoff radii, softening and neighbour radius,
// and a pair of two special particles its own softening and, when it is not
// split, no soft part at all (the pair is integrated wholly by Hermite).
//
// The tree and its lists cover the normal particles only.  Here:
//   * the soft force and potential of every pair that involves a special
//     particle (O(N n_special) direct sums): added to the normal particles'
//     rows, written to the special particles' rows;
//   * the neighbour lists of all particles: a normal particle's tree row
//     followed by the special particles within the normal-special radius; a
//     special particle's row by the normal particles within that radius and
//     the other special particles (all of them when their pair is not split),
//     every row ascending.
// Special particles are few (the paper uses two), so one block per special
// particle sweeps the normal particles, in the launch whose other blocks take a
// normal particle per thread: these sweeps are as short as launches are for a few
// thousand particles.
#include <math.h>

#include "device_util.h"
#include "internal.h"

namespace p3t {

constexpr int kKindThreads = 1024;
constexpr int kKindWaves = kKindThreads / kWave;

// constants of one kind of pair for the soft sums
struct SoftPair {
    double eps2, inv_rout, gamma, inv_1mg, C_over_rout;
    double w[7];
    double wl, wm;
    int split;
};

struct KindsConsts {
    SoftPair ns, ss;
    int64_t first_sp, n;
};

static SoftPair soft_pair(double eps, double r_in, double r_out, int split) {
    SoftPair q{};
    q.eps2 = eps * eps;
    q.split = split;
    if (!split) return q;
    const Changeover c = make_changeover(r_in, r_out);
    q.inv_rout = c.inv_rout;
    q.gamma = c.gamma;
    q.inv_1mg = c.inv_1mg;
    q.C_over_rout = c.C * c.inv_rout;
    for (int k = 0; k < 7; ++k) q.w[k] = c.w[k];
    q.wl = c.wl;
    q.wm = c.wm;
    return q;
}

// soft pull of j on i: a += m_j K d / s^3, phi -= m_j W / s (FP64)
__device__ inline void soft_pull(const double *xi, const double *xj, double mj, const SoftPair &q,
                                 double a[3], double &ph) {
    if (!q.split) return;
    const double dx = xj[0] - xi[0], dy = xj[1] - xi[1], dz = xj[2] - xi[2];
    const double s2 = dx * dx + dy * dy + dz * dz + q.eps2;
    const double s = sqrt(s2);
    const double y = s * q.inv_rout;
    double K, Ws;
    if (y >= 1.0) {
        K = 1.0;
        Ws = 1.0 / s;
    } else if (y < q.gamma) {
        K = 0.0;
        Ws = q.C_over_rout;
    } else {
        const double x = (y - q.gamma) * q.inv_1mg;
        const double x2 = x * x;
        K = x2 * x2 * (35.0 + x * (-84.0 + x * (70.0 - 20.0 * x)));
        double p = q.w[6];
        for (int k = 5; k >= 0; --k) p = p * y + q.w[k];
        Ws = (p + q.wl * log(y) + q.wm / y) * q.inv_rout;
    }
    const double f = mj * K / (s2 * s);
    a[0] += f * dx;
    a[1] += f * dy;
    a[2] += f * dz;
    ph -= mj * Ws;
}

// Blocks of normal particles come first, then one for each special particle.
__host__ __device__ inline int64_t normal_blocks(int64_t first_sp) {
    return (first_sp + kKindThreads - 1) / kKindThreads;
}

// normal particles: add the pulls of the special particles (SHARE threads to a
// particle); special particles: the pulls of every other particle, summed over the
// block
template <int SHARE>
__global__ __launch_bounds__(kKindThreads) void k_kinds_soft(
    const double *__restrict__ pos, const double *__restrict__ mass, KindsConsts kc,
    double *__restrict__ acc, double *__restrict__ pot) {
    __shared__ double s_r[kKindWaves][4];
    const int64_t nb = normal_blocks(SHARE * kc.first_sp);
    double r[4] = {0.0, 0.0, 0.0, 0.0};          // a and phi
    if (blockIdx.x < nb) {
        const int64_t i = ((int64_t)blockIdx.x * kKindThreads + threadIdx.x) / SHARE;
        if (i >= kc.first_sp) return;
        const int part = threadIdx.x % SHARE;
        for (int64_t b = kc.first_sp + part; b < kc.n; b += SHARE)
            soft_pull(pos + 3 * i, pos + 3 * b, mass[b], kc.ns, r, r[3]);
        for (int d = 1; d < SHARE; d <<= 1)
            for (int q = 0; q < 4; ++q) r[q] += __shfl_xor(r[q], d, kWave);
        if (part != 0) return;
        for (int q = 0; q < 3; ++q) acc[3 * i + q] += r[q];
        if (pot) pot[i] += r[3];
        return;
    }
    const int64_t b = kc.first_sp + (blockIdx.x - nb);
    for (int64_t j = threadIdx.x; j < kc.n; j += kKindThreads) {
        if (j == b) continue;
        soft_pull(pos + 3 * b, pos + 3 * j, mass[j], j >= kc.first_sp ? kc.ss : kc.ns, r, r[3]);
    }
    for (int q = 0; q < 4; ++q) {
        r[q] = wave_sum(r[q]);
        if (threadIdx.x % kWave == 0) s_r[threadIdx.x / kWave][q] = r[q];
    }
    __syncthreads();
    if (threadIdx.x >= 4) return;
    double t = 0.0;
    for (int w = 0; w < kKindWaves; ++w) t += s_r[w][threadIdx.x];
    if (threadIdx.x < 3) acc[3 * b + threadIdx.x] = t;
    else if (pot) pot[b] = t;
}

// ---------------------------------------------------------------------------
// Neighbour lists with a radius per kind of pair.
// ---------------------------------------------------------------------------
struct KindsNbr {
    double h2_ns, h2_ss;
    int split_ss;
    int64_t first_sp, n;
};

__device__ inline bool within(const double *xi, const double *xj, double h2) {
    const double dx = xj[0] - xi[0], dy = xj[1] - xi[1], dz = xj[2] - xi[2];
    return dx * dx + dy * dy + dz * dz < h2;
}

// the special particles on special particle b's row
__device__ inline bool ss_listed(const double *pos, int64_t b, int64_t c, const KindsNbr &kn) {
    return c != b && (!kn.split_ss || within(pos + 3 * b, pos + 3 * c, kn.h2_ss));
}

// row lengths; cnt[n] = 0 for the scan
__global__ __launch_bounds__(kKindThreads) void k_kn_count(const double *__restrict__ pos,
                                                           const int64_t *__restrict__ nn_off,
                                                           KindsNbr kn, int64_t *__restrict__ cnt) {
    __shared__ int64_t s_c[kKindWaves];
    const int64_t nb = normal_blocks(kn.first_sp);
    if (blockIdx.x == 0 && threadIdx.x == 0) cnt[kn.n] = 0;
    int64_t c = 0;
    if (blockIdx.x < nb) {
        const int64_t i = (int64_t)blockIdx.x * kKindThreads + threadIdx.x;
        if (i >= kn.first_sp) return;
        c = nn_off[i + 1] - nn_off[i];
        for (int64_t b = kn.first_sp; b < kn.n; ++b)
            c += within(pos + 3 * i, pos + 3 * b, kn.h2_ns);
        cnt[i] = c;
        return;
    }
    const int64_t b = kn.first_sp + (blockIdx.x - nb);
    for (int64_t j = threadIdx.x; j < kn.first_sp; j += kKindThreads)
        c += within(pos + 3 * b, pos + 3 * j, kn.h2_ns);
    for (int64_t j = kn.first_sp + threadIdx.x; j < kn.n; j += kKindThreads)
        c += ss_listed(pos, b, j, kn);
    c = wave_sum(c);
    if (threadIdx.x % kWave == 0) s_c[threadIdx.x / kWave] = c;
    __syncthreads();
    if (threadIdx.x != 0) return;
    c = 0;
    for (int w = 0; w < kKindWaves; ++w) c += s_c[w];
    cnt[b] = c;
}

// The rows, ascending, and the caller's offsets.  A special particle's row is an
// ordered compaction of the hits over chunks of the block.
__global__ __launch_bounds__(kKindThreads) void k_kn_fill(
    const double *__restrict__ pos, const int64_t *__restrict__ nn_off,
    const int32_t *__restrict__ nn_idx, KindsNbr kn, const int64_t *__restrict__ start,
    int64_t *__restrict__ off, int32_t *__restrict__ idx) {
    __shared__ int s_hits[2][kKindWaves];
    const int64_t nb = normal_blocks(kn.first_sp);
    if (blockIdx.x == 0 && threadIdx.x == 0) off[kn.n] = start[kn.n];
    if (blockIdx.x < nb) {
        const int64_t i = (int64_t)blockIdx.x * kKindThreads + threadIdx.x;
        if (i >= kn.first_sp) return;
        int64_t o = start[i];
        off[i] = o;
        for (int64_t e = nn_off[i]; e < nn_off[i + 1]; ++e) idx[o++] = nn_idx[e];
        for (int64_t b = kn.first_sp; b < kn.n; ++b)
            if (within(pos + 3 * i, pos + 3 * b, kn.h2_ns)) idx[o++] = (int32_t)b;
        return;
    }
    const int64_t b = kn.first_sp + (blockIdx.x - nb);
    const int w = threadIdx.x / kWave;
    int64_t o = start[b];
    if (threadIdx.x == 0) off[b] = o;
    int side = 0;   // the counts of two chunks in turn: one barrier per chunk
    for (int64_t j0 = 0; j0 < kn.n; j0 += kKindThreads, side ^= 1) {
        const int64_t j = j0 + threadIdx.x;
        bool hit = false;
        if (j < kn.first_sp) hit = within(pos + 3 * b, pos + 3 * j, kn.h2_ns);
        else if (j < kn.n) hit = ss_listed(pos, b, j, kn);
        const uint64_t hits = ballot(hit);
        if (threadIdx.x % kWave == 0) s_hits[side][w] = __popcll(hits);
        __syncthreads();
        int64_t at = o + count_below(hits);
        for (int v = 0; v < kKindWaves; ++v) {
            at += v < w ? s_hits[side][v] : 0;
            o += s_hits[side][v];
        }
        if (hit) idx[at] = (int32_t)j;
    }
}

static KindsConsts kinds_consts(int64_t n, const p3t_kinds *kd) {
    KindsConsts kc;
    kc.ns = soft_pair(kd->eps_ns, kd->r_in_ns, kd->r_out_ns, 1);
    kc.ss = soft_pair(kd->eps_ss, kd->r_in_ss, kd->r_out_ss, kd->split_ss);
    kc.first_sp = n - kd->n_special;
    kc.n = n;
    return kc;
}

int launch_kinds_soft(p3t_ctx *ctx, int64_t n, const double *pos, const double *mass,
                      const p3t_params *p, const p3t_kinds *kd, double *acc, double *pot) {
    (void)p;
    if (!kd || kd->n_special == 0) return P3T_OK;
    const KindsConsts kc = kinds_consts(n, kd);
    // A normal particle's sum is a chain as long as the special particles are many, a
    // special one's as long as the normal blocks are: several threads to a normal
    // particle where its chain is the longer (us with 1, 4 and 16: 6000 particles, 64 of
    // them special, 43, 15 and 10; 30000, 128: 83, 31 and 41; 60000, 64: 53, 62 and 64;
    // 300000, 512: 973, 842 and 828).
    const int64_t blocks = normal_blocks(kc.first_sp);
    const int share = kd->n_special <= blocks + blocks / 4 ? 1 : kd->n_special <= 8 * blocks ? 4 : 16;
    auto kernel = share == 16 ? k_kinds_soft<16> : share == 4 ? k_kinds_soft<4> : k_kinds_soft<1>;
    kernel<<<(unsigned)(normal_blocks(share * kc.first_sp) + kd->n_special), kKindThreads, 0,
             ctx->stream>>>(pos, mass, kc, acc, pot);
    return check_hip(ctx, hipGetLastError(), "kinds soft");
}

// readback slot (int64 units) used here: the merged lists' total
enum { RB_KNNZ = 60 };

int launch_kinds_neighbors(p3t_ctx *ctx, int64_t n, const double *pos, const p3t_kinds *kd,
                           const int64_t *nn_off, const int32_t *nn_idx, int64_t *off,
                           int32_t *idx, int64_t cap, int64_t *nnz) {
    int rc;
    hipStream_t st = ctx->stream;
    if ((rc = ensure_readback(ctx))) return rc;
    if ((rc = ensure(ctx, ctx->kinds_cnt, (size_t)(n + 1) * sizeof(int64_t)))) return rc;
    int64_t *cnt = ptr<int64_t>(ctx->kinds_cnt);
    KindsNbr kn;
    kn.h2_ns = kd->r_search_ns * kd->r_search_ns;
    kn.h2_ss = kd->r_search_ss * kd->r_search_ss;
    kn.split_ss = kd->split_ss;
    kn.first_sp = n - kd->n_special;
    kn.n = n;
    const unsigned blocks = (unsigned)(normal_blocks(kn.first_sp) + kd->n_special);
    k_kn_count<<<blocks, kKindThreads, 0, st>>>(pos, nn_off, kn, cnt);
    if ((rc = check_hip(ctx, hipGetLastError(), "kinds count"))) return rc;
    if ((rc = scan_exclusive_i64(ctx, cnt, cnt, n + 1, ctx->hpin + RB_KNNZ))) return rc;
    if ((rc = check_hip(ctx, hipStreamSynchronize(st), "sync"))) return rc;
    const int64_t total = ctx->hpin[RB_KNNZ];
    *nnz = total;
    if (total > cap)
        return set_error(ctx, P3T_ECAPACITY, "neighbour capacity %lld < %lld", (long long)cap,
                         (long long)total);
    k_kn_fill<<<blocks, kKindThreads, 0, st>>>(pos, nn_off, nn_idx, kn, cnt, off, idx);
    return check_hip(ctx, hipGetLastError(), "kinds fill");
}

}  // namespace p3t
