// direct.hip -- O(N^2) direct summation of the softened force and potential
// over every pair, for energies and diagnostics (the exact sums the tree
// approximates; Section 2.1):
//   NEWTON  a_i = sum_{j != i} m_j d / s^3,            phi_i = -sum m_j / s
//   SOFT    a_i = sum m_j K(s) d / s^3,                 phi_i = -sum m_j W(s) / s
//   HARD    a_i = sum m_j (1 - K(s)) d / s^3,           phi_i = -sum m_j (1 - W(s)) / s
// with d = x_j - x_i, s^2 = |d|^2 + eps^2 and y = s / r_out.  FP64 throughout.
//
// Every pair is evaluated once for both of its particles (k_direct_pairs),
// except where no workspace can be had.  There (k_direct) a block of 256
// threads owns 512 i-particles (two per thread, two independent accumulation
// chains) and j-particles stream through LDS in tiles of 256 as 32-byte
// records.  Positions stay in L2, so both are bound by FP64 issue, not by HBM.
// Beyond r_out (almost every pair) K = W = 1: SOFT is the NEWTON pair, HARD
// contributes nothing, and the changeover polynomials run only inside r_out.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "device_util.h"
#include "internal.h"

namespace p3t {

constexpr int kDirThreads = 256;
constexpr int kDirPerThread = 2;
constexpr int kDirTile = 256;

struct DirectConsts {
    double eps2, rout2, inv_rout, gamma, inv_1mg, C_over_rout;
    double w[7];
    double wl, wm;
};

struct alignas(32) DJ {
    double x, y, z, m;
};

// 1/sqrt(x), x > 0: the hardware estimate r and one step of the series
// (1 - e)^(-1/2) = 1 + e/2 + 3e^2/8, e = 1 - x r^2, which cubes the estimate's
// relative error (~2^-22) to below the FP64 rounding level
__device__ __forceinline__ double rsq_nr(double x) {
    const double r = __builtin_amdgcn_rsq(x);
    const double e = __builtin_fma(-x * r, r, 1.0);
    return __builtin_fma(r * e, __builtin_fma(e, 0.375, 0.5), r);
}

// K(y) and W(y)/s on y < 1
__device__ __forceinline__ void changeover_in(double s, double rinv, const DirectConsts &dc,
                                              double &K, double &Ws) {
    const double y = s * dc.inv_rout;
    if (y < dc.gamma) {
        K = 0.0;
        Ws = dc.C_over_rout;
        return;
    }
    const double x = (y - dc.gamma) * dc.inv_1mg;
    const double x2 = x * x;
    K = x2 * x2 * __builtin_fma(x, __builtin_fma(x, __builtin_fma(x, -20.0, 70.0), -84.0), 35.0);
    double p = dc.w[6];
    for (int k = 5; k >= 0; --k) p = __builtin_fma(p, y, dc.w[k]);
    Ws = (p + dc.wl * log(y) + dc.wm / y) * dc.inv_rout;
    (void)rinv;
}

// SELF: the tile may hold particle i itself, whose pair is excluded (and kept
// finite when eps = 0)
template <int MODE, bool SELF>
__device__ __forceinline__ void pair(double xi, double yi, double zi, int64_t i, const DJ &j,
                                     int64_t jid, const DirectConsts &dc, double a[4]) {
    const double dx = j.x - xi, dy = j.y - yi, dz = j.z - zi;
    double r2 = __builtin_fma(dx, dx, __builtin_fma(dy, dy, __builtin_fma(dz, dz, dc.eps2)));
    double mf = j.m;
    if (SELF && jid == i) {
        mf = 0.0;
        r2 = 1.0;
    }
    const double rinv = rsq_nr(r2);
    if (MODE == P3T_DIRECT_NEWTON) {
        const double mr = mf * rinv;
        const double mr3 = mr * rinv * rinv;
        a[0] = __builtin_fma(mr3, dx, a[0]);
        a[1] = __builtin_fma(mr3, dy, a[1]);
        a[2] = __builtin_fma(mr3, dz, a[2]);
        a[3] -= mr;
        return;
    }
    if (r2 >= dc.rout2) {                  // K = W = 1
        if (MODE == P3T_DIRECT_SOFT) {
            const double mr = mf * rinv;
            const double mr3 = mr * rinv * rinv;
            a[0] = __builtin_fma(mr3, dx, a[0]);
            a[1] = __builtin_fma(mr3, dy, a[1]);
            a[2] = __builtin_fma(mr3, dz, a[2]);
            a[3] -= mr;
        }
        return;
    }
    double K, Ws;
    changeover_in(r2 * rinv, rinv, dc, K, Ws);
    const double kf = MODE == P3T_DIRECT_SOFT ? K : 1.0 - K;
    const double wf = MODE == P3T_DIRECT_SOFT ? Ws : rinv - Ws;
    const double f = mf * kf * rinv * rinv * rinv;
    a[0] = __builtin_fma(f, dx, a[0]);
    a[1] = __builtin_fma(f, dy, a[1]);
    a[2] = __builtin_fma(f, dz, a[2]);
    a[3] -= mf * wf;
}

template <int MODE>
__global__ __launch_bounds__(kDirThreads) void k_direct(int64_t n, const double *__restrict__ pos,
                                                       const double *__restrict__ mass,
                                                       DirectConsts dc, double *__restrict__ acc,
                                                       double *__restrict__ pot) {
    __shared__ DJ s_j[kDirTile];
    const int tid = threadIdx.x;
    int64_t ii[kDirPerThread];
    double xi[kDirPerThread], yi[kDirPerThread], zi[kDirPerThread];
    double a[kDirPerThread][4];
#pragma unroll
    for (int q = 0; q < kDirPerThread; ++q) {
        const int64_t i = (int64_t)blockIdx.x * (kDirThreads * kDirPerThread) + q * kDirThreads + tid;
        ii[q] = i;
        const int64_t ic = i < n ? i : n - 1;
        xi[q] = pos[3 * ic];
        yi[q] = pos[3 * ic + 1];
        zi[q] = pos[3 * ic + 2];
        a[q][0] = a[q][1] = a[q][2] = a[q][3] = 0.0;
    }
    for (int64_t t0 = 0; t0 < n; t0 += kDirTile) {
        const int tl = (int)min<int64_t>(kDirTile, n - t0);
        __syncthreads();
        if (tid < tl) {
            const int64_t j = t0 + tid;
            s_j[tid] = DJ{pos[3 * j], pos[3 * j + 1], pos[3 * j + 2], mass[j]};
        }
        __syncthreads();
        // only the tiles that overlap the block's own particles can hold i
        const int64_t i0 = (int64_t)blockIdx.x * (kDirThreads * kDirPerThread);
        if (t0 + tl > i0 && t0 < i0 + kDirThreads * kDirPerThread) {
            for (int k = 0; k < tl; ++k) {
                const DJ jj = s_j[k];
#pragma unroll
                for (int q = 0; q < kDirPerThread; ++q)
                    pair<MODE, true>(xi[q], yi[q], zi[q], ii[q], jj, t0 + k, dc, a[q]);
            }
        } else {
            for (int k = 0; k < tl; ++k) {
                const DJ jj = s_j[k];
#pragma unroll
                for (int q = 0; q < kDirPerThread; ++q)
                    pair<MODE, false>(xi[q], yi[q], zi[q], ii[q], jj, t0 + k, dc, a[q]);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < kDirPerThread; ++q) {
        const int64_t i = ii[q];
        if (i >= n) continue;
        acc[3 * i] = a[q][0];
        acc[3 * i + 1] = a[q][1];
        acc[3 * i + 2] = a[q][2];
        if (pot) pot[i] = a[q][3];
    }
}

// ---------------------------------------------------------------------------
// The same sums with every pair evaluated once for both of its particles.
//
// The particles form nb blocks of B = 64 K WAVES.  Item (x, d) takes the pairs
// of block x with block y = x + d (mod nb): d = 0 the block with itself (every
// ordered pair), d = 1 .. nb / 2 each pair of blocks once.  A wavefront keeps K
// particles per lane; 64 particles of y at a time meet them in 64 steps: lane l
// meets particle (l + s) mod 64 in step s, read from LDS (stored twice, so that
// the steps read at immediate offsets), and the sums of y's particles move on
// by one lane per step.  The pair costs 24 FP64 operations and 1/K of eight
// lane moves where two one-sided evaluations cost 38, and FP64 issue is the
// bound: 2^18 particles, Newton 46.4 -> 28.6 ms, soft 62.2 -> 31.4, hard
// 30.3 -> 11.5.  The one-sided kernel also has too few blocks for fewer
// particles: 65536, Newton, 6.6 -> 1.9 ms; 4096, 420 -> 39 us.
// Three wavefronts per SIMD hold Newton's registers (158) without spilling,
// two those of the changeover.
//
// Each item writes its sums of x's and of y's particles to rows of its own, so
// the order of every addition is fixed; k_direct_add adds the rows of a launch.
// The distances go in launches of as many as the workspace's rows allow.
// ---------------------------------------------------------------------------
struct alignas(32) Sum4 {
    double x, y, z, p;
};

// lane l gets lane l + 1's value, lane 63 lane 0's
__device__ __forceinline__ double rotate_lanes(double v) { return dpp_src<0x134>(v); }

// The pair's factors: acceleration of i is m_j f d, its potential -m_j w.  False
// where the pair adds nothing, which is not the same as adding zero times a mass or
// an offset that is not finite.
template <int MODE>
__device__ __forceinline__ bool pair_factors(double r2, const DirectConsts &dc, double &f,
                                             double &w) {
    if (MODE == P3T_DIRECT_NEWTON) {
        w = rsq_nr(r2);
        f = w * w * w;
        return true;
    }
    const bool near = !(r2 >= dc.rout2);
    if (MODE == P3T_DIRECT_HARD && !near) return false;
    const double rinv = rsq_nr(r2);
    f = rinv * rinv * rinv;
    w = rinv;
    if (near) {
        double K, Ws;
        changeover_in(r2 * rinv, rinv, dc, K, Ws);
        f *= MODE == P3T_DIRECT_SOFT ? K : 1.0 - K;
        w = MODE == P3T_DIRECT_SOFT ? Ws : rinv - Ws;
    }
    return true;
}

// Whether any lane has a particle within r_out of (x, y, z) (HARD: the others add
// nothing).  One branch for a lane's K pairs, most of which are farther apart: 11.1 ms
// for 2^18 particles, where one for each took 18.2.
template <int K>
__device__ __forceinline__ bool any_near(const DJ xi[K], double x, double y, double z,
                                         const DirectConsts &dc) {
    bool near = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const double dx = x - xi[k].x, dy = y - xi[k].y, dz = z - xi[k].z;
        const double r2 =
            __builtin_fma(dx, dx, __builtin_fma(dy, dy, __builtin_fma(dz, dz, dc.eps2)));
        near |= !(r2 >= dc.rout2);
    }
    return __builtin_amdgcn_ballot_w64(near) != 0;
}

template <int MODE, int K, int WAVES>
__global__ __launch_bounds__(WAVES * kWave)
__attribute__((amdgpu_waves_per_eu(MODE == P3T_DIRECT_NEWTON ? 3 : 2))) void k_direct_pairs(
    int64_t n, int32_t nb, int32_t d0, const double *__restrict__ pos,
    const double *__restrict__ mass, DirectConsts dc, Sum4 *__restrict__ rows, int64_t np) {
    constexpr int kOwn = K * kWave, B = kOwn * WAVES;
    __shared__ double2 s_xy[2][2 * kWave], s_zm[2][2 * kWave];
    __shared__ Sum4 s_j[WAVES > 1 ? WAVES : 1][kWave];
    const int tid = threadIdx.x, w = tid / kWave, lane = tid % kWave;
    const int32_t x = blockIdx.x, d = d0 + blockIdx.y;
    // distance nb / 2 of an even number of blocks meets every pair twice
    if (2 * d == nb && d > 0 && x >= d) return;
    const int32_t y = x + d < nb ? x + d : x + d - nb;
    const bool sym = d > 0;
    Sum4 *const row_x = rows + (int64_t)(2 * blockIdx.y) * np + (int64_t)x * B;
    Sum4 *const row_y = rows + (int64_t)(2 * blockIdx.y + 1) * np + (int64_t)y * B;

    // Padding particles are massless and lie where the last particle does: wherever the
    // others are, they are as far from them as that one, and their terms are zero.
    // (It meets them in its own block alone, which leaves them out.)
    auto load = [&](int64_t i) {
        const int64_t p = i < n ? i : n - 1;
        return DJ{pos[3 * p], pos[3 * p + 1], pos[3 * p + 2], i < n ? mass[i] : 0.0};
    };
    DJ xi[K];
    Sum4 ai[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        xi[k] = load((int64_t)x * B + w * kOwn + k * kWave + lane);
        ai[k] = Sum4{0.0, 0.0, 0.0, 0.0};
    }
    constexpr int kChunks = B / kWave;
    DJ pre = tid < kWave ? load((int64_t)y * B + tid) : DJ{0.0, 0.0, 0.0, 0.0};
    for (int c = 0; c < kChunks; ++c) {
        const int buf = c & 1;
        if (tid < kWave) {
            s_xy[buf][tid] = s_xy[buf][tid + kWave] = double2{pre.x, pre.y};
            s_zm[buf][tid] = s_zm[buf][tid + kWave] = double2{pre.z, pre.m};
            if (c + 1 < kChunks) pre = load((int64_t)y * B + (c + 1) * kWave + tid);
        }
        __syncthreads();
        const double2 *xy = s_xy[buf] + lane, *zm = s_zm[buf] + lane;
        if (sym) {
            Sum4 aj{0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
            for (int s = 0; s < kWave; ++s) {
                const double2 a = xy[s], b = zm[s];
                const bool some = MODE != P3T_DIRECT_HARD || any_near<K>(xi, a.x, a.y, b.x, dc);
#pragma unroll
                for (int k = 0; k < K && some; ++k) {
                    const double dx = a.x - xi[k].x, dy = a.y - xi[k].y, dz = b.x - xi[k].z;
                    const double r2 = __builtin_fma(
                        dx, dx, __builtin_fma(dy, dy, __builtin_fma(dz, dz, dc.eps2)));
                    double f, ph;
                    if (!pair_factors<MODE>(r2, dc, f, ph)) continue;
                    const double fi = b.y * f, fj = -xi[k].m * f;
                    ai[k].x = __builtin_fma(fi, dx, ai[k].x);
                    ai[k].y = __builtin_fma(fi, dy, ai[k].y);
                    ai[k].z = __builtin_fma(fi, dz, ai[k].z);
                    ai[k].p = __builtin_fma(-b.y, ph, ai[k].p);
                    aj.x = __builtin_fma(fj, dx, aj.x);
                    aj.y = __builtin_fma(fj, dy, aj.y);
                    aj.z = __builtin_fma(fj, dz, aj.z);
                    aj.p = __builtin_fma(-xi[k].m, ph, aj.p);
                }
                aj = Sum4{rotate_lanes(aj.x), rotate_lanes(aj.y), rotate_lanes(aj.z),
                          rotate_lanes(aj.p)};
            }
            // after 64 moves the sums of particle `lane` are back in its lane
            if (WAVES == 1) {
                row_y[c * kWave + lane] = aj;
            } else {
                s_j[w][lane] = aj;
                __syncthreads();
                if (tid < kWave) {
                    Sum4 t = s_j[0][tid];
#pragma unroll
                    for (int v = 1; v < WAVES; ++v) {
                        const Sum4 o = s_j[v][tid];
                        t.x += o.x; t.y += o.y; t.z += o.z; t.p += o.p;
                    }
                    row_y[c * kWave + tid] = t;
                }
            }
        } else {
            const int64_t left = n - ((int64_t)y * B + c * kWave);
            auto own = [&](auto part) {
                constexpr bool PART = decltype(part)::value;   // padding among the 64
                for (int s = 0; s < kWave; ++s) {
                    if (PART && ((lane + s) & (kWave - 1)) >= left) continue;
                    const double2 a = xy[s], b = zm[s];
                    if (MODE == P3T_DIRECT_HARD && !any_near<K>(xi, a.x, a.y, b.x, dc)) continue;
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        // a particle meets itself in step 0 of its own 64
                        if (s == 0 && w * K + k == c) continue;
                        const double dx = a.x - xi[k].x, dy = a.y - xi[k].y, dz = b.x - xi[k].z;
                        const double r2 = __builtin_fma(
                            dx, dx, __builtin_fma(dy, dy, __builtin_fma(dz, dz, dc.eps2)));
                        double f, ph;
                        if (!pair_factors<MODE>(r2, dc, f, ph)) continue;
                        const double fi = b.y * f;
                        ai[k].x = __builtin_fma(fi, dx, ai[k].x);
                        ai[k].y = __builtin_fma(fi, dy, ai[k].y);
                        ai[k].z = __builtin_fma(fi, dz, ai[k].z);
                        ai[k].p = __builtin_fma(-b.y, ph, ai[k].p);
                    }
                }
            };
            if (left < kWave) own(std::true_type());
            else own(std::false_type());
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) row_x[w * kOwn + k * kWave + lane] = ai[k];
}

// acc, pot = (their values, unless FIRST) + the rows of distances d0 .. d0 + nd - 1
template <bool FIRST>
__global__ __launch_bounds__(kDirThreads) void k_direct_add(int64_t n, int32_t nb, int32_t block,
                                                           int32_t d0, int32_t nd,
                                                           const Sum4 *__restrict__ rows, int64_t np,
                                                           double *__restrict__ acc,
                                                           double *__restrict__ pot) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t x = (int32_t)(i / block);
    Sum4 t{0.0, 0.0, 0.0, 0.0};
    auto add = [&](int32_t row) {
        const Sum4 o = rows[(int64_t)row * np + i];
        t.x += o.x; t.y += o.y; t.z += o.z; t.p += o.p;
    };
    for (int32_t s = 0; s < nd; ++s) {
        const int32_t d = d0 + s;
        const bool half = d > 0 && 2 * d == nb;
        if (!half || x < d) add(2 * s);
        if (d > 0 && (!half || x >= d)) add(2 * s + 1);
    }
    if (!FIRST) {
        t.x += acc[3 * i]; t.y += acc[3 * i + 1]; t.z += acc[3 * i + 2];
    }
    acc[3 * i] = t.x;
    acc[3 * i + 1] = t.y;
    acc[3 * i + 2] = t.z;
    if (pot) pot[i] = FIRST ? t.p : t.p + pot[i];
}

// workspace of the rows (at least one distance's)
constexpr int64_t kDirRows = (int64_t)256 << 20;

template <int MODE, int K, int WAVES>
static int direct_pairs(p3t_ctx *ctx, int64_t n, const double *pos, const double *mass,
                        const DirectConsts &dc, double *acc, double *pot) {
    constexpr int B = K * kWave * WAVES;
    const int64_t nb = (n + B - 1) / B, np = nb * B, dist = nb / 2 + 1;
    int64_t per = kDirRows / (2 * np * (int64_t)sizeof(Sum4));
    per = std::max<int64_t>(1, std::min(per, dist));
    int rc;
    if ((rc = ensure(ctx, ctx->direct_rows, (size_t)(2 * per * np) * sizeof(Sum4)))) return rc;
    Sum4 *rows = ptr<Sum4>(ctx->direct_rows);
    for (int64_t d0 = 0; d0 < dist; d0 += per) {
        const int nd = (int)std::min(per, dist - d0);
        k_direct_pairs<MODE, K, WAVES><<<dim3((unsigned)nb, (unsigned)nd), WAVES * kWave, 0,
                                         ctx->stream>>>(n, (int32_t)nb, (int32_t)d0, pos, mass, dc,
                                                        rows, np);
        auto add = d0 == 0 ? k_direct_add<true> : k_direct_add<false>;
        add<<<blocks_for(n, kDirThreads), kDirThreads, 0, ctx->stream>>>(
            n, (int32_t)nb, B, (int32_t)d0, nd, rows, np, acc, pot);
    }
    return check_hip(ctx, hipGetLastError(), "direct");
}

template <int MODE>
static int launch_direct_mode(p3t_ctx *ctx, int64_t n, const double *pos, const double *mass,
                              const DirectConsts &dc, double *acc, double *pot) {
    // The rows are a workspace: a call that is being captured (which must not
    // allocate, nor keep the address of memory that a later call may replace)
    // and one whose rows cannot be had evaluate both sides of every pair.
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    const bool plain = hipStreamIsCapturing(ctx->stream, &cap) == hipSuccess &&
                       cap == hipStreamCaptureStatusNone;
    if (plain) {
        // Blocks of 64 particles while blocks of 256 would leave most of the GPU
        // idle (us, Newton / soft / hard: 4000 particles 39 / 68 / 34 against 71 / 90 /
        // 46, 5000 54 / 109 / 44 against 73 / 91 / 49, 7000 75 / 169 / 60 against 78 /
        // 102 / 53; one line between the three modes' own), then of 256, then of 1024,
        // whose rows are the shortest (40000 particles 746 / 797 / 334 with 256
        // against 873 / 1038 / 382, 49152 1114 / 1197 / 500 against 1104 / 1290 / 482,
        // 80000 2812 / 3036 / 1232 against 2822 / 3175 / 1160; 2^18 take 9 launches
        // instead of 33).
        const int rc = n <= 5000 ? direct_pairs<MODE, 1, 1>(ctx, n, pos, mass, dc, acc, pot)
                     : n <= 49152 ? direct_pairs<MODE, 4, 1>(ctx, n, pos, mass, dc, acc, pot)
                                  : direct_pairs<MODE, 4, 4>(ctx, n, pos, mass, dc, acc, pot);
        if (rc != P3T_ENOMEM) return rc;
    } else {
        (void)hipGetLastError();
    }
    k_direct<MODE><<<blocks_for(n, kDirThreads * kDirPerThread), kDirThreads, 0, ctx->stream>>>(
        n, pos, mass, dc, acc, pot);
    return check_hip(ctx, hipGetLastError(), "direct");
}

int launch_direct(p3t_ctx *ctx, int64_t n, const double *pos, const double *mass,
                  const p3t_params *p, int mode, double *acc, double *pot) {
    const Changeover c = make_changeover(p->r_in, p->r_out);
    DirectConsts dc{};
    dc.eps2 = p->eps * p->eps;
    dc.rout2 = p->r_out * p->r_out;
    dc.inv_rout = c.inv_rout;
    dc.gamma = c.gamma;
    dc.inv_1mg = c.inv_1mg;
    dc.C_over_rout = c.C * c.inv_rout;
    for (int k = 0; k < 7; ++k) dc.w[k] = c.w[k];
    dc.wl = c.wl;
    dc.wm = c.wm;
    if (mode == P3T_DIRECT_NEWTON)
        return launch_direct_mode<P3T_DIRECT_NEWTON>(ctx, n, pos, mass, dc, acc, pot);
    if (mode == P3T_DIRECT_SOFT)
        return launch_direct_mode<P3T_DIRECT_SOFT>(ctx, n, pos, mass, dc, acc, pot);
    return launch_direct_mode<P3T_DIRECT_HARD>(ctx, n, pos, mass, dc, acc, pot);
}

}  // namespace p3t
