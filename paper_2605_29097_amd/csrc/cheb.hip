// Term sums of signal tracing and the matched filter (Eq. ref_sim, Eq. mf-sm
// and their adjoints) evaluated through Chebyshev moments of the residual
// range.  Same sums as the per-frequency kernels (render.hip, mf.hip), fewer
// operations per (measurement, point) pair.
//
// A pair's phasor at frequency n is exp(s j 2 pi (K0 + n Kd) r), s = -1 for
// the reductions over points (render forward, filter adjoint) and +1 for the
// reductions over frequencies (filter forward, render adjoint).  It is split at
// the centre of the band, Kc = K0 + nc Kd with nc = (n_freq - 1) / 2, and
// dn = n - nc in [-nc, nc].  Every point of a launch lies in an axis-aligned
// box, so for measurement i its range r lies in [rc_i - h_i, rc_i + h_i]
// (distances from the transmitter to the box; for a bistatic pair r is the
// mean of the distances from the transmitter and to the receiver, and the band
// the mean of their two bands).  With x = (r - rc) / h in
// [-1, 1] and z_n = 2 pi dn Kd h (of either sign),
//   exp(s j 2 pi dn Kd r) = exp(s j 2 pi dn Kd rc) exp(s j z_n x)
// and the Jacobi-Anger expansion
//   exp(s j z x) = sum_k eps_k (s j)^k J_k(z) T_k(x),  eps_0 = 1, eps_k = 2,
// (T_k Chebyshev polynomials, J_k Bessel functions of the first kind, with
// J_k(-z) = (-1)^k J_k(z)) turns
//   * a reduction over points into K moments per measurement,
//       M_ik = sum_j a_ij exp(-j 2 pi Kc r_ij) T_k(x_ij),
//       out[i][n] = exp(-j 2 pi dn Kd rc_i) sum_k eps_k (-j)^k J_k(z_in) M_ik;
//   * a reduction over frequencies into a Chebyshev series per measurement,
//       B_ik = eps_k j^k sum_n g[i][n] exp(+j 2 pi dn Kd rc_i) J_k(z_in),
//       sum_n g[i][n] exp(+j 2 pi (K0 + n Kd) r) = exp(+j 2 pi Kc r) sum_k B_ik T_k(x),
//     evaluated per pair with T_k from their three-term recurrence.
// Centring the band halves the largest |z| (against splitting at f0), and with
// it the number of orders the series needs.  Since |T_k| <= 1 on [-1, 1] and
// |J_k(z)| <= (|z|/2)^k / k!, cutting the series at K changes each output by at
// most 2 (z/2)^K / K! / (1 - z / (2K + 2)) (z = max |z_n|) times the sum of the
// magnitudes of its terms' weights.  A one-block plan kernel takes the largest
// z of the launch and picks the smallest K of kChebKs whose
// bound is below 1e-6, or 0 (the per-frequency kernels) when none is (a
// wide range spread) or K is not below the number of frequencies.  The choice
// stays on the device: every candidate kernel is launched and all but the
// chosen one return at once, so no host synchronisation is needed.
//
// Per pair both cost 3 FP32 operations per order (recurrence of T_k and a
// complex multiply-add by a real), against 4 per frequency in the
// per-frequency kernels; the FP64 range and the one phasor exp(-+j 2 pi Kc r)
// (hardware sin / cos of the FP64-reduced phase, at Kc) are set up once per pair.
// The Bessel coefficients themselves are not formed: interpolation at a few
// Chebyshev nodes more than orders gives the same series (k_cheb_coef, k_cheb_out).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "rfvr_impl.hpp"

namespace rfvr {

constexpr int kChebKs[] = {24, 28, 32, 40, 48, 64};
constexpr int kChebKMax = kChebMaxOrder;
// truncation bound, relative to the sum of the term magnitudes: of the order of
// the FP32 rounding of the sums themselves (a lane's moments accumulate a point
// split in FP32, 2048 points at 2^20 x 1024; with cells runs of 64)
constexpr double kChebLogTol = -13.815510557964274;   // log 1e-6
// ... and of the box's series where cells add their own cut to it, so that both
// together stay within the same 1e-6 (orders of the box cost nothing per pair there)
constexpr double kChebCellsLogTol = -14.508657738524219;   // log 5e-7

// ---------------------------------------------------------------------------
// bounding box of a launch's points: per-block min / max, then the plan
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_bbox_partial(const float* __restrict__ xyz, long n, long per,
                                                      float* __restrict__ part) {
    __shared__ float s[6][256];
    const int t = threadIdx.x;
    const long b0 = (long)blockIdx.x * per;
    long b1 = b0 + per;
    if (b1 > n) b1 = n;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (long j = b0 + t; j < b1; j += 256) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float v = xyz[3 * j + c];
            lo[c] = fminf(lo[c], v);
            hi[c] = fmaxf(hi[c], v);
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        s[c][t] = lo[c];
        s[3 + c][t] = hi[c];
    }
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                s[c][t] = fminf(s[c][t], s[c][t + w]);
                s[3 + c][t] = fmaxf(s[3 + c][t], s[3 + c][t + w]);
            }
        }
        __syncthreads();
    }
    if (t < 6) part[(long)blockIdx.x * 6 + t] = s[t][0];
}

// log K! of the candidate orders
constexpr int kChebNK = (int)(sizeof(kChebKs) / sizeof(kChebKs[0]));
__device__ constexpr double kChebLogFact[] = {54.784729398112319, 67.889743137181540, 81.557959456115037,
                                              110.32063971475740, 140.67392364823426, 205.16819948264120};
static_assert(sizeof(kChebLogFact) / sizeof(double) == kChebNK, "one per order");

// orders of a cell's series and log K!; 2.5e-7 bounds 2 (z/2)^K / K! / (1 - ...)
// there: interpolation at K nodes is within twice that of the function
constexpr int kCellKs[] = {8, 10, 12, 14, 16};
constexpr int kCellNK = (int)(sizeof(kCellKs) / sizeof(kCellKs[0]));
static_assert(kCellKs[kCellNK - 1] < kChebKs[0], "cells take fewer orders than any box");
__device__ constexpr double kCellLogFact[] = {10.604602902745250, 15.104412573075516, 19.987214495661885,
                                              25.191221182738680, 30.671860106080672};
constexpr double kCellLogTol = -15.201804919084164;   // log 2.5e-7

// log of 2 (z/2)^K / K! / (1 - z/(2K+2)), the truncation bound; +inf when the
// geometric tail does not converge
__device__ double cheb_log_bound(int K, double log_fact, double z) {
    const double q = 0.5 * z;
    if (q <= 0.0) return -INFINITY;
    if (q >= (double)(K + 1)) return INFINITY;
    return (double)K * log(q) - log_fact + 0.69314718055994531 - log1p(-q / (double)(K + 1));
}

// The launch's plan, one work-group: the measurement records (transmitters, and
// receivers of a bistatic aperture), the bounding box of the points (from the
// partials of k_bbox_partial, or for nb = 0 from the few points themselves), each
// measurement's range interval, and the order.
constexpr int kPlanThreads = 1024;
__global__ __launch_bounds__(kPlanThreads) void k_cheb_plan(const float* __restrict__ xyz, long n,
                                                            const float* __restrict__ part, int nb,
                                                            const float* __restrict__ tx, const float* __restrict__ phi_tx,
                                                            const float* __restrict__ rx, const float* __restrict__ phi_rx,
                                                            AntRec* __restrict__ ant, AntRec* __restrict__ rxa,
                                                            int n_meas, double Kd, int n_freq,
                                                            MeasCheb* __restrict__ meas, ChebPlan* __restrict__ plan,
                                                            CellGrid* __restrict__ grid, int max_cells) {
    __shared__ float sf[6][kPlanThreads / 64];
    __shared__ double sz[kPlanThreads / 64];
    static_assert(kPlanThreads == 1024, "16 waves");
    const int t = threadIdx.x;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (nb == 0) {
        // four points at a time (the last one repeated): one wait on memory per 4096
        for (long j0 = t; j0 < n; j0 += 4 * kPlanThreads) {
            float v[4][3];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const long j = min(j0 + u * kPlanThreads, n - 1);
#pragma unroll
                for (int c = 0; c < 3; ++c) v[u][c] = xyz[3 * j + c];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    lo[c] = fminf(lo[c], v[u][c]);
                    hi[c] = fmaxf(hi[c], v[u][c]);
                }
        }
    } else {
        for (int b = t; b < nb; b += kPlanThreads) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                lo[c] = fminf(lo[c], part[6 * b + c]);
                hi[c] = fmaxf(hi[c], part[6 * b + 3 + c]);
            }
        }
    }
    // the six extremes of the work-group, side by side: over the wave, then its 16 waves'
    // in every 16 lanes
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            lo[c] = fminf(lo[c], __shfl_xor(lo[c], o, 64));
            hi[c] = fmaxf(hi[c], __shfl_xor(hi[c], o, 64));
        }
    if ((t & 63) == 0)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            sf[c][t >> 6] = lo[c];
            sf[3 + c][t >> 6] = hi[c];
        }
    __syncthreads();
    double bl[3], bh[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        lo[c] = sf[c][t & 15];
        hi[c] = sf[3 + c][t & 15];
    }
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            lo[c] = fminf(lo[c], __shfl_xor(lo[c], o, 64));
            hi[c] = fmaxf(hi[c], __shfl_xor(hi[c], o, 64));
        }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        bl[c] = (double)lo[c];
        bh[c] = (double)hi[c];
    }
    const bool finite = isfinite(bl[0]) && isfinite(bl[1]) && isfinite(bl[2]) && isfinite(bh[0]) &&
                        isfinite(bh[1]) && isfinite(bh[2]);
    // distances from an antenna to the box: nearest face, farthest corner
    auto band = [&](const AntRec& a, double& lo_, double& hi_) {
        const double p[3] = {a.x, a.y, a.z};
        double n2 = 0.0, f2 = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double qn = fmax(fmax(bl[c] - p[c], p[c] - bh[c]), 0.0);
            const double qf = fmax(fabs(p[c] - bl[c]), fabs(p[c] - bh[c]));
            n2 += qn * qn;
            f2 += qf * qf;
        }
        lo_ = sqrt(n2);
        hi_ = sqrt(f2);
    };
    auto record = [](const float* x, const float* phi, int i) {
        AntRec a;
        a.x = (double)x[3 * i];
        a.y = (double)x[3 * i + 1];
        a.z = (double)x[3 * i + 2];
        a.phi = phi ? phi[i] : 0.0f;
        a.pad = 0.0f;
        return a;
    };
    double zl = 0.0;
    for (int i = t; i < n_meas; i += kPlanThreads) {
        double rlo, rhi;
        const AntRec a = record(tx, phi_tx, i);
        ant[i] = a;
        band(a, rlo, rhi);
        if (rxa) {
            double lo2, hi2;
            const AntRec r = record(rx, phi_rx, i);
            rxa[i] = r;
            band(r, lo2, hi2);
            rlo = 0.5 * (rlo + lo2);
            rhi = 0.5 * (rhi + hi2);
        }
        MeasCheb m;
        m.rc = 0.5 * (rlo + rhi);
        // margin for the rounding of the per-pair FP64 range (relative ~1e-14)
        m.h = 0.5 * (rhi - rlo) * (1.0 + 1e-12) + 1e-12 * (rhi + 1.0);
        m.inv_h = 1.0 / m.h;
        m.pad = 0.0;
        meas[i] = m;
        zl = fmax(zl, 6.283185307179586 * (0.5 * (double)(n_freq - 1)) * Kd * m.h);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) zl = fmax(zl, __shfl_xor(zl, o, 64));
    if ((t & 63) == 0) sz[t >> 6] = zl;
    __syncthreads();
    double zmax = sz[t & 15];
#pragma unroll
    for (int o = 8; o >= 1; o >>= 1) zmax = fmax(zmax, __shfl_xor(zmax, o, 64));
    // one lane per candidate order, the smallest that qualifies
    if (t < 64) {
        const int c = t < kChebNK ? t : kChebNK - 1, k = kChebKs[c];
        const bool fits = t < kChebNK && finite && k < n_freq;
        const double bound = cheb_log_bound(k, kChebLogFact[c], zmax);
        const unsigned long long m = __ballot(fits && bound <= kChebLogTol), mc = __ballot(fits && bound <= kChebCellsLogTol);
        int KC = 0;
        if (grid && mc) {
            // the finest of 1 .. 64 divisions of the box's longest edge, the others
            // cut alike, that gives at most max_cells cells
            const double e[3] = {bh[0] - bl[0], bh[1] - bl[1], bh[2] - bl[2]};
            const double s = fmax(fmax(e[0], e[1]), e[2]) / (double)(t + 1);
            int d[3];
#pragma unroll
            for (int c2 = 0; c2 < 3; ++c2) d[c2] = s > 0.0 ? max(1, (int)ceil(e[c2] / s - 1e-6)) : 1;
            const unsigned long long fit = __ballot((long)d[0] * d[1] * d[2] <= max_cells);
            if (t == 63 - __clzll(fit)) {
                double diag = 0.0;
                CellGrid g;
#pragma unroll
                for (int c2 = 0; c2 < 3; ++c2) {
                    const double w = e[c2] / d[c2];
                    g.n[c2] = d[c2];
                    g.lo[c2] = bl[c2];
                    g.w[c2] = w;
                    g.inv_w[c2] = w > 0.0 ? (float)(1.0 / w) : 0.0f;
                    diag += w * w;
                }
                g.n_cells = d[0] * d[1] * d[2];
                // |range| changes by at most the distance moved, so no interval is
                // wider than the cell's diagonal
                const double h = 0.5 * sqrt(diag) * (1.0 + 1e-5) + 1e-6;
                const double z = 6.283185307179586 * (0.5 * (double)(n_freq - 1)) * Kd * h;
                KC = 0;
                if (g.n_cells > 1)
                    for (int q = kCellNK - 1; q >= 0; --q)
                        if (cheb_log_bound(kCellKs[q], kCellLogFact[q], z) <= kCellLogTol) KC = kCellKs[q];
                *grid = g;
            }
            KC = __shfl(KC, 63 - __clzll(fit), 64);
        }
        if (t == 0) {
            ChebPlan p;
            p.K = m ? kChebKs[__ffsll(KC ? mc : m) - 1] : 0;
            p.KC = KC;                           // below every order of the box
            p.zmax = zmax;
            *plan = p;
        }
    }
}

// ---------------------------------------------------------------------------
// moments over points: signal tracing forward (KIND 0) and filter adjoint
// (KIND 1).  Lane = measurement; the lanes of a work-group walk the same point
// records in step, read as wave-uniform scalar loads; point splits dealt over
// the XCDs as in the per-frequency kernel.
// partial[split][meas][kChebKMax] (k < K written).
// ---------------------------------------------------------------------------
// a pair's range and weight (without its phase) in the point reductions
template <int KIND, int SPEC, bool BI, class Rec>
__device__ __forceinline__ void pair_weight(const Rec& rec, const AntRec& A, const AntRec& Rx, double& r, float& cr, float& ci) {
    if constexpr (KIND == 0 && !BI) {
        const PtRec& P = rec;
        const double dx = P.x - A.x, dy = P.y - A.y, dz = P.z - A.z;
        float y;
        r = range_f64(dx, dy, dz, y);
        float spec, live;
        if constexpr (SPEC == (int)RFVR_SPEC_OFF) {
            spec = 1.0f;
        } else {
            const float nd = (P.nx * (float)dx + P.ny * (float)dy + P.nz * (float)dz) * y;
            spec_factor<SPEC>(nd, spec, live);
        }
        const float T = fminf(fmaxf(P.tp + A.phi, 0.0f), 1.0f);
        cr = P.b * spec * (T * (P.sq != 0.0f ? T : 1.0f)) * (y * y);
        ci = 0.0f;
    } else if constexpr (KIND == 0) {
        // bistatic (sample weight only): b spec T_tx T_rx / (r_t r_r)
        const PtRec& P = rec;
        const double dx = P.x - A.x, dy = P.y - A.y, dz = P.z - A.z;
        const double ex = P.x - Rx.x, ey = P.y - Rx.y, ez = P.z - Rx.z;
        float yt, yr;
        r = 0.5 * (range_f64(dx, dy, dz, yt) + range_f64(ex, ey, ez, yr));
        float spec, live;
        if constexpr (SPEC == (int)RFVR_SPEC_OFF) {
            spec = 1.0f;
        } else {
            const float fdx = (float)dx, fdy = (float)dy, fdz = (float)dz;
            const float fex = (float)ex, fey = (float)ey, fez = (float)ez;
            const float ni = (P.nx * fdx + P.ny * fdy + P.nz * fdz) * yt;
            const float nr = -(P.nx * fex + P.ny * fey + P.nz * fez) * yr;
            const float ir = -(fdx * fex + fdy * fey + fdz * fez) * (yt * yr);
            spec_factor_bi<SPEC>(ni, nr, ir, spec, live);
        }
        const float Tt = fminf(fmaxf(P.tp + A.phi, 0.0f), 1.0f);
        const float Tr = fminf(fmaxf(P.tp + Rx.phi, 0.0f), 1.0f);
        cr = P.b * spec * (Tt * Tr) * (yt * yr);
        ci = 0.0f;
    } else {
        const QRec& Q = rec;
        float y;
        r = range_f64(Q.x - A.x, Q.y - A.y, Q.z - A.z, y);
        if constexpr (BI) {
            float yr;
            r = 0.5 * (r + range_f64(Q.x - Rx.x, Q.y - Rx.y, Q.z - Rx.z, yr));
        }
        cr = Q.hr;
        ci = Q.hi;
    }
}

// adds the moments of points j0 <= j < j1 about (rc, h) to m.
// Every lane of the work-group takes the same point at the same time: its
// record is a wave-uniform (scalar) load.  The next record is requested once the
// current one has been read (scalar loads complete out of order, so any wait is
// for all of them) and lands during the moment updates.
template <int K, int KIND, int SPEC, bool BI, class Rec>
__device__ __forceinline__ void cheb_moments(const AntRec& A, const AntRec& Rx, double rc, double inv_h, double Kc,
                                             const Rec* __restrict__ recs, long j0, long j1, float (&mr)[K], float (&mi)[K]) {
    Rec cur = recs[j0 < j1 ? j0 : 0];
    for (long j = j0; j < j1; ++j) {
        double r;
        float cr, ci;
        pair_weight<KIND, SPEC, BI>(cur, A, Rx, r, cr, ci);
        // weight times exp(-j 2 pi Kc r)
        const float t0 = frac_rev(r * Kc);
        const float c0 = cos_rev(t0), s0 = sin_rev(t0);
        const float br = __builtin_fmaf(cr, c0, ci * s0);
        const float bi = __builtin_fmaf(ci, c0, -cr * s0);
        const float x = (float)((r - rc) * inv_h);
        const Rec nxt = recs[j + 1 < j1 ? j + 1 : j];
        __builtin_amdgcn_sched_barrier(0);
        const float x2 = x + x;
        mr[0] += br;
        mi[0] += bi;
        float tm = 1.0f, tk = x;
        mr[1] = __builtin_fmaf(br, x, mr[1]);
        mi[1] = __builtin_fmaf(bi, x, mi[1]);
#pragma unroll
        for (int k = 2; k < K; ++k) {
            const float tn = __builtin_fmaf(x2, tk, -tm);
            tm = tk;
            tk = tn;
            mr[k] = __builtin_fmaf(br, tn, mr[k]);
            mi[k] = __builtin_fmaf(bi, tn, mi[k]);
        }
        cur = nxt;
    }
}

template <int K, int KIND, int SPEC, bool BI>
__device__ __forceinline__ void cheb_points_body(
    int n_meas, const AntRec* __restrict__ ant, const AntRec* __restrict__ rxa, const MeasCheb* __restrict__ meas,
    double Kc, const void* __restrict__ recs_v, long n_pts,
    long pts_per_split, int n_split, int gx, float2* __restrict__ partial) {
    using Rec = typename std::conditional<KIND == 0, PtRec, QRec>::type;
    const long bid = blockIdx.x;
    const int lb = (int)((bid / 8) % gx);
    const long split = (bid / (8L * gx)) * 8 + (bid % 8);
    if (split >= n_split) return;
    const int i = lb * blockDim.x + threadIdx.x;
    const bool live_lane = i < n_meas;
    const int ic = live_lane ? i : n_meas - 1;
    const AntRec A = ant[ic];
    AntRec Rx = A;
    if constexpr (BI) Rx = rxa[ic];
    const MeasCheb mc = meas[ic];
    float mr[K], mi[K];
#pragma unroll
    for (int k = 0; k < K; ++k) mr[k] = mi[k] = 0.0f;
    const long j0 = split * pts_per_split;
    long j1 = j0 + pts_per_split;
    if (j1 > n_pts) j1 = n_pts;
    cheb_moments<K, KIND, SPEC, BI>(A, Rx, mc.rc, mc.inv_h, Kc, reinterpret_cast<const Rec*>(recs_v), j0, j1, mr, mi);
    if (live_lane) {
        float2* out = partial + ((size_t)split * n_meas + i) * kChebKMax;
#pragma unroll
        for (int k = 0; k < K; ++k) out[k] = make_float2(mr[k], mi[k]);
    }
}

// One launch per order (ORDER), all but the plan's returning at once; or one
// launch for all orders (ORDER 0), in which the larger ones' registers and code
// lie beside the one that runs: see one_launch().
#define RFVR_CP_PARAMS                                                                                               \
    int n_meas, const AntRec* __restrict__ ant, const AntRec* __restrict__ rxa, const MeasCheb* __restrict__ meas,   \
        double Kc, const void* __restrict__ recs_v, long n_pts, long pts_per_split, int n_split, int gx,             \
        float2* __restrict__ partial
#define RFVR_CP_ARGS n_meas, ant, rxa, meas, Kc, recs_v, n_pts, pts_per_split, n_split, gx, partial
// body<K>(args) for the plan's order K, of those that the launch serves
#define RFVR_BY_ORDER(ORDER, CALL)                              \
    const int order = plan->KC ? 0 : plan->K;                   \
    if constexpr (ORDER != 0) {                                 \
        if (order == ORDER) CALL(ORDER);                        \
    } else {                                                    \
        switch (order) {                                        \
            case 24: return CALL(24);                           \
            case 28: return CALL(28);                           \
            case 32: return CALL(32);                           \
            case 40: return CALL(40);                           \
            case 48: return CALL(48);                           \
            case 64: return CALL(64);                           \
            default: return;                                    \
        }                                                       \
    }

template <int ORDER, int KIND, int SPEC, bool BI>
__global__ __launch_bounds__(256) void k_cheb_points(const ChebPlan* __restrict__ plan, RFVR_CP_PARAMS) {
#define RFVR_CALL(K) cheb_points_body<K, KIND, SPEC, BI>(RFVR_CP_ARGS)
    RFVR_BY_ORDER(ORDER, RFVR_CALL)
#undef RFVR_CALL
}

// ---------------------------------------------------------------------------
// Between moments or coefficients and frequencies.  With f(x) = sum_n g_n
// exp(+j 2 pi dn Kd (rc + h x)) the series coefficients are those of f's Chebyshev
// interpolation at N nodes x_l = cos((2l+1) pi / 2N),
//   B_k = (2 - [k=0]) / N sum_l f(x_l) T_k(x_l),
// and the way from moments to frequencies is the transpose.  N = K + 8: what
// interpolation adds to the cut series are its terms from order 2N - K on, below
// 1e-12 wherever the cut at K meets its tolerance.  Everything in FP64, one
// work-group per measurement; the phasors of a node at n = 16 a + b are products
// of two tables in LDS, 32 sines and cosines per node and 256 frequencies, where
// Bessel functions by backward recurrence took 160 dependent FP64 steps per
// frequency (coefficients of 1024 measurements x 128 frequencies: 67 -> 13 us, of
// 64 x 32: 36 -> 6; sum of the splits and outputs of 64 x 32: 38 -> 10).
// ---------------------------------------------------------------------------
constexpr int kNodeMax = kChebKMax + 8, kTabLd = 17;
struct NodeTables {
    double2 A[kNodeMax * kTabLd];    // [node][a]: exp(j 2 pi (n0 + 16 a - nc) Kd r)
    double2 B[kNodeMax * kTabLd];    // [node][b]: exp(j 2 pi b Kd r)
    double r[kNodeMax];              // range of the node
};

__device__ __forceinline__ double2 turn(double rev, double sign) {
    double s, c;
    sincospi(2.0 * (rev - floor(rev)), &s, &c);
    return make_double2(c, sign * s);
}
__device__ __forceinline__ double2 cmul(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }

// nodes and the b table (call once), and the a table of frequencies n0 .. n0 + 255
__device__ __forceinline__ void node_begin(NodeTables& t, int N, const MeasCheb& mc, double Kd, double sign) {
    for (int l = threadIdx.x; l < N; l += 256) t.r[l] = mc.rc + mc.h * cospi((double)(2 * l + 1) / (double)(2 * N));
    __syncthreads();
    for (int e = threadIdx.x; e < 16 * N; e += 256) t.B[(e >> 4) * kTabLd + (e & 15)] = turn((double)(e & 15) * Kd * t.r[e >> 4], sign);
}
__device__ __forceinline__ void node_block(NodeTables& t, int N, int n0, double nc, double Kd, double sign) {
    for (int e = threadIdx.x; e < 16 * N; e += 256)
        t.A[(e >> 4) * kTabLd + (e & 15)] = turn(((double)(n0 + 16 * (e & 15)) - nc) * Kd * t.r[e >> 4], sign);
}

// moments M[i][k] = sum over the splits (FP64, fixed order: 8 thread groups take
// every 8th split, their sums are added in order), then
// out[i][n] (+)= sum_l u_l exp(-j 2 pi dn Kd r_l), u_l = sum_k (2 - [k=0]) / N T_k(x_l) M_k
__global__ __launch_bounds__(256) void k_cheb_out(const ChebPlan* __restrict__ plan, const MeasCheb* __restrict__ meas,
                                                  const float2* __restrict__ partial, int n_split, int n_meas, int n_freq,
                                                  double Kd, int accumulate, float2* __restrict__ out,
                                                  const CellIndex* __restrict__ cells) {
    __shared__ NodeTables t;
    __shared__ double2 grp[8][32];
    __shared__ double2 M[kChebKMax], u[kNodeMax];
    const int K = plan->K;
    if (K == 0) return;
    if (plan->KC) n_split = cells->unit[cells->n_cells];
    const int i = blockIdx.x, N = K + 8, tid = threadIdx.x;
    for (int k0 = 0; k0 < K; k0 += 32) {
        const int k = k0 + (tid & 31), gi = tid >> 5;
        double ar = 0.0, ai = 0.0;
        if (k < K) {
#pragma unroll 8
            for (int s = gi; s < n_split; s += 8) {
                const float2 v = partial[((size_t)s * n_meas + i) * kChebKMax + k];
                ar += v.x;
                ai += v.y;
            }
        }
        grp[gi][tid & 31] = make_double2(ar, ai);
        __syncthreads();
        if (gi == 0 && k < K) {
            double2 m = grp[0][tid];
            for (int g = 1; g < 8; ++g) {
                m.x += grp[g][tid].x;
                m.y += grp[g][tid].y;
            }
            M[k] = m;
        }
        __syncthreads();
    }
    const MeasCheb mc = meas[i];
    node_begin(t, N, mc, Kd, -1.0);
    if (tid < N) {
        const double x = cospi((double)(2 * tid + 1) / (double)(2 * N));
        double tm = 1.0, tk = x, ur = 0.5 * M[0].x + x * M[1].x, ui = 0.5 * M[0].y + x * M[1].y;
        for (int k = 2; k < K; ++k) {
            const double tn = 2.0 * x * tk - tm;
            tm = tk;
            tk = tn;
            ur += tn * M[k].x;
            ui += tn * M[k].y;
        }
        u[tid] = make_double2(2.0 / N * ur, 2.0 / N * ui);
    }
    const double nc = 0.5 * (double)(n_freq - 1);
    for (int n0 = 0; n0 < n_freq; n0 += 256) {
        node_block(t, N, n0, nc, Kd, -1.0);
        __syncthreads();
        for (int e = tid; e < 16 * N; e += 256) {
            double2& a = t.A[(e >> 4) * kTabLd + (e & 15)];
            a = cmul(a, u[e >> 4]);
        }
        __syncthreads();
        const int n = n0 + tid;
        if (n < n_freq) {
            double re = 0.0, im = 0.0;
            for (int l = 0; l < N; ++l) {
                const double2 v = cmul(t.A[l * kTabLd + (tid >> 4)], t.B[l * kTabLd + (tid & 15)]);
                re += v.x;
                im += v.y;
            }
            float2* o = out + (size_t)i * n_freq + n;
            float2 v = make_float2((float)re, (float)im);
            if (accumulate) {
                v.x += o->x;
                v.y += o->y;
            }
            *o = v;
        }
        __syncthreads();
    }
}

// B[i][k], k < K, from g[i][n]
__global__ __launch_bounds__(256) void k_cheb_coef(const ChebPlan* __restrict__ plan,
                                                   const MeasCheb* __restrict__ meas,
                                                   const float2* __restrict__ g, int n_meas, int n_freq,
                                                   double Kd, float2* __restrict__ B) {
    __shared__ NodeTables t;
    __shared__ double2 f[kNodeMax];
    __shared__ float2 gs[256];
    const int K = plan->K;
    if (K == 0) return;
    const int i = blockIdx.x, N = K + 8, tid = threadIdx.x;
    const MeasCheb mc = meas[i];
    const double nc = 0.5 * (double)(n_freq - 1);
    if (tid < N) f[tid] = make_double2(0.0, 0.0);
    node_begin(t, N, mc, Kd, 1.0);
    for (int n0 = 0; n0 < n_freq; n0 += 256) {
        gs[tid] = n0 + tid < n_freq ? g[(size_t)i * n_freq + n0 + tid] : make_float2(0.0f, 0.0f);
        node_block(t, N, n0, nc, Kd, 1.0);
        __syncthreads();
        // (node, a): sum over b, times the a phasor
        for (int e = tid; e < 16 * N; e += 256) {
            const int l = e >> 4, a = e & 15;
            double sr = 0.0, si = 0.0;
#pragma unroll 4
            for (int b = 0; b < 16; ++b) {
                const double2 w = t.B[l * kTabLd + b];
                const float2 v = gs[16 * a + b];
                sr += w.x * v.x - w.y * v.y;
                si += w.x * v.y + w.y * v.x;
            }
            double2& o = t.A[l * kTabLd + a];
            o = cmul(o, make_double2(sr, si));
        }
        __syncthreads();
        if (tid < N) {
            double2 v = f[tid];
            for (int a = 0; a < 16; ++a) {
                v.x += t.A[tid * kTabLd + a].x;
                v.y += t.A[tid * kTabLd + a].y;
            }
            f[tid] = v;
        }
        __syncthreads();
    }
    if (tid < K) {
        // cos(k (2l+1) pi / 2N) for l = 0, 1, ... by its recurrence in l
        const double w = (double)tid / (double)(2 * N);
        double cm = cospi(w), c0 = cm;                   // l = -1 and l = 0 (even in 2l+1)
        const double c2 = 2.0 * cospi(2.0 * w);
        double br = 0.0, bi = 0.0;
        for (int l = 0; l < N; ++l) {
            br += c0 * f[l].x;
            bi += c0 * f[l].y;
            const double cn = c2 * c0 - cm;
            cm = c0;
            c0 = cn;
        }
        const double e = (tid == 0 ? 1.0 : 2.0) / N;
        B[(size_t)i * kChebKMax + tid] = make_float2((float)(e * br), (float)(e * bi));
    }
}

// sum_k B_k T_k(x) (complex coefficients, real x) with T_k from their
// three-term recurrence: 3 operations per order (Clenshaw's backward form
// takes 4), the coefficients being wave-uniform scalar operands
template <int K>
__device__ __forceinline__ void cheb_series(const float2* __restrict__ Bi, float x, float& sr, float& si) {
    const float x2 = x + x;
    float2 c = Bi[0];
    sr = c.x;
    si = c.y;
    c = Bi[1];
    sr = __builtin_fmaf(c.x, x, sr);
    si = __builtin_fmaf(c.y, x, si);
    float tm = 1.0f, tk = x;
#pragma unroll
    for (int k = 2; k < K; ++k) {
        const float tn = __builtin_fmaf(x2, tk, -tm);
        tm = tk;
        tk = tn;
        c = Bi[k];
        sr = __builtin_fmaf(c.x, tn, sr);
        si = __builtin_fmaf(c.y, tn, si);
    }
}

// two series with the same argument, sharing the recurrence
template <int K>
__device__ __forceinline__ void cheb_series2(const float2* __restrict__ Bi, const float2* __restrict__ Ci, float x,
                                             float& sr, float& si, float& s2r, float& s2i) {
    const float x2 = x + x;
    float2 c = Bi[0], d = Ci[0];
    sr = c.x;
    si = c.y;
    s2r = d.x;
    s2i = d.y;
    c = Bi[1];
    d = Ci[1];
    sr = __builtin_fmaf(c.x, x, sr);
    si = __builtin_fmaf(c.y, x, si);
    s2r = __builtin_fmaf(d.x, x, s2r);
    s2i = __builtin_fmaf(d.y, x, s2i);
    float tm = 1.0f, tk = x;
#pragma unroll
    for (int k = 2; k < K; ++k) {
        const float tn = __builtin_fmaf(x2, tk, -tm);
        tm = tk;
        tk = tn;
        c = Bi[k];
        d = Ci[k];
        sr = __builtin_fmaf(c.x, tn, sr);
        si = __builtin_fmaf(c.y, tn, si);
        s2r = __builtin_fmaf(d.x, tn, s2r);
        s2i = __builtin_fmaf(d.y, tn, s2i);
    }
}

// ---------------------------------------------------------------------------
// matched filter forward: lane = query point, loop over measurements
// (records, plan and coefficients are wave-uniform loads)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void mf_store(float2* z, float* power, long q, float zr, float zi) {
    if (z) z[q] = make_float2(zr, zi);
    if (power) power[q] = sqrtf(zr * zr + zi * zi);
}

// Per split of the measurements (blockIdx.y) `per` of them.  part: of several
// splits the sums [split][1 or 2][n_q], else NULL.  (The arrays the loop reads
// are kernel arguments of their own, marked as not aliased: only then are the
// wave-uniform reads scalar loads.)
#define RFVR_MF_PARAMS                                                                                              \
    long n_q, const float* __restrict__ xq, int n_meas, int per, const AntRec* __restrict__ ant,                    \
        const AntRec* __restrict__ rxa, const MeasCheb* __restrict__ meas, const float2* __restrict__ B,            \
        const float2* __restrict__ B2, double Kc, float2* __restrict__ z, float* __restrict__ power,                \
        float2* __restrict__ z2, float* __restrict__ power2, float2* __restrict__ part
#define RFVR_MF_ARGS n_q, xq, n_meas, per, ant, rxa, meas, B, B2, Kc, z, power, z2, power2, part

template <int K, bool TWO, bool BI>
__device__ __forceinline__ void cheb_mf_body(RFVR_MF_PARAMS) {
    const int i0 = blockIdx.y * per, i1 = min(i0 + per, n_meas);
    const long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const long qc = q < n_q ? q : n_q - 1;
    const double px = (double)xq[3 * qc], py = (double)xq[3 * qc + 1], pz = (double)xq[3 * qc + 2];
    float zr = 0.0f, zi = 0.0f, z2r = 0.0f, z2i = 0.0f;
    for (int i = i0; i < i1; ++i) {
        const AntRec A = ant[i];
        const MeasCheb mc = meas[i];
        float y;
        double r = range_f64(px - A.x, py - A.y, pz - A.z, y);
        if constexpr (BI) {
            const AntRec Rx = rxa[i];
            float yr;
            r = 0.5 * (r + range_f64(px - Rx.x, py - Rx.y, pz - Rx.z, yr));
        }
        const float x = (float)((r - mc.rc) * mc.inv_h);
        const float t0 = frac_rev(r * Kc);
        const float c0 = cos_rev(t0), s0 = sin_rev(t0);       // exp(+j 2 pi Kc r)
        float sr, si;
        if constexpr (TWO) {
            float s2r, s2i;
            cheb_series2<K>(B + (size_t)i * kChebKMax, B2 + (size_t)i * kChebKMax, x, sr, si, s2r, s2i);
            z2r = __builtin_fmaf(c0, s2r, __builtin_fmaf(-s0, s2i, z2r));
            z2i = __builtin_fmaf(c0, s2i, __builtin_fmaf(s0, s2r, z2i));
        } else {
            cheb_series<K>(B + (size_t)i * kChebKMax, x, sr, si);
        }
        zr = __builtin_fmaf(c0, sr, __builtin_fmaf(-s0, si, zr));
        zi = __builtin_fmaf(c0, si, __builtin_fmaf(s0, sr, zi));
    }
    if (q >= n_q) return;
    if (part) {
        float2* p = part + (size_t)blockIdx.y * (TWO ? 2 : 1) * n_q + q;
        p[0] = make_float2(zr, zi);
        if constexpr (TWO) p[n_q] = make_float2(z2r, z2i);
        return;
    }
    mf_store(z, power, q, zr, zi);
    if constexpr (TWO) mf_store(z2, power2, q, z2r, z2i);
}

template <int ORDER, bool TWO, bool BI>
__global__ __launch_bounds__(256) void k_cheb_mf(const ChebPlan* __restrict__ plan, RFVR_MF_PARAMS) {
#define RFVR_CALL(K) cheb_mf_body<K, TWO, BI>(RFVR_MF_ARGS)
    RFVR_BY_ORDER(ORDER, RFVR_CALL)
#undef RFVR_CALL
}

// fixed-order sum over the measurement splits
__global__ __launch_bounds__(256) void k_cheb_mf_sum(const ChebPlan* __restrict__ plan, long n_q,
                                                     const float2* __restrict__ part, int n_split, int two,
                                                     float2* z, float* power, float2* z2, float* power2) {
    if (plan->K == 0 || plan->KC) return;
    const long q = (long)blockIdx.x * 256 + threadIdx.x;
    if (q >= n_q) return;
    for (int w = 0; w <= two; ++w) {
        float zr = 0.0f, zi = 0.0f;
        for (int s = 0; s < n_split; ++s) {
            const float2 v = part[((size_t)s * (two + 1) + w) * n_q + q];
            zr += v.x;
            zi += v.y;
        }
        mf_store(w ? z2 : z, w ? power2 : power, q, zr, zi);
    }
}

// ---------------------------------------------------------------------------
// signal tracing adjoint: lane = point, loop over measurements; the pair's
// G = Re(sum_n g[i][n] exp(+j 2 pi (K0 + n Kd) r)) then the chain rule of the
// per-frequency kernel
// ---------------------------------------------------------------------------
// a pair's share of its point's gradient sums, from its series value (sr, si)
template <int SPEC, bool BI>
__device__ __forceinline__ void bwd_pair(const PtRec& P, const AntRec& A, const AntRec& Rx, double dx, double dy, double dz,
                                         double ex, double ey, double ez, double r, float y, float yr, double Kc, float sr,
                                         float si, float& gb, float& gt, float& gn0, float& gn1, float& gn2) {
    const float t0 = frac_rev(r * Kc);
    const float c0 = cos_rev(t0), s0 = sin_rev(t0);
    const float G = c0 * sr - s0 * si;                     // Re(exp(+j 2 pi Kc r) S)
    if constexpr (BI) {
        // c = b spec T_tx T_rx y_t y_r (sample weight): dc/db, dc/dT
        // (times b after the loop) and dc/dn_hat (times -2 b after the loop)
        const float fdx = (float)dx, fdy = (float)dy, fdz = (float)dz;
        const float fex = (float)ex, fey = (float)ey, fez = (float)ez;
        float spec, live = 0.0f, ni = 0.0f, nr = 0.0f;
        if constexpr (SPEC == (int)RFVR_SPEC_OFF) {
            spec = 1.0f;
        } else {
            ni = (P.nx * fdx + P.ny * fdy + P.nz * fdz) * y;
            nr = -(P.nx * fex + P.ny * fey + P.nz * fez) * yr;
            const float ir = -(fdx * fex + fdy * fey + fdz * fez) * (y * yr);
            spec_factor_bi<SPEC>(ni, nr, ir, spec, live);
        }
        const float Ut = P.tp + A.phi, Ur = P.tp + Rx.phi;
        const float Tt = fminf(fmaxf(Ut, 0.0f), 1.0f), Tr = fminf(fmaxf(Ur, 0.0f), 1.0f);
        const float dT = (Tt == Ut ? Tr : 0.0f) + (Tr == Ur ? Tt : 0.0f);
        const float gy = G * (y * yr);
        const float gs = gy * spec, T2 = Tt * Tr;
        gb = __builtin_fmaf(gs, T2, gb);
        gt = __builtin_fmaf(gs, dT, gt);
        if constexpr (SPEC != (int)RFVR_SPEC_OFF) {
            // nr w_i + ni w_r with w_i = d_t y_t, w_r = -d_r y_r
            const float ct = gy * T2 * live * (nr * y), cq = -gy * T2 * live * (ni * yr);
            gn0 = __builtin_fmaf(ct, fdx, __builtin_fmaf(cq, fex, gn0));
            gn1 = __builtin_fmaf(ct, fdy, __builtin_fmaf(cq, fey, gn1));
            gn2 = __builtin_fmaf(ct, fdz, __builtin_fmaf(cq, fez, gn2));
        }
        return;
    }
    const float fdx = (float)dx, fdy = (float)dy, fdz = (float)dz;
    float spec, live = 0.0f, nd = 0.0f;
    if constexpr (SPEC == (int)RFVR_SPEC_OFF) {
        spec = 1.0f;
    } else {
        nd = (P.nx * fdx + P.ny * fdy + P.nz * fdz) * y;
        spec_factor<SPEC>(nd, spec, live);
    }
    const float Tr = P.tp + A.phi;
    const float T = fminf(fmaxf(Tr, 0.0f), 1.0f);
    // transmittance factor T^2 (sample weight) or T (segment weight) and
    // its derivative where the clamp is inactive
    const float dT = T == Tr ? (P.sq != 0.0f ? T + T : 1.0f) : 0.0f;
    const float gy = G * (y * y);
    const float gs = gy * spec, T2 = T * (P.sq != 0.0f ? T : 1.0f);
    gb = __builtin_fmaf(gs, T2, gb);
    gt = __builtin_fmaf(gs, dT, gt);                       // times b after the loop
    if constexpr (SPEC != (int)RFVR_SPEC_OFF) {
        const float cn = gy * T2 * (nd * y) * live;        // times 4 b after the loop
        gn0 = __builtin_fmaf(cn, fdx, gn0);
        gn1 = __builtin_fmaf(cn, fdy, gn1);
        gn2 = __builtin_fmaf(cn, fdz, gn2);
    }
}

// part: of several measurement splits the sums [split][5][n_pts], else NULL
#define RFVR_BWD_PARAMS                                                                                       \
    long n_pts, const PtRec* __restrict__ rec, int n_meas, int per, const AntRec* __restrict__ ant,           \
        const AntRec* __restrict__ rxa, const MeasCheb* __restrict__ meas, const float2* __restrict__ B,      \
        double Kc, float* __restrict__ g_b, float* __restrict__ g_T, float* __restrict__ g_n, float* __restrict__ part
#define RFVR_BWD_ARGS n_pts, rec, n_meas, per, ant, rxa, meas, B, Kc, g_b, g_T, g_n, part

// a point's sums over its pairs, times the factors common to them
template <bool BI>
__device__ __forceinline__ void bwd_store(float* g_b, float* g_T, float* g_n, long j, float b, float gb, float gt,
                                          float gn0, float gn1, float gn2) {
    g_b[j] = gb;
    g_T[j] = b * gt;
    const float b4 = (BI ? -2.0f : 4.0f) * b;
    g_n[3 * j] = b4 * gn0;
    g_n[3 * j + 1] = b4 * gn1;
    g_n[3 * j + 2] = b4 * gn2;
}

template <int K, int SPEC, bool BI>
__device__ __forceinline__ void cheb_bwd_body(RFVR_BWD_PARAMS) {
    const int i0 = blockIdx.y * per, i1 = min(i0 + per, n_meas);
    const long j = (long)blockIdx.x * blockDim.x + threadIdx.x;
    const PtRec P = rec[j < n_pts ? j : n_pts - 1];
    float gb = 0.0f, gt = 0.0f, gn0 = 0.0f, gn1 = 0.0f, gn2 = 0.0f;
    for (int i = i0; i < i1; ++i) {
        const AntRec A = ant[i];
        const MeasCheb mc = meas[i];
        const double dx = P.x - A.x, dy = P.y - A.y, dz = P.z - A.z;
        float y;
        double r = range_f64(dx, dy, dz, y);
        AntRec Rx = A;
        double ex = 0.0, ey = 0.0, ez = 0.0;
        float yr = 0.0f;
        if constexpr (BI) {
            Rx = rxa[i];
            ex = P.x - Rx.x; ey = P.y - Rx.y; ez = P.z - Rx.z;
            r = 0.5 * (r + range_f64(ex, ey, ez, yr));
        }
        const float x = (float)((r - mc.rc) * mc.inv_h);
        float sr, si;
        cheb_series<K>(B + (size_t)i * kChebKMax, x, sr, si);
        bwd_pair<SPEC, BI>(P, A, Rx, dx, dy, dz, ex, ey, ez, r, y, yr, Kc, sr, si, gb, gt, gn0, gn1, gn2);
    }
    if (j >= n_pts) return;
    if (part) {
        float* p = part + (size_t)blockIdx.y * 5 * n_pts + j;
        p[0] = gb;
        p[n_pts] = gt;
        p[2 * n_pts] = gn0;
        p[3 * n_pts] = gn1;
        p[4 * n_pts] = gn2;
        return;
    }
    bwd_store<BI>(g_b, g_T, g_n, j, P.b, gb, gt, gn0, gn1, gn2);
}

template <int ORDER, int SPEC, bool BI>
__global__ __launch_bounds__(256) void k_cheb_render_bwd(const ChebPlan* __restrict__ plan, RFVR_BWD_PARAMS) {
#define RFVR_CALL(K) cheb_bwd_body<K, SPEC, BI>(RFVR_BWD_ARGS)
    RFVR_BY_ORDER(ORDER, RFVR_CALL)
#undef RFVR_CALL
}

// fixed-order sum over the measurement splits
template <bool BI>
__global__ __launch_bounds__(256) void k_cheb_bwd_sum(const ChebPlan* __restrict__ plan, long n_pts,
                                                      const PtRec* __restrict__ rec, const float* __restrict__ part,
                                                      int n_split, float* g_b, float* g_T, float* g_n) {
    if (plan->K == 0 || plan->KC) return;
    const long j = (long)blockIdx.x * 256 + threadIdx.x;
    if (j >= n_pts) return;
    float v[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    for (int s = 0; s < n_split; ++s)
#pragma unroll
        for (int c = 0; c < 5; ++c) v[c] += part[((size_t)s * 5 + c) * n_pts + j];
    bwd_store<BI>(g_b, g_T, g_n, j, rec[j].b, v[0], v[1], v[2], v[3], v[4]);
}

// ---------------------------------------------------------------------------
// Cells.  The orders that a series needs grow with the width of its range
// interval, so a large launch sorts its points into the cells of a grid over
// their box and evaluates per pair only the few orders of the cell's own
// interval (10 for 2.5 cm cells in place of 24 for the 20 cm cube).  The way between
// the cell's series and the launch's (order K, over the whole box) is
// interpolation at the cell's KC Chebyshev nodes x_l, done once per (cell,
// measurement) and work-group:
//   down  f_l = sum_k B_k T_k(X_l), X_l the node in the box's interval,
//         b_m = (2 - [m=0]) / KC sum_l f_l T_m(x_l)
//   up    u_l = sum_m (2 - [m=0]) / KC T_m(x_l) m_m, M_k = sum_l u_l T_k(X_l)
// i.e. some thousand operations against 512 or more points of 3 (24 - KC) each.
// Bound: vector issue, 47 (filter) to 77 (render adjoint) instructions per pair
// counted, in place of 96 to 126.  2^20 points in a 20 cm cube, 1024 measurements, 64 frequencies:
// render 2.73 -> 1.84 ms, its adjoint 3.11 -> 1.90, filter 2.43 -> 1.38, its adjoint
// 2.45 -> 1.47 (with the polynomials' recurrence instead of powers of x below: 2.27
// and 1.79 for the two over frequencies).
// The sort is a stable counting sort (fixed order, no floating point atomics):
// k_cell_hist counts each wave's share of the points per cell, k_cell_scan turns
// the counts of a cell into offsets, k_cell_scatter writes the order.
// ---------------------------------------------------------------------------
// position of a point of either kind
struct PosXyz {
    const float* p;
    __device__ __forceinline__ void at(long j, float (&x)[3]) const {
        x[0] = p[3 * j];
        x[1] = p[3 * j + 1];
        x[2] = p[3 * j + 2];
    }
};
struct PosQ {
    const QRec* p;
    __device__ __forceinline__ void at(long j, float (&x)[3]) const {
        x[0] = (float)p[j].x;
        x[1] = (float)p[j].y;
        x[2] = (float)p[j].z;
    }
};
struct PosRec {
    const PtRec* p;
    __device__ __forceinline__ void at(long j, float (&x)[3]) const {
        x[0] = (float)p[j].x;
        x[1] = (float)p[j].y;
        x[2] = (float)p[j].z;
    }
};
__device__ __forceinline__ int cell_of(const CellGrid& g, const float (&x)[3]) {
    int c[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        // a NaN coordinate goes to cell 0 of its axis
        c[d] = (int)fminf(fmaxf((x[d] - (float)g.lo[d]) * g.inv_w[d], 0.0f), (float)(g.n[d] - 1));
    }
    return (c[2] * g.n[1] + c[1]) * g.n[0] + c[0];
}

// hist[cell][wave], a wave taking `per` consecutive points
template <class Pos>
__global__ __launch_bounds__(256) void k_cell_hist(const ChebPlan* __restrict__ plan, const CellGrid* __restrict__ grid, Pos pos,
                                                   long n, int per, int n_wave, int* __restrict__ hist) {
    __shared__ int sh[4][kMaxCells];
    if (plan->KC == 0) return;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, w = blockIdx.x * 4 + wv;
    const CellGrid g = *grid;
    for (int c = lane; c < g.n_cells; c += 64) sh[wv][c] = 0;
    __syncthreads();
    const long j0 = (long)w * per, j1 = min(j0 + per, n);
    for (long j = j0 + lane; j < j1; j += 64) {
        float x[3];
        pos.at(j, x);
        atomicAdd(&sh[wv][cell_of(g, x)], 1);
    }
    __syncthreads();
    if (w >= n_wave) return;
    for (int c = lane; c < g.n_cells; c += 64) hist[(size_t)c * n_wave + w] = sh[wv][c];
}

// exclusive scan of a cell's counts over the waves, in place; its total
__global__ __launch_bounds__(256) void k_cell_scan(const ChebPlan* __restrict__ plan, const CellGrid* __restrict__ grid, int n_wave,
                                                   int* __restrict__ hist, CellIndex* __restrict__ cells) {
    __shared__ int sh[4];
    if (plan->KC == 0 || (int)blockIdx.x >= grid->n_cells) return;
    int* h = hist + (size_t)blockIdx.x * n_wave;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int base = 0;
    for (int w0 = 0; w0 < n_wave; w0 += 256) {
        const int w = w0 + threadIdx.x;
        const int v = w < n_wave ? h[w] : 0;
        int s = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(s, d, 64);
            if (lane >= d) s += t;
        }
        if (lane == 63) sh[wv] = s;
        __syncthreads();
        int before = base;
        for (int q = 0; q < wv; ++q) before += sh[q];
        if (w < n_wave) h[w] = before + s - v;
        for (int q = 0; q < 4; ++q) base += sh[q];
        __syncthreads();
    }
    if (threadIdx.x == 0) cells->total[blockIdx.x] = base;
}

// the order: perm[position] = point (and the point's record, Rec, if out is given).
// A work-group's first step is the prefix sum of the totals; work-group 0 writes
// the index that the consumers read, with cells cut into units of at most `unit` points.
template <class Pos, class Rec>
__global__ __launch_bounds__(256) void k_cell_scatter(const ChebPlan* __restrict__ plan, const CellGrid* __restrict__ grid, Pos pos,
                                                      long n, int per, int n_wave, int unit, const int* __restrict__ hist,
                                                      CellIndex* __restrict__ cells, int* __restrict__ perm,
                                                      const Rec* __restrict__ rec, Rec* __restrict__ out) {
    __shared__ int start[kMaxCells + 1];
    __shared__ int next[4][kMaxCells];
    if (plan->KC == 0) return;
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, w = blockIdx.x * 4 + wv;
    const CellGrid g = *grid;
    const bool first = blockIdx.x == 0;
    if (wv == 0) {
        int base = 0, ubase = 0;
        for (int c0 = 0; c0 < g.n_cells; c0 += 64) {
            const int c = c0 + lane, v = c < g.n_cells ? cells->total[c] : 0, uv = (v + unit - 1) / unit;
            int s = v, us = uv;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int t = __shfl_up(s, d, 64), ut = __shfl_up(us, d, 64);
                if (lane >= d) {
                    s += t;
                    us += ut;
                }
            }
            if (c < g.n_cells) {
                start[c] = base + s - v;
                if (first) {
                    cells->start[c] = base + s - v;
                    cells->unit[c] = ubase + us - uv;
                }
            }
            base += __shfl(s, 63, 64);
            ubase += __shfl(us, 63, 64);
        }
        if (first && lane == 0) {
            cells->start[g.n_cells] = base;
            cells->unit[g.n_cells] = ubase;
            cells->n_cells = g.n_cells;
        }
    }
    __syncthreads();
    if (w < n_wave)
        for (int c = lane; c < g.n_cells; c += 64) next[wv][c] = start[c] + hist[(size_t)c * n_wave + w];
    __syncthreads();
    const long j0 = (long)w * per, j1 = min(j0 + per, n);
    for (long b = j0; b < j1; b += 64) {
        const long j = b + lane;
        const bool live = j < j1;
        int c = -1;
        if (live) {
            float x[3];
            pos.at(j, x);
            c = cell_of(g, x);
        }
        // lanes of one cell take consecutive positions in lane order
        unsigned long long todo = __ballot(live);
        int at = 0;
        while (todo) {
            const int lead = __ffsll(todo) - 1, cl = __shfl(c, lead, 64);
            const unsigned long long same = __ballot(c == cl);
            const int base = next[wv][cl];
            if (c == cl) at = base + __popcll(same & ((1ull << lane) - 1));
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (lane == lead) next[wv][cl] = base + __popcll(same);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            todo &= ~same;
        }
        if (live) {
            if (perm) perm[at] = (int)j;
            if (out) out[at] = rec[j];
        }
    }
}

// T_m(x_l) at the K nodes
template <int K>
struct NodeCos {
    float c[K][K];
    constexpr NodeCos() : c() {
        for (int l = 0; l < K; ++l)
            for (int m = 0; m < K; ++m) {
                int q = (m * (2 * l + 1)) % (4 * K);             // angle q pi / 2K
                if (q > 2 * K) q = 4 * K - q;
                const bool neg = q > K;
                if (neg) q = 2 * K - q;
                const double v = phase_table::taylor_cos(q * (phase_table::kPi / (2 * K)));
                c[l][m] = (float)(neg ? -v : v);
            }
    }
};
template <int K>
__device__ constexpr NodeCos<K> kNodeCos{};

// Up to kPowerK orders a cell's series is kept in powers of x: Horner's scheme takes
// two operations per order and pair where the polynomials' recurrence takes three.  The powers
// are safe there: the coefficients are those of exp(j z x), at most z^k / k!, and
// z <= 2.8 at 12 orders (largest term 3.9; at 16 orders, z = 5, it would be 26
// and cost that factor in rounding).
constexpr int kPowerK = 12;
struct ChebPowers {
    float c[kPowerK][kPowerK];                   // T_m(x) = sum_k c[m][k] x^k, all exact
    constexpr ChebPowers() : c() {
        c[0][0] = 1.0f;
        c[1][1] = 1.0f;
        for (int m = 2; m < kPowerK; ++m)
            for (int k = 0; k < kPowerK; ++k) c[m][k] = (k ? 2.0f * c[m - 1][k - 1] : 0.0f) - c[m - 2][k];
    }
};
__device__ constexpr ChebPowers kChebPowers{};

// the range interval of measurement (A, Rx) over cell c: centre and half width
template <bool BI>
__device__ __forceinline__ void cell_interval(const CellGrid& g, int c, const AntRec& A, const AntRec& Rx, double& rc, double& h) {
    double lo[3], hi[3];
    int q = c;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int k = q % g.n[d];
        q /= g.n[d];
        // the margin covers the FP32 rounding of cell_of
        const double m = 1e-6 * (g.w[d] * g.n[d]) + 1e-7 * (fabs(g.lo[d]) + g.w[d] * g.n[d]);
        lo[d] = g.lo[d] + g.w[d] * k - m;
        hi[d] = g.lo[d] + g.w[d] * (k + 1) + m;
    }
    auto band = [&](const AntRec& a, double& near_, double& far_) {
        const double p[3] = {a.x, a.y, a.z};
        double n2 = 0.0, f2 = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double qn = fmax(fmax(lo[d] - p[d], p[d] - hi[d]), 0.0);
            const double qf = fmax(fabs(p[d] - lo[d]), fabs(p[d] - hi[d]));
            n2 += qn * qn;
            f2 += qf * qf;
        }
        near_ = sqrt(n2);
        far_ = sqrt(f2);
    };
    double a, b;
    band(A, a, b);
    if constexpr (BI) {
        double a2, b2;
        band(Rx, a2, b2);
        a = 0.5 * (a + a2);
        b = 0.5 * (b + b2);
    }
    rc = 0.5 * (a + b);
    h = 0.5 * (b - a);
}

// the cell's nodes in the box's normalised range, X_l = x_l + d_l: a node's rounding is
// shared by all of the cell's points, so its remainder goes into the recurrences too
template <int K>
__device__ __forceinline__ void node_args(double rc, double h, const MeasCheb& box, float (&x)[K], float (&d)[K]) {
#pragma unroll
    for (int l = 0; l < K; ++l) {
        const double X = (rc + h * (double)kNodeCos<K>.c[l][1] - box.rc) * box.inv_h;
        x[l] = (float)X;
        d[l] = (float)(X - (double)x[l]);
    }
}

// a cell's series coefficients b from the box's, B[0 .. KP)
template <int K>
__device__ __forceinline__ void cell_down(const float2* __restrict__ B, int KP, double rc, double h, const MeasCheb& box,
                                          float2* __restrict__ b) {
    float x[K], d[K], tm[K], tk[K], fr[K], fi[K];
    node_args<K>(rc, h, box, x, d);
    // two orders per step (all KP are even), the next two on the way meanwhile
    const float4* B4 = reinterpret_cast<const float4*>(B);
    float4 v = B4[0], w = B4[1];
#pragma unroll
    for (int l = 0; l < K; ++l) {
        tm[l] = 1.0f;
        tk[l] = x[l];
        fr[l] = __builtin_fmaf(v.z, x[l], v.x);
        fi[l] = __builtin_fmaf(v.w, x[l], v.y);
    }
    for (int k = 2; k < KP; k += 2) {
        v = w;
        w = B4[min(k / 2 + 1, KP / 2 - 1)];
#pragma unroll
        for (int l = 0; l < K; ++l) {
            const float x2 = x[l] + x[l], d2 = d[l] + d[l];
            tm[l] = __builtin_fmaf(x2, tk[l], __builtin_fmaf(d2, tk[l], -tm[l]));
            tk[l] = __builtin_fmaf(x2, tm[l], __builtin_fmaf(d2, tm[l], -tk[l]));
            fr[l] = __builtin_fmaf(v.z, tk[l], __builtin_fmaf(v.x, tm[l], fr[l]));
            fi[l] = __builtin_fmaf(v.w, tk[l], __builtin_fmaf(v.y, tm[l], fi[l]));
        }
    }
    float cr[K], ci[K];
#pragma unroll
    for (int m = 0; m < K; ++m) {
        float sr = 0.0f, si = 0.0f;
#pragma unroll
        for (int l = 0; l < K; ++l) {
            sr = __builtin_fmaf(kNodeCos<K>.c[l][m], fr[l], sr);
            si = __builtin_fmaf(kNodeCos<K>.c[l][m], fi[l], si);
        }
        const float e = (m == 0 ? 1.0f : 2.0f) / K;
        cr[m] = e * sr;
        ci[m] = e * si;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        float pr = cr[k], pi = ci[k];
        if constexpr (K <= kPowerK) {
            pr *= kChebPowers.c[k][k];
            pi *= kChebPowers.c[k][k];
#pragma unroll
            for (int m = k + 2; m < K; m += 2) {
                pr = __builtin_fmaf(kChebPowers.c[m][k], cr[m], pr);
                pi = __builtin_fmaf(kChebPowers.c[m][k], ci[m], pi);
            }
        }
        b[k] = make_float2(pr, pi);
    }
}

// a cell's series at x
template <int K>
__device__ __forceinline__ void cell_series(const float2 (&b)[K], float x, float& sr, float& si) {
    if constexpr (K <= kPowerK) {
        sr = b[K - 1].x;
        si = b[K - 1].y;
#pragma unroll
        for (int k = K - 2; k >= 0; --k) {
            sr = __builtin_fmaf(sr, x, b[k].x);
            si = __builtin_fmaf(si, x, b[k].y);
        }
    } else {
        cheb_series<K>(b, x, sr, si);
    }
}

// the box's moments M[0 .. KP) from a cell's
template <int K>
__device__ __forceinline__ void cell_up(const float (&mr)[K], const float (&mi)[K], int KP, double rc, double h,
                                        const MeasCheb& box, float2* __restrict__ M) {
    float x[K], d[K], tm[K], tk[K], ur[K], ui[K];
    node_args<K>(rc, h, box, x, d);
    float m0r = 0.0f, m0i = 0.0f, m1r = 0.0f, m1i = 0.0f;
#pragma unroll
    for (int l = 0; l < K; ++l) {
        float sr = 0.5f * mr[0], si = 0.5f * mi[0];
#pragma unroll
        for (int m = 1; m < K; ++m) {
            sr = __builtin_fmaf(kNodeCos<K>.c[l][m], mr[m], sr);
            si = __builtin_fmaf(kNodeCos<K>.c[l][m], mi[m], si);
        }
        ur[l] = 2.0f / K * sr;
        ui[l] = 2.0f / K * si;
        tm[l] = 1.0f;
        tk[l] = x[l];
        m0r += ur[l];
        m0i += ui[l];
        m1r = __builtin_fmaf(ur[l], x[l], m1r);
        m1i = __builtin_fmaf(ui[l], x[l], m1i);
    }
    float4* M4 = reinterpret_cast<float4*>(M);
    M4[0] = make_float4(m0r, m0i, m1r, m1i);
    for (int k = 2; k < KP; k += 2) {            // all KP are even
        float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
        for (int l = 0; l < K; ++l) {
            const float x2 = x[l] + x[l], d2 = d[l] + d[l];
            tm[l] = __builtin_fmaf(x2, tk[l], __builtin_fmaf(d2, tk[l], -tm[l]));
            tk[l] = __builtin_fmaf(x2, tm[l], __builtin_fmaf(d2, tm[l], -tk[l]));
            v.x = __builtin_fmaf(ur[l], tm[l], v.x);
            v.y = __builtin_fmaf(ui[l], tm[l], v.y);
            v.z = __builtin_fmaf(ur[l], tk[l], v.z);
            v.w = __builtin_fmaf(ui[l], tk[l], v.w);
        }
        M4[k / 2] = v;
    }
}

// cell of a unit, and the unit's points: positions [first, first + count)
__device__ __forceinline__ bool unit_points(const CellIndex* __restrict__ cells, int u, int& c, int& first, int& count) {
    const int n = cells->n_cells;
    if (u >= cells->unit[n]) return false;
    int lo = 0, hi = n;                          // unit[lo] <= u < unit[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cells->unit[mid] <= u) lo = mid;
        else hi = mid;
    }
    c = lo;
    // equal shares
    const int nu = cells->unit[c + 1] - cells->unit[c], k = u - cells->unit[c];
    const int s = cells->start[c], e = cells->start[c + 1], per = (e - s + nu - 1) / nu;
    first = s + k * per;
    count = min(per, e - first);
    return true;
}

// moments over the sorted points: a unit's moments of the box's series
template <int K, int KIND, int SPEC, bool BI>
__global__ __launch_bounds__(256) void k_cell_points(const ChebPlan* __restrict__ plan, const CellGrid* __restrict__ grid,
                                                     const CellIndex* __restrict__ cells, int n_meas,
                                                     const AntRec* __restrict__ ant, const AntRec* __restrict__ rxa,
                                                     const MeasCheb* __restrict__ meas, double Kc,
                                                     const void* __restrict__ recs_v, int gx, float2* __restrict__ partial) {
    using Rec = typename std::conditional<KIND == 0, PtRec, QRec>::type;
    if (plan->KC != K) return;
    const long bid = blockIdx.x;
    const int lb = (int)((bid / 8) % gx), unit = (int)((bid / (8L * gx)) * 8 + (bid % 8));
    int c, first, count;
    if (!unit_points(cells, unit, c, first, count)) return;
    c = __builtin_amdgcn_readfirstlane(c);
    first = __builtin_amdgcn_readfirstlane(first);
    count = __builtin_amdgcn_readfirstlane(count);
    const int i = lb * blockDim.x + threadIdx.x;
    const int ic = i < n_meas ? i : n_meas - 1;
    const AntRec A = ant[ic];
    AntRec Rx = A;
    if constexpr (BI) Rx = rxa[ic];
    double rc, h;
    cell_interval<BI>(*grid, c, A, Rx, rc, h);
    float mr[K], mi[K];
#pragma unroll
    for (int k = 0; k < K; ++k) mr[k] = mi[k] = 0.0f;
    // Runs of kCellRun points summed by themselves: the FP32 sums of a whole unit (4096
    // points at 2^20 points x 1024 measurements) round twice as long as those of a split
    // without cells, which was 16 to 33 % of the outputs' error (against 64 bits: 2^19 points
    // in a 25 cm cube 5.8e-7, 4.3e-7 without cells, 3.1e-7 in runs of 64; 128: 3.3e-7,
    // 256: 3.7e-7, all within 1 % of the time).
    constexpr int kCellRun = 64;
    const double inv_h = 1.0 / h;
    const long end = (long)first + count;
    for (long j = first; j < end; j += kCellRun) {
        float br[K], bi[K];
#pragma unroll
        for (int k = 0; k < K; ++k) br[k] = bi[k] = 0.0f;
        cheb_moments<K, KIND, SPEC, BI>(A, Rx, rc, inv_h, Kc, reinterpret_cast<const Rec*>(recs_v), j, min(j + kCellRun, end),
                                        br, bi);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            mr[k] += br[k];
            mi[k] += bi[k];
        }
    }
    if (i < n_meas)
        cell_up<K>(mr, mi, plan->K, rc, h, meas[ic], partial + ((size_t)unit * n_meas + i) * kChebKMax);
}

// Reductions over frequencies: a work-group takes the points of a unit (two per
// lane) and the measurements 256 at a time: each lane forms one measurement's
// interval and cell coefficients in LDS, then all lanes walk them in step.
constexpr int kCellUnit = 512;
template <int K>
struct CellBatch {
    double2 iv[256];                             // rc, 1 / h
    float2 b[256 * K];
};

template <int K, bool BI>
__device__ __forceinline__ void batch_fill(CellBatch<K>& s, float2* b2, const CellGrid* __restrict__ grid, int c, int i, int n_meas,
                                           const AntRec* __restrict__ ant, const AntRec* __restrict__ rxa,
                                           const MeasCheb* __restrict__ meas, const float2* __restrict__ B,
                                           const float2* __restrict__ B2, int KP) {
    if (i >= n_meas) return;
    const AntRec A = ant[i];
    AntRec Rx = A;
    if constexpr (BI) Rx = rxa[i];
    double rc, h;
    cell_interval<BI>(*grid, c, A, Rx, rc, h);
    const MeasCheb box = meas[i];
    s.iv[threadIdx.x] = make_double2(rc, 1.0 / h);
    cell_down<K>(B + (size_t)i * kChebKMax, KP, rc, h, box, &s.b[threadIdx.x * K]);
    if (b2) cell_down<K>(B2 + (size_t)i * kChebKMax, KP, rc, h, box, &b2[threadIdx.x * K]);
}

template <int K, bool TWO, bool BI>
__global__ __launch_bounds__(256) void k_cell_mf(const ChebPlan* __restrict__ plan, const CellGrid* __restrict__ grid,
                                                 const CellIndex* __restrict__ cells, const int* __restrict__ perm,
                                                 const float* __restrict__ xq, int n_meas, const AntRec* __restrict__ ant,
                                                 const AntRec* __restrict__ rxa, const MeasCheb* __restrict__ meas,
                                                 const float2* __restrict__ B, const float2* __restrict__ B2, double Kc,
                                                 float2* __restrict__ z, float* __restrict__ power,
                                                 float2* __restrict__ z2, float* __restrict__ power2) {
    __shared__ CellBatch<K> sm;
    __shared__ float2 sb2[TWO ? 256 * K : 1];
    if (plan->KC != K) return;
    int c, first, count;
    if (!unit_points(cells, blockIdx.x, c, first, count)) return;
    const int tid = threadIdx.x, KP = plan->K;
    long q[2];
    double px[2], py[2], pz[2];
    float zr[2], zi[2], z2r[2], z2i[2];
    // a lane's second point exists where the wave's share reaches beyond 256
    const int nu = __builtin_amdgcn_readfirstlane(count > 256 + (tid & ~63) ? 2 : 1);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int p = tid + 256 * u;
        q[u] = perm[first + (p < count ? p : count - 1)];
        px[u] = (double)xq[3 * q[u]];
        py[u] = (double)xq[3 * q[u] + 1];
        pz[u] = (double)xq[3 * q[u] + 2];
        zr[u] = zi[u] = z2r[u] = z2i[u] = 0.0f;
    }
    auto pair = [&](int u, const AntRec& A, const AntRec& Rx, const double2& iv, const float2 (&b)[K],
                    const float2 (&b2)[TWO ? K : 1]) {
        float y;
        double r = range_f64(px[u] - A.x, py[u] - A.y, pz[u] - A.z, y);
        if constexpr (BI) {
            float yr;
            r = 0.5 * (r + range_f64(px[u] - Rx.x, py[u] - Rx.y, pz[u] - Rx.z, yr));
        }
        const float x = (float)((r - iv.x) * iv.y);
        const float t0 = frac_rev(r * Kc);
        const float c0 = cos_rev(t0), s0 = sin_rev(t0);       // exp(+j 2 pi Kc r)
        float sr, si;
        if constexpr (TWO) {
            float s2r, s2i;
            if constexpr (K <= kPowerK) {
                cell_series<K>(b, x, sr, si);
                cell_series<K>(b2, x, s2r, s2i);
            } else {
                cheb_series2<K>(b, b2, x, sr, si, s2r, s2i);
            }
            z2r[u] = __builtin_fmaf(c0, s2r, __builtin_fmaf(-s0, s2i, z2r[u]));
            z2i[u] = __builtin_fmaf(c0, s2i, __builtin_fmaf(s0, s2r, z2i[u]));
        } else {
            cell_series<K>(b, x, sr, si);
        }
        zr[u] = __builtin_fmaf(c0, sr, __builtin_fmaf(-s0, si, zr[u]));
        zi[u] = __builtin_fmaf(c0, si, __builtin_fmaf(s0, sr, zi[u]));
    };
    for (int i0 = 0; i0 < n_meas; i0 += 256) {
        __syncthreads();
        batch_fill<K, BI>(sm, TWO ? sb2 : nullptr, grid, c, i0 + tid, n_meas, ant, rxa, meas, B, B2, KP);
        __syncthreads();
        const int nb = min(256, n_meas - i0);
        for (int k = 0; k < nb; ++k) {
            const AntRec A = ant[i0 + k];
            AntRec Rx = A;
            if constexpr (BI) Rx = rxa[i0 + k];
            const double2 iv = sm.iv[k];
            float2 b[K], b2[TWO ? K : 1];
#pragma unroll
            for (int m = 0; m < K; ++m) b[m] = sm.b[k * K + m];
            if constexpr (TWO) {
#pragma unroll
                for (int m = 0; m < K; ++m) b2[m] = sb2[k * K + m];
            }
            pair(0, A, Rx, iv, b, b2);
            if (nu == 2) pair(1, A, Rx, iv, b, b2);
        }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (tid + 256 * u >= count) continue;
        mf_store(z, power, q[u], zr[u], zi[u]);
        if constexpr (TWO) mf_store(z2, power2, q[u], z2r[u], z2i[u]);
    }
}

template <int K, int SPEC, bool BI>
__global__ __launch_bounds__(256) void k_cell_render_bwd(const ChebPlan* __restrict__ plan, const CellGrid* __restrict__ grid,
                                                         const CellIndex* __restrict__ cells, const int* __restrict__ perm,
                                                         const PtRec* __restrict__ rec, int n_meas,
                                                         const AntRec* __restrict__ ant, const AntRec* __restrict__ rxa,
                                                         const MeasCheb* __restrict__ meas, const float2* __restrict__ B,
                                                         double Kc, float* __restrict__ g_b, float* __restrict__ g_T,
                                                         float* __restrict__ g_n) {
    __shared__ CellBatch<K> sm;
    if (plan->KC != K) return;
    int c, first, count;
    if (!unit_points(cells, blockIdx.x, c, first, count)) return;
    const int tid = threadIdx.x, KP = plan->K;
    const int nu = __builtin_amdgcn_readfirstlane(count > 256 + (tid & ~63) ? 2 : 1);
    long j[2];
    PtRec P[2];
    float gb[2], gt[2], gn0[2], gn1[2], gn2[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int p = tid + 256 * u;
        j[u] = perm[first + (p < count ? p : count - 1)];
        P[u] = rec[j[u]];
        gb[u] = gt[u] = gn0[u] = gn1[u] = gn2[u] = 0.0f;
    }
    auto pair = [&](int u, const AntRec& A, const AntRec& Rx, const double2& iv, const float2 (&b)[K]) {
        const double dx = P[u].x - A.x, dy = P[u].y - A.y, dz = P[u].z - A.z;
        float y, yr = 0.0f;
        double r = range_f64(dx, dy, dz, y);
        double ex = 0.0, ey = 0.0, ez = 0.0;
        if constexpr (BI) {
            ex = P[u].x - Rx.x; ey = P[u].y - Rx.y; ez = P[u].z - Rx.z;
            r = 0.5 * (r + range_f64(ex, ey, ez, yr));
        }
        const float x = (float)((r - iv.x) * iv.y);
        float sr, si;
        cell_series<K>(b, x, sr, si);
        bwd_pair<SPEC, BI>(P[u], A, Rx, dx, dy, dz, ex, ey, ez, r, y, yr, Kc, sr, si, gb[u], gt[u], gn0[u], gn1[u], gn2[u]);
    };
    for (int i0 = 0; i0 < n_meas; i0 += 256) {
        __syncthreads();
        batch_fill<K, BI>(sm, nullptr, grid, c, i0 + tid, n_meas, ant, rxa, meas, B, nullptr, KP);
        __syncthreads();
        const int nb = min(256, n_meas - i0);
        for (int k = 0; k < nb; ++k) {
            const AntRec A = ant[i0 + k];
            AntRec Rx = A;
            if constexpr (BI) Rx = rxa[i0 + k];
            const double2 iv = sm.iv[k];
            float2 b[K];
#pragma unroll
            for (int m = 0; m < K; ++m) b[m] = sm.b[k * K + m];
            pair(0, A, Rx, iv, b);
            if (nu == 2) pair(1, A, Rx, iv, b);
        }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
        if (tid + 256 * u < count) bwd_store<BI>(g_b, g_T, g_n, j[u], P[u].b, gb[u], gt[u], gn0[u], gn1[u], gn2[u]);
}

__global__ void k_cheb_order(const ChebPlan* __restrict__ plan, int32_t* __restrict__ order) {
    if (threadIdx.x == 0) *order = plan->K;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// up to this many points the plan's work-group takes the bounding box itself (a
// launch less; 16 points per thread).  Filter of 64 measurements x 32 frequencies, with
// it | with a launch of its own, in us: 4096 points 26.4 | 29.8, 16384 26.3 | 30.2, 32768
// 28.6 | 30.4, 65536 36.9 | 33.6.
constexpr long kPlanPoints = 16384;
int cheb_bbox_blocks(long n) {
    long b = (n + 4095) / 4096;
    return (int)(b < 1 ? 1 : (b > 1024 ? 1024 : b));
}

hipError_t launch_cheb_order(const ChebPlan* plan, int32_t* order, hipStream_t st) {
    hipLaunchKernelGGL(k_cheb_order, dim3(1), dim3(64), 0, st, plan, order);
    return hipGetLastError();
}

hipError_t launch_cheb_plan(const float* xyz, long n, const float* tx, const float* phi_tx, const float* rx,
                            const float* phi_rx, AntRec* ant, AntRec* rxa, int n_meas, double Kd, int n_freq,
                            float* bbox_part, MeasCheb* meas, ChebPlan* plan, CellGrid* grid, int max_cells, hipStream_t st) {
    int nb = 0;
    if (n > kPlanPoints) {
        nb = cheb_bbox_blocks(n);
        const long per = (n + nb - 1) / nb;
        hipLaunchKernelGGL(k_bbox_partial, dim3(nb), dim3(256), 0, st, xyz, n, per, bbox_part);
    }
    hipLaunchKernelGGL(k_cheb_plan, dim3(1), dim3(kPlanThreads), 0, st, xyz, n, bbox_part, nb, tx, phi_tx, rx, phi_rx, ant,
                       rxa, n_meas, Kd, n_freq, meas, plan, grid, max_cells);
    return hipGetLastError();
}

// wavenumber at the centre of the band (revolutions per metre of range)
static double band_centre(const RenderGeom& g) { return g.K0 + 0.5 * (double)(g.n_freq - 1) * g.Kd; }

// Below 2^23 pairs one launch serves every order: an empty launch costs 2 to 5 us,
// a moment kernel of 4096 points x 64 measurements 14.  Above, one per order:
// the order that runs does not pay for the registers and the schedule of the
// others (10^9 pairs at K = 28: 5.8 ms against 6.8 of a kernel for 24 and 28).
static bool one_launch(long n_pts, int n_meas) { return (double)n_pts * n_meas < 8388608.0; }

template <class Go>
static void by_order(long n_pts, int n_meas, Go go) {
    if (one_launch(n_pts, n_meas)) return go(std::integral_constant<int, 0>{});
    go(std::integral_constant<int, 24>{});
    go(std::integral_constant<int, 28>{});
    go(std::integral_constant<int, 32>{});
    go(std::integral_constant<int, 40>{});
    go(std::integral_constant<int, 48>{});
    go(std::integral_constant<int, 64>{});
}

// waves per work-group of the point reductions: as many of four as leave few lanes
// without a measurement
static int point_waves(int n_meas) {
    int w = 4;
    while (w > 1 && (n_meas + 64 * w - 1) / (64 * w) * w > (n_meas + 63) / 64 * 9 / 8) w /= 2;
    return w;
}

template <int KIND, int SPEC, bool BI>
static void launch_cp_all(const RenderGeom& g, const AntRec* ant, const MeasCheb* meas, const ChebPlan* plan,
                          const void* rec, int n_split, float2* partial, hipStream_t st) {
    const dim3 block(64 * point_waves(g.n_meas));
    const int gx = (g.n_meas + block.x - 1) / block.x;
    const long groups = (n_split + 7) / 8;
    dim3 grid((unsigned)(groups * 8 * gx));
    const long per = (g.n_pts + n_split - 1) / n_split;
    const double Kc = band_centre(g);
    by_order(g.n_pts, g.n_meas, [&](auto order) {
        hipLaunchKernelGGL((k_cheb_points<decltype(order)::value, KIND, SPEC, BI>), grid, block, 0, st, plan, g.n_meas, ant,
                           g.rxa, meas, Kc, rec, g.n_pts, per, n_split, gx, partial);
    });
}

// Measurement splits of the reductions over frequencies (a lane per point): as
// many as bring the launch to 8192 waves, eight per SIMD, of at least 8
// measurements each.  32768 points x 3200 measurements, 512 waves of points:
// filter forward 1458 us with one split, 286 with 16; render adjoint 1643, 362.
int cheb_meas_splits(long n_pts, int n_meas) {
    const long waves = (n_pts + 63) / 64;
    long ns = (8192 + waves - 1) / waves;
    if (ns > n_meas / 8) ns = n_meas / 8;
    return (int)(ns < 1 ? 1 : ns);
}

// Point splits of the moment kernels: twice the waves of the per-frequency
// kernels' rule (8192, eight per SIMD).  A lane's work per point is short at
// the lower orders, where five waves per SIMD fit, and more resident waves
// hide the scalar loads; >= 32 points per split (4096 points x 64
// measurements: 48 us with 32 splits of 128 points, 14 with 128).
int cheb_point_splits(long n_pts, int n_meas) {
    const long waves_per_split = (n_meas + 63) / 64;
    long ns = (8192 + waves_per_split - 1) / waves_per_split;
    const long max_by_pts = (n_pts + 31) / 32;
    if (ns > max_by_pts) ns = max_by_pts;
    if (ns < 1) ns = 1;
    if (ns > 65535) ns = 65535;
    return (int)ns;
}

// Where cells pay: the sort costs 50 to 100 us (hist, scan and scatter of 2^20 points
// 45 us, the idle kernels of the other orders the rest), the two ways between the series
// some per cent.  Measured without and with cells (20 cm cube, 64 frequencies, order
// 24 to 10 or 14; us per call):
//   over points (render, filter adjoint)   2^10 meas 2^16 pts 234 | 274, 215 | 245
//     2^10 x 2^17  392 | 381, 360 | 326    2^8 x 2^20   773 | 845, 654 | 695
//     2^10 x 2^19 1368 | 1152, 1204 | 935  2^12 x 2^15  402 | 417, 364 | 415
//     2^9 x 2^18   445 | 459, 411 | 392: fewer than 2^10 measurements from 2^28 pairs on
//   over frequencies (render adjoint, filter), whose work-groups take the points
//   of one cell and are too few below 2^19 points
//     2^10 x 2^18  925 | 985, 697 | 663    2^8 x 2^20  1138 | 1087, 597 | 552
//     2^10 x 2^19 1870 | 1598, 1339 | 1038
// At most one cell per 256 points, so that a cell's coefficients are used often enough,
// and of 2^21 cell-measurement pairs, whose moments take 1 GiB.  Positions are 32-bit.
int cell_count(long n_pts, int n_meas, bool over_points) {
    const double pairs = (double)n_pts * n_meas;
    const bool pays = over_points ? pairs >= (n_meas < 1024 ? 268435456.0 : 134217728.0) && n_meas >= 512 && n_pts >= (1L << 16)
                                  : pairs >= 268435456.0 && n_pts >= (1L << 19);
    if (!pays || n_pts > (1L << 24)) return 0;
    return (int)std::min({(long)kMaxCells, n_pts / 256, (1L << 21) / n_meas});
}
static int cell_per(long n) { return n >= (1L << 19) ? 1024 : 256; }
int cell_waves(long n) { return (int)((n + cell_per(n) - 1) / cell_per(n)); }
// points per unit of the point reductions: twice the per-split share of the launch
// without cells (few cells are cut then)
static int points_unit(long n_pts, int n_meas) {
    const int ns = cheb_point_splits(n_pts, n_meas);
    return (int)std::max<long>(2 * ((n_pts + ns - 1) / ns), 256);
}
int cell_point_units(long n_pts, int n_meas) {
    const int nc = cell_count(n_pts, n_meas, true);
    return nc ? (int)(n_pts / points_unit(n_pts, n_meas)) + nc : 0;
}

template <class Pos, class Rec>
static void cell_sort(const CellWs& w, const ChebPlan* plan, Pos pos, long n, int nc, int unit, int* perm, const Rec* rec,
                      Rec* out, hipStream_t st) {
    const int nw = cell_waves(n), per = cell_per(n);
    const dim3 grid((unsigned)((nw + 3) / 4));
    hipLaunchKernelGGL((k_cell_hist<Pos>), grid, dim3(256), 0, st, plan, w.grid, pos, n, per, nw, w.hist);
    hipLaunchKernelGGL(k_cell_scan, dim3(nc), dim3(256), 0, st, plan, w.grid, nw, w.hist, w.cells);
    hipLaunchKernelGGL((k_cell_scatter<Pos, Rec>), grid, dim3(256), 0, st, plan, w.grid, pos, n, per, nw, unit, w.hist,
                       w.cells, perm, rec, out);
}

template <class Go>
static void by_cell_order(Go go) {
    go(std::integral_constant<int, 8>{});
    go(std::integral_constant<int, 10>{});
    go(std::integral_constant<int, 12>{});
    go(std::integral_constant<int, 14>{});
    go(std::integral_constant<int, 16>{});
}

template <int KIND, int SPEC, bool BI>
static void launch_cell_points(const RenderGeom& g, const AntRec* ant, const MeasCheb* meas, const ChebPlan* plan,
                               const CellWs& cw, float2* partial, hipStream_t st) {
    const dim3 block(64 * point_waves(g.n_meas));
    const int gx = (g.n_meas + block.x - 1) / block.x;
    const long groups = (cell_point_units(g.n_pts, g.n_meas) + 7) / 8;
    by_cell_order([&](auto order) {
        hipLaunchKernelGGL((k_cell_points<decltype(order)::value, KIND, SPEC, BI>), dim3((unsigned)(groups * 8 * gx)), block, 0,
                           st, plan, cw.grid, cw.cells, g.n_meas, ant, g.rxa, meas, band_centre(g), cw.sorted, gx, partial);
    });
}

hipError_t launch_cheb_points(const RenderGeom& g, int kind, uint32_t flags, const AntRec* ant,
                              const MeasCheb* meas, const ChebPlan* plan, const void* rec, int n_split,
                              float2* partial, float2* out, int accumulate, const CellWs& cw, hipStream_t st) {
    const int nc = cw.max_cells;
    if (nc) {
        const int unit = points_unit(g.n_pts, g.n_meas);
        if (kind == 0) {
            const PtRec* r = static_cast<const PtRec*>(rec);
            cell_sort(cw, plan, PosRec{r}, g.n_pts, nc, unit, nullptr, r, static_cast<PtRec*>(cw.sorted), st);
        } else {
            const QRec* r = static_cast<const QRec*>(rec);
            cell_sort(cw, plan, PosQ{r}, g.n_pts, nc, unit, nullptr, r, static_cast<QRec*>(cw.sorted), st);
        }
    }
    const auto all = [&](auto kind_c, auto spec_c) {
        constexpr int KI = decltype(kind_c)::value, SP = decltype(spec_c)::value;
        if (nc) {
            if (g.rxa) launch_cell_points<KI, SP, true>(g, ant, meas, plan, cw, partial, st);
            else launch_cell_points<KI, SP, false>(g, ant, meas, plan, cw, partial, st);
        }
        if (g.rxa) launch_cp_all<KI, SP, true>(g, ant, meas, plan, rec, n_split, partial, st);
        else launch_cp_all<KI, SP, false>(g, ant, meas, plan, rec, n_split, partial, st);
    };
    using I1 = std::integral_constant<int, 1>;
    using I0 = std::integral_constant<int, 0>;
    if (kind == 1) {
        all(I1{}, std::integral_constant<int, RFVR_SPEC_OFF>{});
    } else {
        switch (flags & RFVR_SPEC_MASK) {
            case RFVR_SPEC_RAW: all(I0{}, std::integral_constant<int, RFVR_SPEC_RAW>{}); break;
            case RFVR_SPEC_OFF: all(I0{}, std::integral_constant<int, RFVR_SPEC_OFF>{}); break;
            default: all(I0{}, std::integral_constant<int, RFVR_SPEC_CLAMP>{}); break;
        }
    }
    hipLaunchKernelGGL(k_cheb_out, dim3(g.n_meas), dim3(256), 0, st, plan, meas, partial, n_split, g.n_meas, g.n_freq,
                       g.Kd, accumulate, out, cw.cells);
    return hipGetLastError();
}

hipError_t launch_cheb_coef(const RenderGeom& g, const ChebPlan* plan, const MeasCheb* meas, const float2* sig,
                            float2* B, hipStream_t st) {
    hipLaunchKernelGGL(k_cheb_coef, dim3(g.n_meas), dim3(256), 0, st, plan, meas, sig, g.n_meas, g.n_freq, g.Kd,
                       B);
    return hipGetLastError();
}

hipError_t launch_cheb_mf(const RenderGeom& g, const ChebPlan* plan, long n_q, const float* xq,
                          const AntRec* ant, const MeasCheb* meas, const float2* B, const float2* B2,
                          float2* z, float* power, float2* z2, float* power2, int n_split, float2* part,
                          const CellWs& cw, hipStream_t st) {
    const int nc = cw.max_cells;
    if (nc) cell_sort<PosXyz, QRec>(cw, plan, PosXyz{xq}, n_q, nc, kCellUnit, cw.perm, nullptr, nullptr, st);
    const int per = (g.n_meas + n_split - 1) / n_split;
    const dim3 grid((unsigned)((n_q + 255) / 256), (unsigned)n_split);
    if (n_split == 1) part = nullptr;
    const double Kc = band_centre(g);
    const auto all = [&](auto two, auto bi) {
        if (nc)
            by_cell_order([&](auto order) {
                hipLaunchKernelGGL((k_cell_mf<decltype(order)::value, decltype(two)::value, decltype(bi)::value>),
                                   dim3((unsigned)(n_q / kCellUnit + nc)), dim3(256), 0, st, plan, cw.grid, cw.cells, cw.perm,
                                   xq, g.n_meas, ant, g.rxa, meas, B, B2, Kc, z, power, z2, power2);
            });
        by_order(n_q, g.n_meas, [&](auto order) {
            hipLaunchKernelGGL((k_cheb_mf<decltype(order)::value, decltype(two)::value, decltype(bi)::value>), grid, dim3(256),
                               0, st, plan, n_q, xq, g.n_meas, per, ant, g.rxa, meas, B, B2, Kc, z, power, z2, power2, part);
        });
    };
    if (B2) {
        if (g.rxa) all(std::true_type{}, std::true_type{});
        else all(std::true_type{}, std::false_type{});
    } else {
        if (g.rxa) all(std::false_type{}, std::true_type{});
        else all(std::false_type{}, std::false_type{});
    }
    if (n_split > 1)
        hipLaunchKernelGGL(k_cheb_mf_sum, dim3(grid.x), dim3(256), 0, st, plan, n_q, part, n_split, B2 ? 1 : 0, z, power,
                           z2, power2);
    return hipGetLastError();
}

hipError_t launch_cheb_render_bwd(const RenderGeom& g, uint32_t flags, const ChebPlan* plan, const AntRec* ant,
                                  const MeasCheb* meas, const PtRec* rec, const float2* B, float* g_b,
                                  float* g_T, float* g_n, int n_split, float* part, const CellWs& cw,
                                  hipStream_t st) {
    const int nc = cw.max_cells;
    if (nc) cell_sort<PosRec, PtRec>(cw, plan, PosRec{rec}, g.n_pts, nc, kCellUnit, cw.perm, nullptr, nullptr, st);
    const int per = (g.n_meas + n_split - 1) / n_split;
    const dim3 grid((unsigned)((g.n_pts + 255) / 256), (unsigned)n_split);
    if (n_split == 1) part = nullptr;
    const double Kc = band_centre(g);
    const auto all = [&](auto spec_c) {
        constexpr int SP = decltype(spec_c)::value;
        const auto cell = [&](auto order, auto bi) {
            hipLaunchKernelGGL((k_cell_render_bwd<decltype(order)::value, SP, decltype(bi)::value>),
                               dim3((unsigned)(g.n_pts / kCellUnit + nc)), dim3(256), 0, st, plan, cw.grid, cw.cells, cw.perm,
                               rec, g.n_meas, ant, g.rxa, meas, B, Kc, g_b, g_T, g_n);
        };
        if (nc)
            by_cell_order([&](auto order) {
                if (g.rxa) cell(order, std::true_type{});
                else cell(order, std::false_type{});
            });
        by_order(g.n_pts, g.n_meas, [&](auto order) {
            constexpr int O = decltype(order)::value;
            if (g.rxa)
                hipLaunchKernelGGL((k_cheb_render_bwd<O, SP, true>), grid, dim3(256), 0, st, plan, g.n_pts, rec, g.n_meas,
                                   per, ant, g.rxa, meas, B, Kc, g_b, g_T, g_n, part);
            else
                hipLaunchKernelGGL((k_cheb_render_bwd<O, SP, false>), grid, dim3(256), 0, st, plan, g.n_pts, rec, g.n_meas,
                                   per, ant, g.rxa, meas, B, Kc, g_b, g_T, g_n, part);
        });
    };
    switch (flags & RFVR_SPEC_MASK) {
        case RFVR_SPEC_RAW: all(std::integral_constant<int, RFVR_SPEC_RAW>{}); break;
        case RFVR_SPEC_OFF: all(std::integral_constant<int, RFVR_SPEC_OFF>{}); break;
        default: all(std::integral_constant<int, RFVR_SPEC_CLAMP>{}); break;
    }
    if (n_split > 1) {
        const auto sum = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(grid.x), dim3(256), 0, st, plan, g.n_pts, rec, part, n_split, g_b, g_T, g_n);
        };
        if (g.rxa) sum(k_cheb_bwd_sum<true>);
        else sum(k_cheb_bwd_sum<false>);
    }
    return hipGetLastError();
}

}  // namespace rfvr
