// Refine, Gather and iterate (Steps 4-6 of Sec. 2.1) on the GPU.
//
// Step 4 fits a straight trajectory to each cluster by the multivariate
// regression of Sec. 2 (X = t, Y = (x, y)), with the mean and covariance of
// the Minimum Covariance Determinant subset in place of the sample ones.
// FAST-MCD (Rousseeuw and Van Driessen 1999) finds that subset: from random
// 4-point starts (an input table), C-steps - the mean and covariance of the
// current subset, the Mahalanobis distance of every point, the h closest as
// the next subset - never raise the determinant; two C-steps per start, the
// 10 lowest determinants iterated to convergence, the lowest wins.  Step 5
// gathers the catalog detections within the radius of the fitted line
// through the vote's window index; Step 6 repeats until the gathered set
// stops changing.
//
// One workgroup per cluster (grid-stride over clusters).  The point set
// (at most kMaxPoints) lives in LDS as t (h since t0), x, y (px) in FP64.
// The starts of FAST-MCD are independent, and their C-steps are nearly all
// the arithmetic.  A start takes one row of 16 lanes (4 starts a wave, 32 a
// workgroup; a whole wave above 128 points); a lane holds every 16th (64th)
// point in registers.  The sums cross the row by data-parallel primitive
// moves, the six or three divisions of a C-step are made by six or three
// lanes at once, and the h closest points come from a bisection on the upper
// 32 bits of the distances (ordered as integers), which ends as soon as a
// bound separates h points: about 12 passes of two instructions a point.
// Points whose upper bits tie across that bound are taken in the exact order
// (distance, position), so the subset is that of a full sort.  The sums keep
// the order of a butterfly over 64 lanes for every L, so a fit's bits do not
// depend on the form.  The kernel is bound by vector instructions (about 800
// a C-step of 4 starts at 64 points, half of them FP64) and by the rounds of
// the slowest cluster, which follow one another.
//   With one start a wave, ranks by comparing all pairs through LDS and
// reductions by LDS permutes, the 160 clusters of a fast chip (500 starts)
// took 5.9 ms, now 0.63 ms; the more of them gather sets in a cycle until the
// round limit, the longer (a chip of 8.0 ms: 1.5 ms before rounds that repeat
// were recognised, 0.64 after).
//
// Rules shared with the reference definition: a point set is ordered by
// catalog index; h = (n + 4) / 2; a start whose 4 points repeat, or whose
// covariance is degenerate (det <= 1e-12 S_tt S_xx S_yy), is dropped; a
// degenerate subset ends its C-steps; at most 30 C-steps per refined start
// and 10 rounds; fewer than 5 points end the iteration.
#include <math.h>

#include "internal.h"

namespace sas {
namespace {

// Threads per cluster workgroup.  512 leave a lane 256 registers; 1024 leave 128,
// with 116 more in scratch: 1000 clusters of 16 points and 30 starts took 1.7 times
// as long, 256 of 8 points 1.4 times what one start a wave had taken.
// Clusters, points and starts, in us for 1024 / 512 / 256 threads: 1000, 16, 30
// 712 / 417 / 416; 1000, 40, 500 1512 / 1367 / 1578; 160 of a fast chip, 500 starts
// 644 / 633 / 934.
constexpr int RT = 512;
constexpr int RW = RT / 64;
constexpr int kMaxPoints = 512;     // points of one set held in LDS
constexpr int kMaskWords = kMaxPoints / 32;
constexpr int kRowLanes = 16;
constexpr int kBest = 10;
constexpr int kMaxCsteps = 30;
constexpr int kMaxRounds = 10;
constexpr int kMinPoints = 5;
constexpr double kDegenerate = 1e-12;

struct Cov {
    double mu[3];
    double s[6];  // tt, tx, ty, xx, xy, yy (normalised by the point count)
};

__device__ inline double det3(const double *s) {
    return s[0] * (s[3] * s[5] - s[4] * s[4]) - s[1] * (s[1] * s[5] - s[4] * s[2]) +
           s[2] * (s[1] * s[4] - s[3] * s[2]);
}

__device__ inline bool degenerate(const double *s) {
    return det3(s) <= kDegenerate * s[0] * s[3] * s[5];
}

// Moves within a row of 16 lanes.
template <int CTRL>
__device__ inline int32_t dpp(int32_t v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ inline double dpp(double v) {
    return __hiloint2double(dpp<CTRL>(__double2hiint(v)), dpp<CTRL>(__double2loint(v)));
}
constexpr int kRor8 = 0x128, kRor4 = 0x124, kXor2 = 0x4e, kXor1 = 0xb1;  // 0x4e: quad 2,3,0,1
constexpr int kBcast = 0x150;                                            // row broadcast of lane n
// Sum over the row, in every lane: lanes l and l ^ 8 are added, then ^ 4, 2, 1
// (after the first step the values repeat with period 8, so a rotation by 4
// brings lane l ^ 4's).
template <class T>
__device__ inline T row_sum(T v) {
    v += dpp<kRor8>(v);
    v += dpp<kRor4>(v);
    v += dpp<kXor2>(v);
    return v + dpp<kXor1>(v);
}
__device__ inline uint32_t row_min(uint32_t v) {
    v = min(v, (uint32_t)dpp<kRor8>((int32_t)v));
    v = min(v, (uint32_t)dpp<kRor4>((int32_t)v));
    v = min(v, (uint32_t)dpp<kXor2>((int32_t)v));
    return min(v, (uint32_t)dpp<kXor1>((int32_t)v));
}
__device__ inline uint32_t row_max(uint32_t v) { return ~row_min(~v); }

// Inverse of the symmetric 3x3 matrix s (same layout), by cofactors; lane q
// of the row divides the q-th.
__device__ inline void inv3(const double *s, double *v) {
    const double c00 = s[3] * s[5] - s[4] * s[4];
    const double c01 = s[2] * s[4] - s[1] * s[5];
    const double c02 = s[1] * s[4] - s[2] * s[3];
    const double c11 = s[0] * s[5] - s[2] * s[2];
    const double c12 = s[1] * s[2] - s[0] * s[4];
    const double c22 = s[0] * s[3] - s[1] * s[1];
    const double d = s[0] * c00 + s[1] * c01 + s[2] * c02;
    const int q = __lane_id() & (kRowLanes - 1);
    double c = c00;
    c = q == 1 ? c01 : c;
    c = q == 2 ? c02 : c;
    c = q == 3 ? c11 : c;
    c = q == 4 ? c12 : c;
    c = q == 5 ? c22 : c;
    c /= d;
    v[0] = dpp<kBcast + 0>(c);
    v[1] = dpp<kBcast + 1>(c);
    v[2] = dpp<kBcast + 2>(c);
    v[3] = dpp<kBcast + 3>(c);
    v[4] = dpp<kBcast + 4>(c);
    v[5] = dpp<kBcast + 5>(c);
}

struct Shared {
    double zt[kMaxPoints], zx[kMaxPoints], zy[kMaxPoints];
    double dets[kMaxRefineStarts];
    // round r fits set r - 1 and gathers set r (catalog indices, ascending)
    int32_t sets[kMaxRounds + 1][kMaxPoints];
    int32_t n_set[kMaxRounds + 1];
    sas_refined fit[kMaxRounds];               // of round r at r - 1
    uint32_t subset[kMaxRounds][kMaskWords];   // its MCD subset of set r - 1
    int32_t tmp[kMaxPoints];
    uint32_t mask[kBest][kMaskWords];
    Cov cov[kBest];
    double cdet[kBest];
    int32_t top[kBest];
    int32_t n_top, n_nxt, overflow;
};

// A start's lanes: L = 16 (a row) or 64 (the wave).
template <int L, class T>
__device__ inline T lanes_sum(T v) {
    if (L == 64) {
        v += __shfl_xor(v, 32, 64);
        v += __shfl_xor(v, 16, 64);
    }
    return row_sum(v);
}
template <int L>
__device__ inline uint32_t lanes_min(uint32_t v) {
    v = row_min(v);
    if (L == 64) {
        v = min(v, (uint32_t)__shfl_xor((int32_t)v, 16, 64));
        v = min(v, (uint32_t)__shfl_xor((int32_t)v, 32, 64));
    }
    return v;
}

// The lane's points i = r + L k, k < P, with r = lane % L (L P >= n).
template <int L, int P>
struct Points {
    int n, r;
    double t[P], x[P], y[P];
    __device__ Points(const Shared &sh, int n_) : n(n_), r(__lane_id() & (L - 1)) {
#pragma unroll
        for (int k = 0; k < P; ++k) {
            t[k] = sh.zt[r + L * k];
            x[k] = sh.zx[r + L * k];
            y[k] = sh.zy[r + L * k];
        }
    }
};

// Partial sums of a lane of A, combined as a butterfly over 64 lanes with
// every 64th point each would: sums over every 64th point, then halves 32 and
// 16 apart (L = 16: within the lane), then the row.
template <int A>
__device__ __attribute__((always_inline)) inline double fold(const double *a) {
    return A == 1 ? a[0] : A == 2 ? a[0] + a[1] : (a[0] + a[2]) + (a[1] + a[3]);
}

// Mean and covariance of the points whose bit is set in `in`, cnt of them;
// every lane of the start gets the result.
template <int L, int P>
__device__ __attribute__((always_inline)) inline void moments(const Points<L, P> &pt, uint32_t in,
                                                              int cnt, Cov &c) {
    constexpr int A = L == 64 ? 1 : P < 4 ? P : 4;
    const int q = __lane_id() & (kRowLanes - 1);
    const double n = (double)cnt;
    double a0[A] = {}, a1[A] = {}, a2[A] = {};
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const bool on = (in >> k) & 1u;
        a0[k % A] += on ? pt.t[k] : 0.0;
        a1[k % A] += on ? pt.x[k] : 0.0;
        a2[k % A] += on ? pt.y[k] : 0.0;
    }
    const double m0 = lanes_sum<L>(fold<A>(a0)), m1 = lanes_sum<L>(fold<A>(a1)),
                 m2 = lanes_sum<L>(fold<A>(a2));
    double m = m0;
    m = q == 1 ? m1 : m;
    m = q == 2 ? m2 : m;
    m /= n;
    c.mu[0] = dpp<kBcast + 0>(m);
    c.mu[1] = dpp<kBcast + 1>(m);
    c.mu[2] = dpp<kBcast + 2>(m);
    double s[6][A] = {};
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const bool on = (in >> k) & 1u;
        const double dt = on ? pt.t[k] - c.mu[0] : 0.0, dx = on ? pt.x[k] - c.mu[1] : 0.0,
                     dy = on ? pt.y[k] - c.mu[2] : 0.0;
        s[0][k % A] += dt * dt;
        s[1][k % A] += dt * dx;
        s[2][k % A] += dt * dy;
        s[3][k % A] += dx * dx;
        s[4][k % A] += dx * dy;
        s[5][k % A] += dy * dy;
    }
    double v = 0.0;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        const double w = lanes_sum<L>(fold<A>(s[j]));
        v = q == j ? w : v;
    }
    v /= n;
    c.s[0] = dpp<kBcast + 0>(v);
    c.s[1] = dpp<kBcast + 1>(v);
    c.s[2] = dpp<kBcast + 2>(v);
    c.s[3] = dpp<kBcast + 3>(v);
    c.s[4] = dpp<kBcast + 4>(v);
    c.s[5] = dpp<kBcast + 5>(v);
}

// The h points closest to c.mu in the metric of the inverse of c.s (ties to
// the lower position), as bits of the lane's points.  Starts with live =
// false get no meaningful result.  All lanes of the wave call.
template <int L, int P>
__device__ __attribute__((always_inline)) inline uint32_t c_step(const Points<L, P> &pt, int h,
                                                                 const Cov &c, bool live) {
    double v[6];
    inv3(c.s, v);
    const auto dist = [&](int k) __attribute__((always_inline)) {
        const double a = pt.t[k] - c.mu[0], b = pt.x[k] - c.mu[1], e = pt.y[k] - c.mu[2];
        // + 0.0: a zero distance has one sign
        return a * (v[0] * a + v[1] * b + v[2] * e) + b * (v[1] * a + v[3] * b + v[4] * e) +
               e * (v[2] * a + v[4] * b + v[5] * e) + 0.0;
    };
    // upper halves of the distances, as integers in the same order; points
    // past the set above every bound
    uint32_t key[P], lo = 0xffffffffu, hi = 0;
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int32_t w = __double2hiint(dist(k));
        const bool on = pt.r + L * k < pt.n;
        key[k] = on ? (uint32_t)w ^ ((uint32_t)(w >> 31) | 0x80000000u) : 0xffffffffu;
        lo = min(lo, key[k]);
        hi = max(hi, on ? key[k] : 0u);
    }
    // bisection: fewer than h keys below lo, at least h below hi; a start ends
    // at a bound with exactly h below it, or with hi = lo + 1 (a tie)
    lo = lanes_min<L>(lo);
    hi = ~lanes_min<L>(~hi) + 1;
    uint32_t bound = 0;
    bool done = !live;
    for (;;) {
        const bool on = !done && hi - lo > 1u;
        if (!__any(on)) break;
        const uint32_t mid = lo + ((hi - lo) >> 1);
        int32_t below = 0;
#pragma unroll
        for (int k = 0; k < P; ++k) below += key[k] < mid ? 1 : 0;
        below = lanes_sum<L>(below);
        if (on) {
            if (below == h) {
                bound = mid;
                done = true;
            } else if (below < h) {
                lo = mid;
            } else {
                hi = mid;
            }
        }
    }
    uint32_t in = 0;
    const uint32_t cut = done ? bound : lo;
#pragma unroll
    for (int k = 0; k < P; ++k) in |= key[k] < cut ? 1u << k : 0u;
    if (__any(!done)) {
        // points tied at lo: the first ones by (distance, position)
        uint32_t tied = 0;
        int32_t need = 0;
#pragma unroll
        for (int k = 0; k < P; ++k) {
            tied |= !done && key[k] == lo && pt.r + L * k < pt.n ? 1u << k : 0u;
            need += key[k] < lo ? 1 : 0;
        }
        need = h - lanes_sum<L>(need);
        need = done ? 0 : need;
        constexpr int32_t kNone = kMaxPoints;
        while (__any(need > 0)) {
            double bd = 0.0;
            int32_t bi = kNone;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const double d = dist(k);
                if (((tied >> k) & 1u) && (bi == kNone || d < bd)) {
                    bd = d;
                    bi = pt.r + L * k;
                }
            }
#pragma unroll
            for (int o = L / 2; o > 0; o >>= 1) {
                const double od = __shfl_xor(bd, o, 64);
                const int32_t oi = __shfl_xor(bi, o, 64);
                if (oi != kNone && (bi == kNone || od < bd || (od == bd && oi < bi))) {
                    bd = od;
                    bi = oi;
                }
            }
            if (bi == kNone) {
                need = 0;  // not reached: a start holds more tied points than it needs
            } else if (need > 0) {
                --need;
                if (bi % L == pt.r) {
                    in |= 1u << (bi / L);
                    tied &= ~(1u << (bi / L));
                }
            }
        }
    }
    return in;
}

// Mean and covariance of the 4 points of start s, by every lane of the start.
// False when the start is dropped.
__device__ __attribute__((always_inline)) inline bool start_cov(const Shared &sh, int n,
                                                                const uint32_t *starts, int s,
                                                                Cov &c) {
    const int32_t jq = (int32_t)(starts[4 * s + (__lane_id() & 3)] % (uint32_t)n);
    const int j[4] = {dpp<0x00>(jq), dpp<0x55>(jq), dpp<0xaa>(jq), dpp<0xff>(jq)};  // of the quad
    double mu[3] = {0, 0, 0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        mu[0] += sh.zt[j[q]];
        mu[1] += sh.zx[j[q]];
        mu[2] += sh.zy[j[q]];
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) c.mu[r] = mu[r] / 4;
    double s6[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double dt = sh.zt[j[q]] - c.mu[0], dx = sh.zx[j[q]] - c.mu[1],
                     dy = sh.zy[j[q]] - c.mu[2];
        s6[0] += dt * dt;
        s6[1] += dt * dx;
        s6[2] += dt * dy;
        s6[3] += dx * dx;
        s6[4] += dx * dy;
        s6[5] += dy * dy;
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) c.s[q] = s6[q] / 4;
    return j[0] != j[1] && j[0] != j[2] && j[0] != j[3] && j[1] != j[2] && j[1] != j[3] &&
           j[2] != j[3] && !degenerate(c.s);
}

// Ascending sort of a[0, m) (distinct or not) into out by rank counting.  a
// is padded to a multiple of 4; ends with a barrier.
__device__ void sort_into(int32_t *a, int m, int32_t *out) {
    const int m4 = (m + 3) & ~3;
    if ((int)threadIdx.x < m4 - m) a[m + threadIdx.x] = INT32_MAX;  // above every index
    __syncthreads();
    for (int i = threadIdx.x; i < m; i += RT) {
        const int32_t v = a[i];
        int r = 0;
        for (int j = 0; j < m4; j += 4) {
            const int4 w = *(const int4 *)(a + j);
            r += (w.x < v || (w.x == v && j < i)) ? 1 : 0;
            r += (w.y < v || (w.y == v && j + 1 < i)) ? 1 : 0;
            r += (w.z < v || (w.z == v && j + 2 < i)) ? 1 : 0;
            r += (w.w < v || (w.w == v && j + 3 < i)) ? 1 : 0;
        }
        out[r] = v;
    }
    __syncthreads();
}

// The kBest lowest (determinant, start) of sh.dets, by one wave.
__device__ void best_starts(Shared &sh, int n_starts) {
    const int lane = __lane_id();
    constexpr int kHeld = kMaxRefineStarts / 64;
    double d[kHeld];
#pragma unroll
    for (int k = 0; k < kHeld; ++k)
        d[k] = lane + 64 * k < n_starts ? sh.dets[lane + 64 * k] : INFINITY;
    int nt = 0;
#pragma unroll 1
    for (; nt < kBest; ++nt) {
        double bd = INFINITY;  // of equal determinants the earlier start
        int bs = kMaxRefineStarts;
#pragma unroll
        for (int k = 0; k < kHeld; ++k)
            if (d[k] < bd) {
                bd = d[k];
                bs = lane + 64 * k;
            }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double od = __shfl_xor(bd, o, 64);
            const int os = __shfl_xor(bs, o, 64);
            if (od < bd || (od == bd && os < bs)) {
                bd = od;
                bs = os;
            }
        }
        if (bs == kMaxRefineStarts) break;
        if (lane == 0) sh.top[nt] = bs;
#pragma unroll
        for (int k = 0; k < kHeld; ++k)
            if (lane + 64 * k == bs) d[k] = INFINITY;
    }
    if (lane == 0) sh.n_top = nt;
}

// One stage of FAST-MCD on the n points in LDS (L P >= n).  Stage 0 scores
// every start by the determinant after two C-steps; stage 1 iterates the
// kBest lowest (sh.top; ties to the earlier start) until the subset holds,
// from the start again and one a wave, and leaves their subsets, moments and
// determinants in sh.
template <int L, int P>
__device__ __attribute__((always_inline)) inline void mcd_stage(Shared &sh, const RefineArgs &a,
                                                                int n, int h, int stage) {
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    constexpr int kStarts = 64 / L;  // starts a wave works on at once
    const Points<L, P> pt(sh, n);
    const int n_tasks = stage ? sh.n_top : a.n_starts;
    const int per_wave = stage ? 1 : kStarts;
    for (int t0 = wave * per_wave; t0 < n_tasks; t0 += RW * per_wave) {
        // the last start again past the end
        const int t = stage ? t0 : min(t0 + lane / L, n_tasks - 1);
        const int s = stage ? sh.top[t] : t;
        Cov c;
        const bool ok = start_cov(sh, n, a.starts, s, c);
        // the 4 points' step, the second, and kMaxCsteps more in stage 1; a
        // degenerate covariance or an unchanged subset ends a start
        uint32_t in = 0;
        bool on = ok;
        const int steps = stage ? 2 + kMaxCsteps : 2;
#pragma unroll 1
        for (int it = 0; it < steps; ++it) {
            if (it) on = on && !degenerate(c.s);
            if (!__any(on)) break;
            const uint32_t next = c_step<L, P>(pt, h, c, on);
            if (it) {
                const uint64_t moved = __ballot(next != in);
                on = on && (L == 64 ? moved : (moved >> (lane & ~(L - 1))) & 0xffffu) != 0;
            }
            if (!__any(on)) break;
            in = on ? next : in;
            // the same moments again for starts that have ended
            moments<L, P>(pt, in, h, c);
        }
        if (stage == 0) {
            if (pt.r == 0) sh.dets[s] = ok ? det3(c.s) : INFINITY;
            continue;
        }
#pragma unroll
        for (int k = 0; k < kMaxPoints / L; k += L == 64 ? 1 : 2) {
            uint64_t w = k < P ? __ballot((in >> k) & 1u) : 0;
            if (L == 16) {  // the wave's rows are alike
                const uint64_t w1 = k + 1 < P ? __ballot((in >> (k + 1)) & 1u) : 0;
                w = (w & 0xffffu) | (w1 & 0xffffu) << 16;
            }
            if (lane == 0) {
                sh.mask[t][L * k / 32] = (uint32_t)w;
                if (L == 64) sh.mask[t][2 * k + 1] = (uint32_t)(w >> 32);
            }
        }
        if (lane == 0) {
            sh.cov[t] = c;
            sh.cdet[t] = det3(c.s);
        }
    }
}

__device__ inline bool cell_span(int64_t lo, int64_t hi, int32_t f0, int32_t f1, int cl, int *c0,
                                 int *c1) {
    if (hi <= f0 || lo >= f1) return false;
    *c0 = (int)((max(lo, (int64_t)f0) - f0) >> cl);
    *c1 = (int)((min(hi, (int64_t)f1) - 1 - f0) >> cl);
    return true;
}

__global__ void __launch_bounds__(RT) k_refine_clusters(RefineArgs a) {
    __shared__ Shared sh;
    const int tid = threadIdx.x;
    const PreparedCatalog &c = a.cat;
    const double r2max = a.radius_px * a.radius_px;
    for (int64_t cl = blockIdx.x; cl < a.n_clusters; cl += gridDim.x) {
        const int32_t f = a.first[cl], m0 = a.first[cl + 1] - f;
        int status = SAS_REFINE_TOO_SMALL;
        int n = m0;
        __syncthreads();  // the previous cluster is done with the shared state
        if (tid == 0) sh.overflow = 0;
        __syncthreads();
        if (f < 0 || m0 < 0 || (int64_t)f + m0 > a.n_members) {
            status = SAS_REFINE_BAD_INPUT;
            n = -1;
        } else if (m0 > kMaxPoints) {
            status = SAS_REFINE_TOO_LARGE;
            n = -1;
        } else {
            for (int i = tid; i < m0; i += RT) {
                const int32_t q = a.members[f + i];
                if (q < 0 || q >= a.n) sh.overflow = 1;  // a member outside the catalog
                sh.tmp[i] = q;
            }
            __syncthreads();
            if (sh.overflow) {
                status = SAS_REFINE_BAD_INPUT;
                n = -1;
            } else {
                sort_into(sh.tmp, m0, sh.sets[0]);
                if (tid == 0) sh.n_set[0] = m0;
            }
        }
        int32_t n_g = 0;   // gathered by the last fit
        int rounds = 0;    // fits made
        int last = 0;      // the round whose fit stands (rounds, or its like in a cycle)
        int out_set = 0;   // the set reported as gathered
        for (int rnd = 1; n >= 0 && rnd <= kMaxRounds; ++rnd) {
            __syncthreads();
            if (n < kMinPoints) {
                status = SAS_REFINE_TOO_SMALL;
                break;
            }
            const int32_t *set = sh.sets[rnd - 1];
            for (int i = tid; i < n; i += RT) {
                const int32_t q = set[i];
                sh.zt[i] = (double)c.dt[a.epoch[q]] / 65536.0;
                sh.zx[i] = (double)a.x[q] / 256.0;
                sh.zy[i] = (double)a.y[q] / 256.0;
            }
            const int h = (n + 4) / 2;
            __syncthreads();
            // the smallest form that holds the set: a lane's work is per point held
#pragma unroll 1
            for (int stage = 0; stage < 2; ++stage) {
                if (n <= 32)
                    mcd_stage<16, 2>(sh, a, n, h, stage);
                else if (n <= 64)
                    mcd_stage<16, 4>(sh, a, n, h, stage);
                else if (n <= 128)
                    mcd_stage<16, 8>(sh, a, n, h, stage);
                else if (n <= 256)
                    mcd_stage<64, 4>(sh, a, n, h, stage);
                else
                    mcd_stage<64, 8>(sh, a, n, h, stage);
                __syncthreads();
                if (stage == 0) {
                    if (tid < 64) best_starts(sh, a.n_starts);
                    __syncthreads();
                }
            }
            const int n_top = sh.n_top;
            if (n_top == 0) {
                status = SAS_REFINE_NO_START;
                break;
            }
            int best = 0;
            for (int k = 1; k < n_top; ++k)
                if (sh.cdet[k] < sh.cdet[best]) best = k;
            double bx, by, cx, cy;
            {
                const Cov &cv = sh.cov[best];
                // the regression of Sec. 2 from the MCD mean and covariance
                bx = cv.s[1] / cv.s[0];
                by = cv.s[2] / cv.s[0];
                cx = cv.mu[1] - bx * cv.mu[0];
                cy = cv.mu[2] - by * cv.mu[0];
                if (tid == 0) {
                    sas_refined &r = sh.fit[rnd - 1];
                    r.vx = bx;
                    r.vy = by;
                    r.x0 = cx;
                    r.y0 = cy;
                    r.sxx = cv.s[3] - bx * bx * cv.s[0];
                    r.sxy = cv.s[4] - bx * by * cv.s[0];
                    r.syy = cv.s[5] - by * by * cv.s[0];
                    r.n_points = h;
                    sh.n_nxt = 0;
                }
                if (tid < kMaskWords) sh.subset[rnd - 1][tid] = sh.mask[best][tid];
            }
            rounds = last = rnd;
            __syncthreads();
            // Step 5: the catalog detections within the radius of c + B t, kGatherRows
            // threads an epoch, each every kGatherRows-th index row
            constexpr int kGatherRows = RT / kMaxEpochs;
            {
                const int e = tid / kGatherRows;
                const int32_t d = e < c.n_epochs ? c.dt[e] : -1;
                const double t = (double)d / 65536.0;
                const double px = cx + bx * t, py = cy + by * t;
                const double lo_x = (px - a.radius_px) * 256.0, hi_x = (px + a.radius_px) * 256.0;
                const double lo_y = (py - a.radius_px) * 256.0, hi_y = (py + a.radius_px) * 256.0;
                int cx0 = 0, cx1 = 0, cy0 = 0, cy1 = -1;
                if (d >= 0 && hi_x >= -2147483648.0 && lo_x < 2147483647.0 &&
                    hi_y >= -2147483648.0 && lo_y < 2147483647.0) {
                    const int64_t xlo = (int64_t)floor(lo_x), xhi = (int64_t)floor(hi_x) + 2;
                    const int64_t ylo = (int64_t)floor(lo_y), yhi = (int64_t)floor(hi_y) + 2;
                    if (!cell_span(xlo, xhi, c.x0, c.x1, c.cell_log2_x, &cx0, &cx1) ||
                        !cell_span(ylo, yhi, c.y0, c.y1, c.cell_log2_y, &cy0, &cy1))
                        cy1 = cy0 - 1;  // the window misses the footprint
                }
                for (int cy2 = cy0 + tid % kGatherRows; cy2 <= cy1; cy2 += kGatherRows) {
                    const int64_t base = ((int64_t)e * c.ncy + cy2) * c.ncx;
                    const int32_t j1 = c.off[base + cx1 + 1];
                    for (int32_t j = c.off[base + cx0]; j < j1; ++j) {
                        const int2 p = c.sxy[j];
                        const int32_t xq = a.weighted ? (p.x >> 8) : p.x;
                        const double ex = (double)xq / 256.0 - px, ey = (double)p.y / 256.0 - py;
                        if (ex * ex + ey * ey <= r2max) {
                            const int q = atomicAdd(&sh.n_nxt, 1);
                            if (q < kMaxPoints) sh.tmp[q] = c.sidx[j];
                        }
                    }
                }
            }
            __syncthreads();
            n_g = sh.n_nxt;
            if (n_g > kMaxPoints) {
                status = SAS_REFINE_TOO_LARGE;
                break;  // out_set: the set just fitted
            }
            sort_into(sh.tmp, n_g, sh.sets[rnd]);
            if (tid == 0) sh.n_set[rnd] = n_g;
            out_set = rnd;
            // Step 6: stop when the gathered set is the set just fitted.  A fit
            // depends on its set alone, so when the gathered set was fitted in an
            // earlier round q the rounds from q on repeat: the last round is like
            // the round of the cycle in its place.  (Three to eight of the fast
            // chip's 160 clusters end at the round limit, all in a cycle of two;
            // the others take two to four rounds.)
            int q = rnd;
            for (; q >= 1; --q) {
                if (sh.n_set[q - 1] != n_g) continue;  // block uniform
                int diff = 0;
                for (int i = tid; i < n_g; i += RT) diff |= sh.sets[rnd][i] != sh.sets[q - 1][i];
                if (__syncthreads_or(diff) == 0) break;
            }
            if (q == rnd) {
                status = SAS_REFINE_CONVERGED;
                break;
            }
            status = SAS_REFINE_MAX_ROUNDS;
            if (q >= 1) {
                last = q + (kMaxRounds - q) % (rnd + 1 - q);
                rounds = kMaxRounds;
                out_set = last;
                __syncthreads();  // n_set[rnd] is written
                n_g = sh.n_set[last];
                break;
            }
            n = n_g;
        }
        __syncthreads();
        if (last > 0 && a.subset && cl < a.subset_clusters) {  // the MCD subset (catalog indices)
            const uint32_t *mask = sh.subset[last - 1];
            for (int i = tid; i < sh.n_set[last - 1]; i += RT) {
                const uint32_t w = mask[i >> 5];
                if (!((w >> (i & 31)) & 1u)) continue;
                int r = __popc(w & ((1u << (i & 31)) - 1u));
                for (int j = 0; j < i >> 5; ++j) r += __popc(mask[j]);
                a.subset[cl * (int64_t)kMaxPoints + r] = sh.sets[last - 1][i];
            }
        }
        if (last > 0 && a.gathered) {
            // (a gathered set too large to hold leaves the set just fitted, then -1)
            const int m = min(n_g, min(kMaxPoints, a.gather_cap)), held = sh.n_set[out_set];
            for (int i = tid; i < m; i += RT)
                a.gathered[cl * (int64_t)a.gather_cap + i] = i < held ? sh.sets[out_set][i] : -1;
        }
        if (tid == 0) {
            sas_refined res{};
            if (last > 0) res = sh.fit[last - 1];
            res.n_gathered = n_g;
            res.rounds = rounds;
            res.status = status;
            a.out[cl] = res;
        }
    }
}

}  // namespace

hipError_t launch_refine_clusters(const RefineArgs &a, hipStream_t stream) {
    if (a.n_clusters <= 0) return hipSuccess;
    const unsigned grid = (unsigned)(a.n_clusters < 4096 ? a.n_clusters : 4096);
    hipLaunchKernelGGL(k_refine_clusters, dim3(grid), dim3(RT), 0, stream, a);
    return hipGetLastError();
}

}  // namespace sas
