// Candidate features for learned vetting.
//
// One wave per candidate (v, bx, by).  Lanes take epochs; for its epoch a
// lane reads the window-index runs covering the bin's preimage
// [bx b + S(v), (bx + 1) b + S(v)) x [by b + S(vy), ...) with S(v) =
// ceil(v d / 65536) (the exact Step-2 bin of Sec. 2.1, as in the vote).  The
// contributing detections are packed into a list in LDS, so that each is then
// taken by a lane of its own, which gives in FP64 the SNR, the residuals r_x,
// r_y, their squares, the time coordinate tau = d / D, its square and its
// products with r, and the residuals of the time slice
// (min(3, floor(4 d / D))); counts come from ballots.  The 15 sums are
// reduced together: each exchange of half the lanes halves the number of
// values a lane carries (63 instructions; one butterfly after the other takes
// 360 and as many trips through LDS).  The quotients among the features are
// made by one division, each on the lane of its feature.
//   Neighbouring candidates are looked up in a hash table of the candidates'
// keys (open addressing, at most half full).
//   Bound by instruction issue and the chain index offsets - detections - SNR
// of dependent loads.  2e5 candidates of a wide-style pool: k_features 0.49 ms
// (1.79 ms before, at 5 waves a SIMD; 0.60 ms at the compiler's 3, 0.55 and
// 0.60 ms at 6 and 8, which spill), k_neighbours 0.17 ms with 0.02 ms for the
// table, in place of a sort of the keys (0.24 ms) and binary searches.
// The features, all by k_features but f9 and f10, which k_neighbours writes:
//   f0 c/E  f1 n/E  f2 min d/D  f3 (max d - min d)/D  f4 longest epoch run/E
//   f5 vx/vmax  f6 vy/vmax  f7 |v|/vmax  f8 sum snr/E
//   f9 neighbouring candidates/80  f10 largest count among them/own count
//   f11 mean snr - 3  f12, f13 mean r  f14, f15 std r
//   f16, f17 least-squares slope of r against tau (0 if all d equal)
//   f18..f25 per-slice mean r_x, r_y  f26..f29 slice fractions
//   f30 (n - c)/n  f31 RMS of r about the least-squares lines (x and y)
// with r_x = (65536 x - vx d) / (65536 b) - bx - 1/2.
#include "internal.h"

namespace sas {
namespace {

constexpr int FT = 256;  // threads per block: 4 candidates at a time

__device__ inline int32_t shift_q8(int32_t v, int32_t d) {
    return (int32_t)(((int64_t)v * (int64_t)d + 65535) >> 16);
}

// Neighbour key of a candidate: lattice velocity index (v / s rounded half
// up) and bin, packed 11 + 11 + 15 + 15 bits above a 12-bit count; all ones
// when a component is out of range (such a candidate has no neighbours).
constexpr uint64_t kNoNeighbourKey = ~(uint64_t)0;

// floor((2 v + s) / (2 s)) by a division in FP64: exact while the index is
// below 2^12 (the quotient of two integers below 2^34 that is no integer is
// 2^-34 or more from one, and its rounding error below 2^-41); a larger index
// has no neighbours whatever its value.
__device__ inline int32_t lattice_index(int32_t v, int32_t s) {
    const double q = floor((double)(2 * (int64_t)v + s) / (double)(2 * (int64_t)s));
    return (int32_t)fmin(fmax(q, -4096.0), 4096.0);
}

__device__ inline bool packable(int32_t ix, int32_t iy, int32_t bx, int32_t by) {
    return ix >= -1022 && ix <= 1022 && iy >= -1022 && iy <= 1022 && bx >= -16382 &&
           bx <= 16382 && by >= -16382 && by <= 16382;
}

__device__ inline uint64_t pack_key(int32_t ix, int32_t iy, int32_t bx, int32_t by) {
    return ((uint64_t)(ix + 1024) << 53) | ((uint64_t)(iy + 1024) << 42) |
           ((uint64_t)(bx + 16384) << 27) | ((uint64_t)(by + 16384) << 12);
}

__device__ inline uint64_t slot_of(uint64_t key, int table_log2) {
    return ((key >> 12) * 0x9E3779B97F4A7C15ull) >> (64 - table_log2);
}

__global__ void k_table_clear(uint64_t *__restrict__ table, int64_t n) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        table[i] = kNoNeighbourKey;
}

// Each candidate's key into the table; candidates that share a key keep the
// largest count.
__global__ void k_table_insert(FeatureArgs a) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n_cand) return;
    const sas_candidate cd = a.cand[i];
    const int32_t ix = lattice_index(a.vel[2 * (int64_t)cd.v_idx], a.spacing);
    const int32_t iy = lattice_index(a.vel[2 * (int64_t)cd.v_idx + 1], a.spacing);
    if (!packable(ix, iy, cd.bx, cd.by)) return;  // no neighbours
    const uint64_t key = pack_key(ix, iy, cd.bx, cd.by) | (uint64_t)min((int)cd.count, 4095);
    const uint64_t mask = ((uint64_t)1 << a.table_log2) - 1;
    unsigned long long *table = (unsigned long long *)a.table;
    for (uint64_t h = slot_of(key, a.table_log2);; h = (h + 1) & mask) {
        const uint64_t old = atomicCAS(&table[h], kNoNeighbourKey, key);
        if (old == kNoNeighbourKey) return;
        if ((old ^ key) >> 12 == 0) {
            atomicMax(&table[h], (unsigned long long)key);
            return;
        }
    }
}

// Largest count among the candidates with packed key `want` (count bits
// clear), or -1 when there is none.
__device__ inline int find_key(const uint64_t *table, int table_log2, uint64_t want) {
    const uint64_t mask = ((uint64_t)1 << table_log2) - 1;
    for (uint64_t h = slot_of(want, table_log2);; h = (h + 1) & mask) {
        const uint64_t cur = table[h];
        if (cur == kNoNeighbourKey) return -1;
        if ((cur ^ want) >> 12 == 0) return (int)(cur & 4095);
    }
}

// Neighbour features (f9, f10) of every candidate, a wave each: lane q takes
// offsets q and 64 + q of 81 (base 3 digits - 1).  A kernel of its own: the
// probes are random reads, and a wave that also held the sums of k_features
// would leave too few waves to cover them.
__global__ void __launch_bounds__(FT) k_neighbours(FeatureArgs a) {
    const int lane = __lane_id();
    const int64_t wave_id = ((int64_t)blockIdx.x * FT + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)gridDim.x * FT) >> 6;
    for (int64_t k = wave_id; k < a.n_cand; k += n_waves) {
        const sas_candidate cd = a.cand[k];
        int near = 0, best = 0;
        if (a.spacing > 0) {
            const int32_t ix = lattice_index(a.vel[2 * (int64_t)cd.v_idx], a.spacing);
            const int32_t iy = lattice_index(a.vel[2 * (int64_t)cd.v_idx + 1], a.spacing);
            if (packable(ix, iy, cd.bx, cd.by)) {
                int found[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int q = 64 * h + lane;
                    const int32_t jx = ix + q % 3 - 1, jy = iy + (q / 3) % 3 - 1;
                    const int32_t ex = cd.bx + (q / 9) % 3 - 1, ey = cd.by + q / 27 - 1;
                    found[h] = -1;
                    if (q < 81 && q != 40 && packable(jx, jy, ex, ey))  // 40: itself
                        found[h] = find_key(a.table, a.table_log2, pack_key(jx, jy, ex, ey));
                }
                near = __popcll(__ballot(found[0] >= 0)) + __popcll(__ballot(found[1] >= 0));
                best = max(found[0], found[1]);
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) best = max(best, __shfl_xor(best, o, 64));
            }
        }
        if (lane == 0) {
            const double own = (double)min((int)cd.count, 4095);
            a.feat[k * kFeatures + 9] = (float)((double)near / 80.0);
            a.feat[k * kFeatures + 10] =
                (float)(near > 0 && own > 0 ? (double)best / own : 0.0);
        }
    }
}

template <int CTRL>
__device__ inline int32_t dpp(int32_t v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ inline double dpp(double v) {
    return __hiloint2double(dpp<CTRL>(__double2hiint(v)), dpp<CTRL>(__double2loint(v)));
}
constexpr int kRor8 = 0x128, kRor4 = 0x124, kXor2 = 0x4e, kXor1 = 0xb1;  // within 16 lanes
constexpr int kXor7 = 0x141;                                             // half-row mirror

// Lanes 0..31: a summed over the halves of the wave; lanes 32..63: b (W = 16:
// even rows of 16 lanes a, odd rows b, summed over pairs of rows).
template <int W>
__device__ inline double exchange_add(double a, double b) {
    uint32_t w[2][2] = {{(uint32_t)__double2loint(a), (uint32_t)__double2loint(b)},
                        {(uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b)}};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const auto r = W == 32 ? __builtin_amdgcn_permlane32_swap(w[k][0], w[k][1], false, false)
                               : __builtin_amdgcn_permlane16_swap(w[k][0], w[k][1], false, false);
        w[k][0] = r[0];
        w[k][1] = r[1];
    }
    return __hiloint2double((int32_t)w[1][0], (int32_t)w[0][0]) +
           __hiloint2double((int32_t)w[1][1], (int32_t)w[0][1]);
}

// Wave sums of 16 values: the sum of v[q] ends in the lanes with sum_of() = q.
__device__ inline double reduce16(const double *v, int lane) {
    double u[8], w[4], y[2];
#pragma unroll
    for (int k = 0; k < 8; ++k) u[k] = exchange_add<32>(v[2 * k], v[2 * k + 1]);
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = exchange_add<16>(u[2 * k], u[2 * k + 1]);
    const bool b3 = lane & 8, b2 = lane & 4;
#pragma unroll
    for (int k = 0; k < 2; ++k)
        y[k] = (b3 ? w[2 * k + 1] : w[2 * k]) + dpp<kRor8>(b3 ? w[2 * k] : w[2 * k + 1]);
    double z = (b2 ? y[1] : y[0]) + dpp<kXor7>(b2 ? y[0] : y[1]);
    z += dpp<kXor1>(z);
    return z + dpp<kXor2>(z);
}
__device__ inline int sum_of(int lane) {  // rows hold values 0, 2, 1, 3 of four
    const int row = lane >> 4;
    return 8 * ((lane >> 2) & 1) + 4 * ((lane >> 3) & 1) + 2 * (row & 1) + (row >> 1);
}

__device__ inline int32_t wave_min(int32_t v) {
    v = min(v, dpp<kRor8>(v));
    v = min(v, dpp<kRor4>(v));
    v = min(v, dpp<kXor2>(v));
    v = min(v, dpp<kXor1>(v));
    return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

__device__ inline double lane_value(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Longest run of consecutive set bits of a 256-bit mask.
__device__ inline int longest_run(uint64_t m0, uint64_t m1, uint64_t m2, uint64_t m3) {
    int n = 0;
    while (m0 | m1 | m2 | m3) {
        ++n;
        m3 &= m3 << 1 | m2 >> 63;
        m2 &= m2 << 1 | m1 >> 63;
        m1 &= m1 << 1 | m0 >> 63;
        m0 &= m0 << 1;
    }
    return n;
}

constexpr int kList = 192;  // contributors listed before they are summed (64 more fit per step)

// Values a feature is the quotient of: the sums, then whole numbers and
// constants of the candidate.
enum Slot : int {
    kSnr = 0, kTau, kTau2, kTauX, kTauY, kX2, kY2, kX = 7, kY = 11,  // kX, kY: per slice
    kSums = 15,
    kEpochs = 16, kCount, kDmin, kDspan, kRun, kVx, kVy, kSlice,  // 4
    kDup = kSlice + 4, kE, kD,
    kInts = kD + 1 - kEpochs,
    kRx = kD + 1, kRy, kVmax, kZero, kSlots
};

__global__ void __launch_bounds__(FT) __attribute__((amdgpu_waves_per_eu(5))) k_features(FeatureArgs a) {
    __shared__ int2 list_s[FT / 64][kList + 64];
    __shared__ double val_s[FT / 64][kSlots];
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    int2 *list = list_s[wave];
    double *val = val_s[wave];
    const int64_t wave_id = ((int64_t)blockIdx.x * FT + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)gridDim.x * FT) >> 6;
    const PreparedCatalog &c = a.cat;
    const int E = c.n_epochs;
    const int lb = a.log2b;
    const double D = (double)a.span;
    const double inv_b = 1.0 / (65536.0 * (double)(1 << lb));
    // feature `lane`: numerator and denominator slots (lane 16: mean tau)
    static constexpr uint8_t kNum[32] = {
        kEpochs, kCount, kDmin, kDspan, kRun, kVx, kVy, kZero, kSnr, kZero, kZero, kSnr,
        kRx, kRy, kX2, kY2, kTau, kZero, kX, kY, kX + 1, kY + 1, kX + 2, kY + 2, kX + 3, kY + 3,
        kSlice, kSlice + 1, kSlice + 2, kSlice + 3, kDup, kZero};
    static constexpr uint8_t kDen[32] = {
        kE, kE, kD, kD, kE, kVmax, kVmax, kVmax, kE, kVmax, kVmax, kCount,
        kCount, kCount, kCount, kCount, kCount, kVmax, kSlice, kSlice, kSlice + 1, kSlice + 1,
        kSlice + 2, kSlice + 2, kSlice + 3, kSlice + 3,
        kCount, kCount, kCount, kCount, kCount, kVmax};
    const int num = kNum[lane & 31], den = kDen[lane & 31];
    const int my_sum = sum_of(lane);
    if (lane == 0) {
        val[kVmax] = a.vmax > 0 ? a.vmax : 1.0;
        val[kZero] = 0.0;
    }
    __shared__ int32_t dt_s[kMaxEpochs];
    for (int e = threadIdx.x; e < kMaxEpochs; e += FT) dt_s[e] = e < E ? c.dt[e] : -1;
    __syncthreads();
    sas_candidate next{};
    if (wave_id < a.n_cand) next = a.cand[wave_id];
    for (int64_t k = wave_id; k < a.n_cand; k += n_waves) {
        const sas_candidate cd = next;
        const int32_t vx = a.vel[2 * (int64_t)cd.v_idx], vy = a.vel[2 * (int64_t)cd.v_idx + 1];
        if (k + n_waves < a.n_cand) next = a.cand[k + n_waves];
        double sum = 0.0;  // of the lane's value sum_of(lane)
        int n = 0, slices[4] = {0, 0, 0, 0};  // wave uniform
        int32_t dmin = INT32_MAX, dmax_neg = INT32_MAX;
        uint64_t p0 = 0, p1 = 0, p2 = 0, p3 = 0;  // epoch presence (wave uniform)
        int q = -1;                               // epochs 64 q + lane (wave uniform)
        int e = 0, cx0 = 0, cx1 = 0, cy = 0, cy1 = -1;
        int32_t d = -1, j = 0, j1 = 0;
        int64_t xlo = 0, ylo = 0;
        bool has = false;
        for (bool done = false; !done;) {
            int listed = 0;  // wave uniform
            while (listed <= kList) {
                if (!__any(j < j1 || cy <= cy1)) {  // the next 64 epochs
                    const uint64_t m = __ballot(has);
                    if (q == 0) p0 = m;
                    else if (q == 1) p1 = m;
                    else if (q == 2) p2 = m;
                    else if (q == 3) p3 = m;
                    ++q;
                    if (64 * q >= E) {
                        done = true;
                        break;
                    }
                    has = false;
                    e = 64 * q + lane;
                    d = dt_s[e];
                    if (d >= 0) {
                        xlo = ((int64_t)cd.bx << lb) + shift_q8(vx, d);
                        ylo = ((int64_t)cd.by << lb) + shift_q8(vy, d);
                        const int64_t xhi = xlo + ((int64_t)1 << lb),
                                      yhi = ylo + ((int64_t)1 << lb);
                        if (xhi > c.x0 && xlo < c.x1 && yhi > c.y0 && ylo < c.y1) {
                            cx0 = (int)((max(xlo, (int64_t)c.x0) - c.x0) >> c.cell_log2_x);
                            cx1 = (int)((min(xhi, (int64_t)c.x1) - 1 - c.x0) >> c.cell_log2_x);
                            cy = (int)((max(ylo, (int64_t)c.y0) - c.y0) >> c.cell_log2_y);
                            cy1 = (int)((min(yhi, (int64_t)c.y1) - 1 - c.y0) >> c.cell_log2_y);
                        }
                    }
                    continue;
                }
                // one detection, or the next index row, a lane
                if (j >= j1 && cy <= cy1) {
                    const int64_t base = ((int64_t)e * c.ncy + cy) * c.ncx;
                    j = c.off[base + cx0];
                    j1 = c.off[base + cx1 + 1];
                    ++cy;
                }
                bool hit = false;
                if (j < j1) {
                    const int2 p = c.sxy[j];
                    hit = (uint64_t)((int64_t)p.x - xlo) >> lb == 0 &&
                          (uint64_t)((int64_t)p.y - ylo) >> lb == 0;
                }
                const uint64_t m = __ballot(hit);
                if (hit) {
                    const int at = __builtin_amdgcn_mbcnt_hi(
                        (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                    list[listed + at] = make_int2(j, d);
                    has = true;
                }
                j = j < j1 ? j + 1 : j;
                listed += __popcll(m);
            }
            // sums of the listed contributors
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            double s[16] = {};
            for (int i0 = 0; i0 < listed; i0 += 64) {
                int sl = -1;
                if (i0 + lane < listed) {
                    const int2 en = list[i0 + lane];
                    const int2 p = c.sxy[en.x];
                    const int64_t dd = en.y;
                    const double rx = (double)((int64_t)65536 * p.x - (int64_t)vx * dd) * inv_b -
                                      (double)cd.bx - 0.5;
                    const double ry = (double)((int64_t)65536 * p.y - (int64_t)vy * dd) * inv_b -
                                      (double)cd.by - 0.5;
                    const double tau = (double)dd / D;
                    if (a.snr) s[kSnr] += (double)a.snr[c.sidx[en.x]];
                    s[kTau] += tau;
                    s[kTau2] += tau * tau;
                    s[kTauX] += tau * rx;
                    s[kTauY] += tau * ry;
                    s[kX2] += rx * rx;
                    s[kY2] += ry * ry;
                    sl = (4 * dd >= a.span) + (4 * dd >= 2 * a.span) + (4 * dd >= 3 * a.span);
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        s[kX + t] += t == sl ? rx : 0.0;
                        s[kY + t] += t == sl ? ry : 0.0;
                    }
                    dmin = min(dmin, (int32_t)dd);
                    dmax_neg = min(dmax_neg, -(int32_t)dd);
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) slices[t] += __popcll(__ballot(sl == t));
            }
            sum += reduce16(s, lane);
            n += listed;
        }
        dmin = wave_min(dmin);
        const int32_t dmax = -wave_min(dmax_neg);
        const int cnt = __popcll(p0) + __popcll(p1) + __popcll(p2) + __popcll(p3);
        {   // the whole numbers, one a lane
            const int ints[kInts] = {cnt, n, dmin, (int)((uint32_t)dmax - (uint32_t)dmin), longest_run(p0, p1, p2, p3), vx, vy,
                                     slices[0], slices[1], slices[2], slices[3], n - cnt, E,
                                     (int)a.span};
            int iv = 0;
#pragma unroll
            for (int q = 0; q < kInts; ++q) iv = lane == q ? ints[q] : iv;
            if (lane < kInts) val[kEpochs + lane] = (double)iv;
            if ((lane & 3) == 0) val[my_sum] = sum;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const double rxs = (val[kX] + val[kX + 1]) + (val[kX + 2] + val[kX + 3]);
        const double rys = (val[kY] + val[kY + 1]) + (val[kY + 2] + val[kY + 3]);
        double f;
        {
            double u = val[num];
            u = lane == 7 ? sqrt((double)vx * vx + (double)vy * vy) : u;
            u = lane == 12 ? rxs : u;
            u = lane == 13 ? rys : u;
            const double v = val[den];
            f = v != 0.0 ? u / v : 0.0;  // empty slices, no contributors
        }
        if (n > 0) {
            const double dn = (double)n;
            const double mx = lane_value(f, 12), my = lane_value(f, 13), mt = lane_value(f, 16);
            const double sxx = val[kX2] - dn * mx * mx, syy = val[kY2] - dn * my * my;
            double q = 0.0, sse = sxx + syy;  // about the means, then about the fitted lines
            if (dmax > dmin) {
                const double stt = val[kTau2] - dn * mt * mt;
                const double sxt = val[kTauX] - dn * mt * mx, syt = val[kTauY] - dn * mt * my;
                q = (lane == 16 ? sxt : lane == 17 ? syt : sxt * sxt + syt * syt) / stt;
                sse -= q;  // lane 31
            }
            const double m = lane == 14 ? mx : my;
            const double r = sqrt(fmax(lane == 31 ? sse / (2.0 * dn) : f - m * m, 0.0));
            f = lane == 11 ? f - 3.0 : f;
            f = lane == 16 || lane == 17 ? q : f;
            f = lane == 14 || lane == 15 || lane == 31 ? r : f;
        } else {
            f = 0.0;
        }
        if (lane < kFeatures && lane != 9 && lane != 10)  // those: k_neighbours
            a.feat[k * kFeatures + lane] = (float)f;
        __builtin_amdgcn_wave_barrier();  // val and the list are read before they are refilled
    }
}

}  // namespace

hipError_t launch_features(const FeatureArgs &a, hipStream_t stream) {
    if (a.n_cand <= 0) return hipSuccess;
    if (a.spacing > 0) {
        // up to 2^32 slots, as many as a launch may hold threads: 65536 workgroups stride
        const int64_t slots = (int64_t)1 << a.table_log2;
        const int64_t clear_blocks = slots / 256 < 65536 ? slots / 256 : 65536;
        hipLaunchKernelGGL(k_table_clear, dim3((unsigned)clear_blocks), dim3(256), 0, stream,
                           a.table, slots);
        hipLaunchKernelGGL(k_table_insert, dim3((unsigned)((a.n_cand + 255) / 256)), dim3(256), 0,
                           stream, a);
    }
    const int64_t blocks = (a.n_cand + FT / 64 - 1) / (FT / 64);
    const dim3 grid((unsigned)(blocks < 65536 ? blocks : 65536));
    hipLaunchKernelGGL(k_neighbours, grid, dim3(FT), 0, stream, a);
    hipLaunchKernelGGL(k_features, grid, dim3(FT), 0, stream, a);
    return hipGetLastError();
}

}  // namespace sas
