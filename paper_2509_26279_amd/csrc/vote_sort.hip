// Sort-by-bin-key voting path for gfx950.
//
// Steps 1-2 of Sec. 2.1 with the Step-3 threshold, as a sort instead of a
// histogram: for a block of trial velocities, every (velocity j, detection i)
// vote becomes one 64-bit key
//     key = ((j * nby + (by - by0)) * nbx + (bx - bx0)) << 8 | epoch
// with (bx, by) the exact bin of Step 2 (floor((x - S(v)) / b), S(v) =
// ceil(v d / 65536)).  An LSD radix sort (8-bit digits, stable, only over the
// bits above the epoch byte) brings the votes of each (velocity, bin)
// together; one thread per run then counts its distinct epochs (or its
// length) and emits the run when the count reaches N_min.  The cost is in
// HBM: one key write, then per radix pass one read for the digit histogram
// and one read and one write for the scatter, then one read to count.
//
// Where a velocity's bins fit a few histograms in LDS and it is expected to be
// faster, the sort is left out: k_band_vote counts bands of whole bin rows of a
// velocity, reading for each epoch the contiguous stretch of the window index
// whose rows the band can reach, and counts distinct epochs in further readings
// for the bins whose detections reach N_min.  A vote then costs about 9 bytes of
// L2 reads and one LDS atomic in place of 80 to 104 bytes of HBM traffic: 512 of
// the slowest velocities of the fast grid and 180 k detections, of 4.5 bands
// each, take 5.15 ms by the sort and 0.21 ms with the preparation (0.12 ms
// k_band_vote, 7e11 votes/s).  A band costs its clearing, its dispatch and a walk
// over the epochs however few detections it holds: 1000 detections over 20000
// velocities of 26 bands take 9.5 ms, and 3.4 by the sort.
#include <algorithm>

#include "internal.h"

namespace sas {
namespace {

constexpr int T = 256;                  // threads per block
constexpr int NWV = T / 64;             // waves per block
constexpr int kKeys = kSortKeysPerTile / T;  // keys per thread in a radix tile
constexpr uint64_t kNoKey = ~(uint64_t)0;    // invalid detections sort last and are ignored

__device__ inline int32_t shift_q8(int32_t v, int32_t d) {
    return (int32_t)(((int64_t)v * (int64_t)d + 65535) >> 16);
}

__global__ void __launch_bounds__(T) k_sort_keygen(SortArgs a, SortBlock blk) {
    const int64_t total = (int64_t)blk.nv * a.n;
    const int64_t stride = (int64_t)gridDim.x * T;
    const uint64_t limit = (uint64_t)1 << blk.key_bits;
    for (int64_t t = (int64_t)blockIdx.x * T + threadIdx.x; t < total; t += stride) {
        const int64_t j = t / a.n, i = t - j * a.n;
        const int e = a.epoch[i];
        uint64_t key = kNoKey;
        if (e < a.n_epochs) {
            const int32_t d = a.dt[e];
            const int32_t vx = a.vel[2 * (blk.v_off + j)], vy = a.vel[2 * (blk.v_off + j) + 1];
            // arithmetic shifts: floor for negative positions too
            const int64_t bx = (int64_t)(a.x[i] - shift_q8(vx, d)) >> a.log2b;
            const int64_t by = (int64_t)(a.y[i] - shift_q8(vy, d)) >> a.log2b;
            const int64_t rx = bx - blk.bx0, ry = by - blk.by0;
            if (rx >= 0 && rx < blk.nbx && ry >= 0 && ry < blk.nby) {
                const uint64_t bin = ((uint64_t)j * blk.nby + (uint64_t)ry) * blk.nbx + (uint64_t)rx;
                if (bin < limit) key = bin << 8 | (uint64_t)e;
            }
        }
        a.keys[t] = key;
    }
}

// Digit counts of one radix tile: hist[digit * n_tiles + tile].
__global__ void __launch_bounds__(T) k_rs_hist(const uint64_t *__restrict__ in, int64_t m,
                                                int shift, int32_t *__restrict__ hist,
                                                int64_t n_tiles) {
    __shared__ int32_t cnt[256];
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * kSortKeysPerTile;
#pragma unroll
    for (int k = 0; k < kKeys; ++k) {
        const int64_t i = t0 + k * T + threadIdx.x;
        if (i < m) atomicAdd(&cnt[(int)((in[i] >> shift) & 255)], 1);
    }
    __syncthreads();
    hist[(int64_t)threadIdx.x * n_tiles + blockIdx.x] = cnt[threadIdx.x];
}

// Stable scatter of one radix tile.  The tile is taken in rounds of T
// consecutive keys; within a round, a key's rank among the keys of its wave
// with the same digit comes from eight ballots (one per digit bit), and the
// waves' counts per digit are combined in LDS, so equal digits keep their
// input order.
__global__ void __launch_bounds__(T) k_rs_scatter(const uint64_t *__restrict__ in,
                                                   uint64_t *__restrict__ out, int64_t m,
                                                   int shift, const int32_t *__restrict__ hist,
                                                   int64_t n_tiles) {
    __shared__ int32_t base[256];
    __shared__ int32_t wcnt[NWV][256];
    const int tid = threadIdx.x, lane = __lane_id(), wave = tid >> 6;
    const int64_t t0 = (int64_t)blockIdx.x * kSortKeysPerTile;
    base[tid] = hist[(int64_t)tid * n_tiles + blockIdx.x];
    const uint64_t lt = lane ? (~(uint64_t)0 >> (64 - lane)) : 0;  // lanes below this one
    for (int r = 0; r < kKeys; ++r) {
#pragma unroll
        for (int w = 0; w < NWV; ++w) wcnt[w][tid] = 0;
        __syncthreads();
        const int64_t i = t0 + (int64_t)r * T + tid;
        const bool valid = i < m;
        const uint64_t key = valid ? in[i] : 0;
        const int d = (int)((key >> shift) & 255);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t mb = __ballot((d >> b) & 1);
            peers &= ((d >> b) & 1) ? mb : ~mb;
        }
        const int rank = __popcll(peers & lt);
        if (valid && (peers & lt) == 0) wcnt[wave][d] = __popcll(peers);
        __syncthreads();
        if (valid) {
            int32_t pos = base[d] + rank;
            for (int w = 0; w < wave; ++w) pos += wcnt[w][d];
            out[pos] = key;
        }
        __syncthreads();
        int32_t add = 0;
#pragma unroll
        for (int w = 0; w < NWV; ++w) add += wcnt[w][tid];
        base[tid] += add;
    }
}

// Wave-aggregated append: one global atomic per wave.  All lanes must call.
__device__ inline int64_t wave_append(bool ok, unsigned long long *counter) {
    const uint64_t mask = __ballot(ok);
    if (mask == 0) return 0;
    unsigned long long b = 0;
    if (__lane_id() == 0) b = atomicAdd(counter, (unsigned long long)__popcll(mask));
    b = __shfl(b, 0, 64);
    const uint32_t pre = __builtin_amdgcn_mbcnt_hi(
        (uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    return (int64_t)b + pre;
}

// One thread per run head: count the run's distinct epochs (or its length).
__global__ void __launch_bounds__(T) k_sort_count(SortArgs a, SortBlock blk,
                                                   const uint64_t *__restrict__ keys, int64_t m) {
    __shared__ uint32_t masks[T][kSlotWords + 1];
    uint32_t *mk = masks[threadIdx.x];
    const int64_t stride = (int64_t)gridDim.x * T;
    for (int64_t i0 = (int64_t)blockIdx.x * T; i0 < m; i0 += stride) {
        const int64_t i = i0 + threadIdx.x;
        bool ok = false;
        uint32_t cnt = 0;
        uint64_t bin = 0;
        if (i < m) {
            const uint64_t key = keys[i];
            bin = key >> 8;
            const bool head = key != kNoKey && (i == 0 || (keys[i - 1] >> 8) != bin);
            if (head) {
                if (a.mode_epochs) {
#pragma unroll
                    for (int w = 0; w < kSlotWords; ++w) mk[w] = 0;
                    for (int64_t k = i; k < m && (keys[k] >> 8) == bin; ++k) {
                        const uint32_t e = (uint32_t)(keys[k] & 255);
                        mk[e >> 5] |= 1u << (e & 31);
                    }
#pragma unroll
                    for (int w = 0; w < kSlotWords; ++w) cnt += __popc(mk[w]);
                } else {
                    int64_t k = i;
                    while (k < m && (keys[k] >> 8) == bin) ++k;
                    cnt = (uint32_t)(k - i);
                }
                ok = cnt >= (uint32_t)a.n_min;
            }
        }
        const int64_t idx = wave_append(ok, (unsigned long long *)&a.res->n_cand);
        if (ok && idx < a.cand_cap) {
            const uint64_t plane = (uint64_t)blk.nbx * (uint64_t)blk.nby;
            const int64_t j = (int64_t)(bin / plane);
            const uint64_t rem = bin - (uint64_t)j * plane;
            const int32_t by = blk.by0 + (int32_t)(rem / (uint64_t)blk.nbx);
            const int32_t bx = blk.bx0 + (int32_t)(rem % (uint64_t)blk.nbx);
            const uint32_t sat = (uint32_t)a.count_sat;
            uint4 rec;
            rec.x = (uint32_t)a.v_idx[blk.v_off + j];
            rec.y = (uint32_t)bx;
            rec.z = (uint32_t)by;
            rec.w = (cnt > sat ? sat : cnt) | ((cnt > sat ? 1u : 0u) << 16);
            *(uint4 *)(a.cand + idx) = rec;
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

constexpr int BT = 512;  // threads of a band workgroup; two are resident on a CU
constexpr uint32_t kHot = 0x80000000u;

struct BandOut {
    const int32_t *v_idx;
    sas_candidate *cand;
    int64_t cand_cap;
    sas_vote_result *res;
    uint32_t sat;
};

// Counts of the bins [bx0, bx0 + nbx) x [by0, by0 + rows) of one velocity, nbx *
// rows <= kBandBins.  A workgroup takes one band of a table of them while the
// velocities are few, so that they share the chip evenly, and (EVERY) the bands
// of a velocity one after the other where there are many: dispatching a
// workgroup costs the chip some 15 ns, and the fast grid of 1.2e6 velocities has
// 1.6e7 bands, too many for one launch.  20000 of its velocities: 5.67 ms with
// the loop, 5.84 a band each; 512 fast ones: 208 us a band each, 223 us with the
// loop over eight shares of a velocity's bands, 221 us with bands worked out here
// instead of read.
template <bool EVERY>
__global__ void __launch_bounds__(BT) k_band_vote(SortArgs a, BandArgs b) {
    __shared__ uint32_t hist[kBandBins];
    __shared__ uint32_t mask[kBandMasks];
    __shared__ int32_t n_hot, n_out, n_put;
    __shared__ unsigned long long out_base;
    // what only candidates need: over the loop in LDS, not in scalar registers
    // that it has none left of
    __shared__ BandOut out_s;
    const BandOut out_a{a.v_idx, a.cand, a.cand_cap, a.res, (uint32_t)a.count_sat};
    if (EVERY && threadIdx.x == 0) out_s = out_a;
    const BandOut &out = EVERY ? out_s : out_a;
    const int tid = threadIdx.x;
    const PreparedCatalog &c = a.cat;
    const int E = c.n_epochs, lb = a.log2b;
    const int64_t u = b.first + blockIdx.x;
    int64_t v = u, by = 0, by_end = 0;
    int32_t bx0, nbx, by0, rows, high = 0;
    if constexpr (EVERY) {
        const BandBins r = reached_bins(a.vel[2 * u], a.vel[2 * u + 1], b.span, b.extent, lb);
        bx0 = (int32_t)r.bx0;
        nbx = (int32_t)(r.bx1 - r.bx0 + 1);
        high = __builtin_amdgcn_readfirstlane(r.rows());  // a division ends in a vector register
        by = r.by0;
        by_end = r.by1 + 1;
    } else {
        const int32_t *it = b.items + 5 * u;
        v = it[0];
        bx0 = it[1];
        nbx = it[2];
        by0 = it[3];
        rows = it[4];
    }
    const int32_t vx = a.vel[2 * v], vy = a.vel[2 * v + 1];
    do {
        if constexpr (EVERY) {
            by0 = (int32_t)by;
            rows = (int32_t)min((int64_t)high, by_end - by);
        }
        const int n_bins = nbx * rows;
        for (int i = tid; i < n_bins; i += BT) hist[i] = 0;
        if (tid == 0) n_hot = n_out = n_put = 0;
        __syncthreads();
        // f(word of the histogram, epoch) for every detection that projects into the
        // band: a wave an epoch, or the workgroup when there are few epochs
        const auto each = [&](const auto &f) __attribute__((always_inline)) {
            const bool by_wave = E >= 2 * (BT / 64);
            const int step = by_wave ? 64 : BT;
            const int first = by_wave ? (tid & 63) : tid;
            for (int e = by_wave ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0; e < E;
                 e += by_wave ? BT / 64 : 1) {
                const int32_t d = c.dt[e];
                if (d < 0) continue;
                const int32_t sx = shift_q8(vx, d), sy = shift_q8(vy, d);
                int cy0, cy1;
                if (!cell_span(((int64_t)by0 << lb) + sy, ((int64_t)(by0 + rows) << lb) + sy, c.y0,
                               c.y1, c.cell_log2_y, &cy0, &cy1))
                    continue;
                const int32_t j0 = c.off[((int64_t)e * c.ncy + cy0) * c.ncx];
                const int32_t j1 = c.off[((int64_t)e * c.ncy + cy1 + 1) * c.ncx];
                for (int32_t j = j0 + first; j < j1; j += 4 * step) {
                    int2 p[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (j + u * step < j1) p[u] = c.sxy[j + u * step];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        if (j + u * step >= j1) break;
                        const int32_t ix = ((p[u].x - sx) >> lb) - bx0, iy = ((p[u].y - sy) >> lb) - by0;
                        if ((uint32_t)iy < (uint32_t)rows && (uint32_t)ix < (uint32_t)nbx)
                            f(iy * nbx + ix, e);
                    }
                }
            }
        };
        each([&](int i, int) __attribute__((always_inline)) { atomicAdd(&hist[i], 1u); });
        __syncthreads();
        const uint32_t nmin = (uint32_t)a.n_min;
        // the bins whose count reaches nmin, `mine` of them found by this thread: one
        // global addition a workgroup (one a wave and 64 bins took 14 of the 14 ms of
        // 512 velocities and 4000 detections at a threshold of 1)
        const auto report = [&](int32_t mine, const auto &count_of) __attribute__((always_inline)) {
            if (mine) atomicAdd(&n_out, mine);
            __syncthreads();
            if (n_out == 0) return;  // block uniform
            if (tid == 0)
                out_base = atomicAdd((unsigned long long *)&out.res->n_cand,
                                     (unsigned long long)n_out);
            __syncthreads();
            for (int i = tid; i < n_bins; i += BT) {
                const uint32_t cnt = count_of(i), sat = out.sat;
                if (cnt < nmin) continue;
                const int64_t idx = (int64_t)out_base + atomicAdd(&n_put, 1);
                if (idx >= out.cand_cap) continue;
                uint4 rec;
                rec.x = (uint32_t)out.v_idx[v];
                rec.y = (uint32_t)(bx0 + i % nbx);
                rec.z = (uint32_t)(by0 + i / nbx);
                rec.w = (cnt > sat ? sat : cnt) | ((cnt > sat ? 1u : 0u) << 16);
                *(uint4 *)(out.cand + idx) = rec;
            }
        };
        int32_t mine = 0;
        if (!a.mode_epochs) {
            for (int i = tid; i < n_bins; i += BT) mine += hist[i] >= nmin ? 1 : 0;
            report(mine, [&](int i) __attribute__((always_inline)) { return hist[i]; });
            if (EVERY) __syncthreads();  // the counts are read before they are cleared
            continue;
        }
        // distinct epochs of the bins with nmin detections: each gets a number, and
        // the catalog is read again for as many of them as the masks hold
        const int W = (E + 31) / 32, held = kBandMasks / W;
        for (int i = tid; i < n_bins; i += BT)
            hist[i] = hist[i] >= nmin ? kHot | (uint32_t)atomicAdd(&n_hot, 1) : 0;
        __syncthreads();
        const int hot = n_hot;
        for (int s0 = 0; s0 < hot; s0 += held) {  // block uniform
            for (int i = tid; i < kBandMasks; i += BT) mask[i] = 0;
            if (tid == 0) n_out = n_put = 0;
            __syncthreads();
            each([&](int i, int e) __attribute__((always_inline)) {
                const uint32_t s = (hist[i] & ~kHot) - (uint32_t)s0;
                if (hist[i] & kHot && s < (uint32_t)held)
                    atomicOr(&mask[s * W + (e >> 5)], 1u << (e & 31));
            });
            __syncthreads();
            // the masks are counted first, in their first words: few bins are hot, and
            // most bands report none of them
            mine = 0;
            for (int s = tid; s < min(held, hot - s0); s += BT) {
                uint32_t n = 0;
                for (int w = 0; w < W; ++w) n += __popc(mask[s * W + w]);
                mask[s * W] = n;
                mine += n >= nmin ? 1 : 0;
            }
            report(mine, [&](int i) __attribute__((always_inline)) {
                const uint32_t h = hist[i], s = (h & ~kHot) - (uint32_t)s0;
                return h & kHot && s < (uint32_t)held ? mask[s * W] : 0u;
            });
            __syncthreads();
        }
    } while (EVERY && (by += high) < by_end);
}

inline unsigned grid_for(int64_t n, int64_t cap) {
    const int64_t b = (n + T - 1) / T;
    return (unsigned)(b < cap ? (b > 0 ? b : 1) : cap);
}

}  // namespace

hipError_t launch_radix_sort_u64(uint64_t *keys, uint64_t *alt, int64_t m, int lo_bit, int hi_bit,
                                 int32_t *hist, int32_t *hist_blocksum, hipStream_t stream,
                                 uint64_t **sorted) {
    const int64_t n_tiles = (m + kSortKeysPerTile - 1) / kSortKeysPerTile;
    uint64_t *in = keys, *out = alt;
    for (int shift = lo_bit; shift < hi_bit && m > 0; shift += 8) {
        hipLaunchKernelGGL(k_rs_hist, dim3((unsigned)n_tiles), dim3(T), 0, stream, in, m, shift,
                           hist, n_tiles);
        hipError_t e = launch_scan_exclusive(hist, 256 * n_tiles, hist_blocksum, stream);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_rs_scatter, dim3((unsigned)n_tiles), dim3(T), 0, stream, in, out, m,
                           shift, hist, n_tiles);
        uint64_t *tmp = in;
        in = out;
        out = tmp;
    }
    *sorted = in;
    return hipGetLastError();
}

hipError_t launch_band_vote(const SortArgs &a, const BandArgs &b, hipStream_t stream) {
    constexpr int64_t kGroups = (int64_t)1 << 22;
    static_assert(kGroups * BT < (int64_t)1 << 32, "a launch holds less than 2^32 threads");
    const int64_t n = b.items ? b.n_items : b.n_v;
    BandArgs l = b;
    for (; l.first < n; l.first += kGroups) {
        const dim3 grid((unsigned)std::min(n - l.first, kGroups));
        if (b.items)
            hipLaunchKernelGGL(k_band_vote<false>, grid, dim3(BT), 0, stream, a, l);
        else
            hipLaunchKernelGGL(k_band_vote<true>, grid, dim3(BT), 0, stream, a, l);
    }
    return hipGetLastError();
}

hipError_t launch_vote_sort_block(const SortArgs &a, const SortBlock &blk, hipStream_t stream) {
    const int64_t m = (int64_t)blk.nv * a.n;
    if (m <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_sort_keygen, dim3(grid_for(m, 1 << 16)), dim3(T), 0, stream, a, blk);
    uint64_t *in = nullptr;
    hipError_t e = launch_radix_sort_u64(a.keys, a.keys_alt, m, 8, 8 + blk.key_bits, a.hist,
                                         a.hist_blocksum, stream, &in);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sort_count, dim3(grid_for(m, 1 << 15)), dim3(T), 0, stream, a, blk,
                       (const uint64_t *)in, m);
    return hipGetLastError();
}

}  // namespace sas
