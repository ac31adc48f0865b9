// Greedy cluster extraction (Step 3 of Sec. 2.1) on the GPU.
//
// The vote reports every (velocity, bin) at or above N_min.  Step 3 takes
// the maximum cell, calls the points that contributed to it a cluster,
// removes them from every cell they counted in, and repeats while the
// maximum still reaches N_min.  Counts only fall, so the loop runs over the
// reported cells; ties of the maximum go to the smaller (v_idx, by, bx).
//
//   1. k_contrib: one wave per reported cell gathers its contributors (the
//      detections whose exact Step-2 bin at the cell's velocity is the
//      cell) through the window index, as the vote does: lanes take epochs,
//      the contributors are packed into a list in LDS, counted (distinct
//      epochs by ballots) and written where the workgroup's share of the
//      list memory begins;
//   2. parallel rounds: a cell whose key (count, then the tie rule) beats
//      every open cell sharing a live detection with it is taken by the
//      sequential loop too, with exactly its current contributors - counts
//      only fall, so no neighbour can overtake it, and what is taken
//      elsewhere meanwhile shares none of its detections.  Each round takes
//      all such local maxima at once (every detection keeps the best open
//      cell holding it; a cell is a local maximum when it is the best of all
//      its live detections), removes their detections and recounts;
//   3. where the rounds leave open cells, an inverse index (detection -> cells
//      that hold it) by counting sort, and k_greedy: one workgroup finishes
//      one take at a time.  Each step a block reduction finds the maximum of
//      the stored counts under the tie rule (cells below N_min close), the
//      maximum's live contributors are taken and every open cell that held
//      one of them is queued; only the queued cells are recounted (one wave
//      each);
//   4. the keys taken by the sequential loop strictly increase (counts only
//      fall and the tie rule is total), so ranking the clusters by key
//      restores its order; the owners are renumbered to that order.
// On a chip's few thousand cells the call is the latency of its launches: 22
// now, 40 before with the lists counted and then written, the inverse index
// always built and one same-address atomic per cell (3128 cells of the wide
// chip: 382 us a call before, 261 us now, 120 us of them kernels).
#include <algorithm>

#include "internal.h"

namespace sas {
namespace {

constexpr int CT = 256;    // threads per gather block (4 cells at a time)
constexpr int GT = 1024;   // threads of the greedy workgroup
constexpr int GW = GT / 64;

__device__ inline int32_t shift_q8(int32_t v, int32_t d) {
    return (int32_t)(((int64_t)v * (int64_t)d + 65535) >> 16);
}

__device__ inline bool cell_span(int64_t lo, int64_t hi, int32_t f0, int32_t f1, int cl, int *c0,
                                 int *c1) {
    if (hi <= f0 || lo >= f1) return false;
    *c0 = (int)((max(lo, (int64_t)f0) - f0) >> cl);
    *c1 = (int)((min(hi, (int64_t)f1) - 1 - f0) >> cl);
    return true;
}

// f(hit, position, epoch) for the detections the lanes meet on the way to the
// contributors of cell cd, lanes over epochs; every lane calls f at every
// step.  chunk(): after each 64 epochs.
template <class F, class C>
__device__ __attribute__((always_inline)) inline void walk_cell(const ExtractArgs &a,
                                                                const sas_candidate &cd,
                                                                const F &f, const C &chunk) {
    const PreparedCatalog &c = a.cat;
    const int lane = __lane_id(), lb = a.log2b;
    const int32_t vx = a.vel[2 * (int64_t)cd.v_idx], vy = a.vel[2 * (int64_t)cd.v_idx + 1];
    for (int e0 = 0; e0 < c.n_epochs; e0 += 64) {
        const int e = e0 + lane;
        const int32_t d = e < c.n_epochs ? c.dt[e] : -1;
        const int64_t xlo = ((int64_t)cd.bx << lb) + shift_q8(vx, d);
        const int64_t ylo = ((int64_t)cd.by << lb) + shift_q8(vy, d);
        int cx0 = 0, cx1 = 0, cy = 0, cy1 = -1;
        if (d >= 0) {
            if (!cell_span(xlo, xlo + ((int64_t)1 << lb), c.x0, c.x1, c.cell_log2_x, &cx0, &cx1) ||
                !cell_span(ylo, ylo + ((int64_t)1 << lb), c.y0, c.y1, c.cell_log2_y, &cy, &cy1))
                cy1 = cy - 1;
        }
        int32_t j = 0, j1 = 0;
        for (;;) {
            if (j >= j1 && cy <= cy1) {
                const int64_t base = ((int64_t)e * c.ncy + cy) * c.ncx;
                j = c.off[base + cx0];
                j1 = c.off[base + cx1 + 1];
                ++cy;
            }
            const bool on = j < j1;
            if (!__any(on || cy <= cy1)) break;
            bool hit = false;
            if (on) {
                const int2 p = c.sxy[j];
                hit = (uint64_t)((int64_t)p.x - xlo) >> lb == 0 &&
                      (uint64_t)((int64_t)p.y - ylo) >> lb == 0;
            }
            f(hit, j, e);
            if (on) ++j;
        }
        chunk();
    }
}

__device__ inline int lane_rank(uint64_t m) {  // set bits of m below this lane
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

constexpr int kList = 256;  // contributors listed in LDS; longer lists are walked twice

__global__ void __launch_bounds__(CT) k_contrib(ExtractArgs a) {
    __shared__ int2 list_s[CT / 64][kList];
    __shared__ int32_t n_s[CT / 64];
    __shared__ unsigned long long base;
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    int2 *list = list_s[wave];
    for (int64_t k0 = (int64_t)blockIdx.x * (CT / 64); k0 < a.n_cand;
         k0 += (int64_t)gridDim.x * (CT / 64)) {
        const int64_t k = k0 + wave;
        const bool on = k < a.n_cand;  // wave uniform
        sas_candidate cd{};
        int32_t n = 0, epochs = 0;  // wave uniform
        if (on) {
            cd = a.cand[k];
            bool has = false;
            walk_cell(
                a, cd,
                [&](bool hit, int32_t j, int e) __attribute__((always_inline)) {
                    const uint64_t m = __ballot(hit);
                    const int at = n + lane_rank(m);
                    if (hit && at < kList) list[at] = make_int2(j, e);
                    has |= hit;
                    n += __popcll(m);
                },
                [&]() __attribute__((always_inline)) {
                    epochs += __popcll(__ballot(has));
                    has = false;
                });
        }
        if (lane == 0) n_s[wave] = n;
        __syncthreads();
        if (threadIdx.x == 0) {  // one allocation a workgroup
            int64_t sum = 0;
            for (int w = 0; w < CT / 64; ++w) sum += n_s[w];
            base = atomicAdd(a.n_members, (unsigned long long)sum);
        }
        __syncthreads();
        int64_t at = (int64_t)base;
        for (int w = 0; w < wave; ++w) at += n_s[w];
        const bool fits = at + n <= a.member_cap;
        if (on && lane == 0) {
            a.first[k] = (int32_t)min(at, (int64_t)INT32_MAX);
            a.len[k] = n;
            const int32_t cnt = a.mode_epochs ? epochs : n;
            a.count[k] = cnt;
            a.open[k] = cnt >= a.n_min;
            if (cnt >= a.n_min) a.counters[2] = 1;  // an open cell
        }
        if (on && fits && n <= kList) {
            for (int i = lane; i < n; i += 64) {
                const int2 m = list[i];
                a.member[at + i] = m.x;
                a.member_epoch[at + i] = (uint8_t)m.y;
                a.member_cell[at + i] = (int32_t)k;
            }
        } else if (on && fits) {
            int64_t to = at;  // wave uniform
            walk_cell(
                a, cd,
                [&](bool hit, int32_t j, int e) __attribute__((always_inline)) {
                    const uint64_t m = __ballot(hit);
                    if (hit) {
                        const int64_t q = to + lane_rank(m);
                        a.member[q] = j;
                        a.member_epoch[q] = (uint8_t)e;
                        a.member_cell[q] = (int32_t)k;
                    }
                    to += __popcll(m);
                },
                []() {});
        }
        __syncthreads();  // base, n_s and the lists are read before they are refilled
    }
}

// (count, v_idx, by, bx) order of the maximum: larger count, then smaller
// v_idx, by, bx.
struct Best {
    int32_t count, k;
    uint32_t v;
    int32_t by, bx;
};

__device__ inline bool better(const Best &p, const Best &q) {
    if (p.k < 0) return false;
    if (q.k < 0) return true;
    if (p.count != q.count) return p.count > q.count;
    if (p.v != q.v) return p.v < q.v;
    if (p.by != q.by) return p.by < q.by;
    return p.bx < q.bx;
}

__device__ inline Best shfl_best(const Best &b, int src) {
    Best o;
    o.count = __shfl(b.count, src, 64);
    o.k = __shfl(b.k, src, 64);
    o.v = (uint32_t)__shfl((int32_t)b.v, src, 64);
    o.by = __shfl(b.by, src, 64);
    o.bx = __shfl(b.bx, src, 64);
    return o;
}

// Whether the contributor lists fit (all kernels after the lists read it).
__device__ inline bool lists_fit(const ExtractArgs &a) {
    return *a.n_members <= (unsigned long long)a.member_cap;
}

// Whether the rounds left an open cell (or there were none): the sequential
// finish and its inverse index are needed.
__device__ inline bool cells_left(const ExtractArgs &a) {
    return lists_fit(a) && a.counters[2 + a.rounds] != 0;
}

// Per-detection state, the inverse index counts and the counters.
__global__ void k_extract_init(ExtractArgs a) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t j = t0; j < a.n; j += stride) {
        a.died[j] = 0;
        a.best[j] = -1;
        a.cluster_of[j] = -1;
    }
    if (t0 < kExtractCounters) a.counters[t0] = 0;
    if (t0 == 0) *a.n_members = 0;
    for (int64_t k = t0; k < a.n_cand; k += stride) a.dirty[k] = 0;
}

__global__ void k_inv_zero(ExtractArgs a) {
    if (!cells_left(a)) return;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j <= a.n; j += stride) {
        a.inv_first[j] = 0;
        if (j < a.n) a.inv_cursor[j] = 0;
    }
}

__global__ void k_inv_count(ExtractArgs a) {
    if (!cells_left(a)) return;
    const int64_t n_members = (int64_t)*a.n_members;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; m < n_members; m += stride)
        atomicAdd(&a.inv_first[a.member[m]], 1);
}

__global__ void k_inv_fill(ExtractArgs a) {
    if (!cells_left(a)) return;
    const int64_t n_members = (int64_t)*a.n_members;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; m < n_members; m += stride) {
        const int32_t j = a.member[m];
        a.inv[a.inv_first[j] + atomicAdd(&a.inv_cursor[j], 1)] = a.member_cell[m];
    }
}

// Count of cell k over its live contributors, by one wave (wave uniform);
// wmask: 8 words of LDS for this wave.
__device__ int32_t recount(const ExtractArgs &a, int64_t k, uint32_t *wmask) {
    const int lane = __lane_id();
    if (lane < kSlotWords) wmask[lane] = 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int32_t f = a.first[k], l = f + a.len[k];
    int32_t n = 0;
    for (int32_t m = f + lane; m < l; m += 64) {
        if (a.died[a.member[m]]) continue;
        if (a.mode_epochs) {
            const uint32_t e = a.member_epoch[m];
            atomicOr(&wmask[e >> 5], 1u << (e & 31));
        } else {
            ++n;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (a.mode_epochs) n = lane < kSlotWords ? __popc(wmask[lane]) : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
    return n;
}

// Whether cell k beats cell c (c < 0: no cell) under the order of the
// maximum: larger count, then smaller v_idx, by, bx.
__device__ inline bool cell_better(const ExtractArgs &a, int32_t k, int32_t c) {
    if (c < 0) return true;
    const int32_t ck = a.count[k], cc = a.count[c];
    if (ck != cc) return ck > cc;
    const sas_candidate &p = a.cand[k], &q = a.cand[c];
    if (p.v_idx != q.v_idx) return p.v_idx < q.v_idx;
    if (p.by != q.by) return p.by < q.by;
    return p.bx < q.bx;
}

// A parallel round may run: the lists fit and the previous round left an
// open cell.
__device__ inline bool round_active(const ExtractArgs &a, int r) {
    return lists_fit(a) && a.counters[2 + r - 1] != 0;
}

#define FOR_CELLS(k)                                                                    \
    const int64_t wave_id = ((int64_t)blockIdx.x * CT + threadIdx.x) >> 6;             \
    const int64_t n_waves = ((int64_t)gridDim.x * CT) >> 6;                              \
    for (int64_t k = wave_id; k < a.n_cand; k += n_waves)

// Record of a cluster taken as number s: its cell, with the key of the order.
__device__ inline void record_taken(const ExtractArgs &a, int32_t s, int32_t k) {
    const sas_candidate cd = a.cand[k];
    a.taken[s] = make_int4(a.count[k], (int32_t)cd.v_idx, cd.by, cd.bx);
}

// Round r, step 1: every live detection of an open cell keeps the best
// open cell holding it (compare-and-swap until it holds the better one).
__global__ void __launch_bounds__(CT) k_round_best(ExtractArgs a, int r) {
    if (!round_active(a, r)) return;
    FOR_CELLS(k) {
        if (!a.open[k]) continue;  // wave uniform
        const int32_t f = a.first[k], l = f + a.len[k];
        for (int32_t m = f + __lane_id(); m < l; m += 64) {
            const int32_t j = a.member[m];
            if (a.died[j]) continue;
            int32_t cur = a.best[j];
            while (cell_better(a, (int32_t)k, cur)) {
                const int32_t old = atomicCAS(&a.best[j], cur, (int32_t)k);
                if (old == cur) break;
                cur = old;
            }
        }
    }
}

// Step 2: a cell that is the best of all its live detections is taken, and
// they leave.  A detection that leaves in this round counts as live until it
// ends (died = r), so the cells it keeps from being taken still see it; the
// live sets of the taken cells are disjoint (a detection has one best cell).
__global__ void __launch_bounds__(CT) k_round_take(ExtractArgs a, int r) {
    if (!round_active(a, r)) return;
    FOR_CELLS(k) {
        if (!a.open[k]) continue;
        const int32_t f = a.first[k], l = f + a.len[k];
        bool mine = true;
        for (int32_t m = f + __lane_id(); m < l; m += 64) {
            const int32_t j = a.member[m];
            const int d = a.died[j];
            if ((d == 0 || d == r) && a.best[j] != (int32_t)k) mine = false;
        }
        if (!__all(mine)) continue;
        int32_t s = 0;
        if (__lane_id() == 0) {
            s = atomicAdd(&a.counters[0], 1);
            record_taken(a, s, (int32_t)k);
            a.open[k] = 0;
        }
        s = __shfl(s, 0, 64);
        for (int32_t m = f + __lane_id(); m < l; m += 64) {
            const int32_t j = a.member[m];
            if (a.died[j]) continue;
            a.cluster_of[a.cat.sidx[j]] = s;
            a.died[j] = (uint8_t)r;
        }
    }
}

// Step 3: recount the open cells, close those below N_min, note whether any
// is left, and clear the best cell of their detections for the next round.
__global__ void __launch_bounds__(CT) k_round_recount(ExtractArgs a, int r) {
    __shared__ uint32_t wmask[CT / 64][kSlotWords];
    if (!round_active(a, r)) return;
    const int wave = threadIdx.x >> 6;
    FOR_CELLS(k) {
        if (!a.open[k]) continue;
        const int32_t n = recount(a, k, wmask[wave]);
        if (__lane_id() == 0) {
            a.count[k] = n;
            if (n < a.n_min)
                a.open[k] = 0;
            else
                a.counters[2 + r] = 1;
        }
        const int32_t f = a.first[k], l = f + a.len[k];
        for (int32_t m = f + __lane_id(); m < l; m += 64) a.best[a.member[m]] = -1;
    }
}

constexpr int kQueueCap = 4096;  // cells recounted after one take

__global__ void __launch_bounds__(GT) k_greedy(ExtractArgs a) {
    __shared__ uint32_t wmask[GW][kSlotWords];
    __shared__ int32_t queue[kQueueCap];
    __shared__ int32_t queue_n;
    __shared__ Best wbest[GW];
    __shared__ Best best_all;
    const int tid = threadIdx.x, lane = __lane_id(), wave = tid >> 6;
    if (!lists_fit(a)) {  // nothing was extracted
        if (tid == 0) {
            a.res->n_clusters = 0;
            a.res->n_members = (int64_t)*a.n_members;
            a.res->status = SAS_EXTRACT_MEMBERS_FULL;
        }
        return;
    }
    int32_t n_out = a.counters[0];  // clusters taken by the parallel rounds
    const bool left = a.counters[2 + a.rounds] != 0;
    while (left) {
        // the maximum of the stored counts; cells below N_min close
        Best mine{0, -1, 0, 0, 0};
        for (int64_t k = tid; k < a.n_cand; k += GT) {
            if (!a.open[k]) continue;
            const int32_t cnt = a.count[k];
            if (cnt < a.n_min) {
                a.open[k] = 0;
                continue;
            }
            if (cnt < mine.count) continue;
            const sas_candidate cd = a.cand[k];
            const Best b{cnt, (int32_t)k, cd.v_idx, cd.by, cd.bx};
            if (better(b, mine)) mine = b;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const Best other = shfl_best(mine, lane ^ o);
            if (better(other, mine)) mine = other;
        }
        if (lane == 0) wbest[wave] = mine;
        __syncthreads();
        if (tid == 0) {
            Best b = wbest[0];
            for (int w = 1; w < GW; ++w)
                if (better(wbest[w], b)) b = wbest[w];
            best_all = b;
            queue_n = 0;
        }
        __syncthreads();
        const Best b = best_all;
        if (b.k < 0) break;  // block uniform
        if (tid == 0) {
            record_taken(a, n_out, b.k);
            a.open[b.k] = 0;
        }
        // take its live contributors; queue the open cells that held them
        const int32_t f = a.first[b.k], l = f + a.len[b.k];
        for (int32_t m = f + tid; m < l; m += GT) {
            const int32_t j = a.member[m];
            if (a.died[j]) continue;
            a.cluster_of[a.cat.sidx[j]] = (int32_t)n_out;
            for (int32_t i = a.inv_first[j]; i < a.inv_first[j + 1]; ++i) {
                const int32_t c = a.inv[i];
                if (c == b.k || !a.open[c]) continue;
                if (atomicExch(&a.dirty[c], 1u) == 0u) {
                    const int32_t q = atomicAdd(&queue_n, 1);
                    if (q < kQueueCap) queue[q] = c;
                }
            }
        }
        __syncthreads();  // every mark reads died before it is set
        for (int32_t m = f + tid; m < l; m += GT) a.died[a.member[m]] = 255;
        __syncthreads();
        // recount the queued cells (all open cells if the queue overflowed)
        const int32_t nq = queue_n;
        if (nq <= kQueueCap) {
            for (int32_t q = wave; q < nq; q += GW) {
                const int32_t c = queue[q];
                const int32_t n = recount(a, c, wmask[wave]);
                if (lane == 0) {
                    a.count[c] = n;
                    a.dirty[c] = 0;
                }
            }
        } else {
            for (int64_t c = wave; c < a.n_cand; c += GW) {
                if (!a.open[c]) continue;  // wave uniform
                const int32_t n = recount(a, c, wmask[wave]);
                if (lane == 0) {
                    a.count[c] = n;
                    a.dirty[c] = 0;
                }
            }
        }
        ++n_out;
        __syncthreads();
    }
    if (tid == 0) {
        a.counters[1] = n_out;
        a.res->n_clusters = n_out;
        a.res->n_members = (int64_t)*a.n_members;
        a.res->status = n_out > a.cluster_cap ? SAS_EXTRACT_CLUSTERS_FULL : 0;
    }
}

// Key of a cluster for the extraction order: (count at the take, v_idx, by,
// bx); p comes before q when its count is larger, then its v_idx, by, bx
// smaller.
__device__ inline bool key_before(const int4 &p, const int4 &q) {
    if (p.x != q.x) return p.x > q.x;
    if (p.y != q.y) return (uint32_t)p.y < (uint32_t)q.y;
    if (p.z != q.z) return p.z < q.z;
    return p.w < q.w;
}

constexpr int kRankTile = 1024;  // keys staged in LDS at a time
constexpr int kRankEach = 4;     // clusters ranked by a wave at once

// Extraction order: the rank of each cluster's key among all clusters (keys
// are distinct); the records in that order.  The keys are walked in tiles
// staged in LDS; the lanes of a wave share the keys of a tile.
__global__ void __launch_bounds__(256) k_rank(ExtractArgs a) {
    __shared__ int4 tile[kRankTile];
    if (!lists_fit(a)) return;
    const int32_t total = a.counters[1];
    const uint32_t sat = (uint32_t)a.count_sat;
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    constexpr int kBlock = kRankEach * 4;  // clusters of a workgroup
    for (int64_t c0 = (int64_t)blockIdx.x * kBlock; c0 < total; c0 += (int64_t)gridDim.x * kBlock) {
        const int64_t cw = c0 + wave * kRankEach;
        int4 mine[kRankEach];
        int32_t r[kRankEach] = {};
#pragma unroll
        for (int i = 0; i < kRankEach; ++i)
            mine[i] = a.taken[min(cw + i, (int64_t)total - 1)];
        for (int32_t d0 = 0; d0 < total; d0 += kRankTile) {
            const int32_t nd = min(kRankTile, total - d0);
            __syncthreads();
            for (int32_t i = threadIdx.x; i < nd; i += 256) tile[i] = a.taken[d0 + i];
            __syncthreads();
            for (int32_t t = lane; t < nd; t += 64) {
                const int4 q = tile[t];
#pragma unroll
                for (int i = 0; i < kRankEach; ++i) r[i] += key_before(q, mine[i]) ? 1 : 0;
            }
        }
#pragma unroll
        for (int i = 0; i < kRankEach; ++i) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) r[i] += __shfl_xor(r[i], o, 64);
            if (lane != 0 || cw + i >= total) continue;
            a.perm[cw + i] = r[i];
            if (r[i] >= a.cluster_cap) continue;
            const uint32_t cnt = (uint32_t)mine[i].x;  // its count when taken
            uint4 rec;
            rec.x = (uint32_t)mine[i].y;
            rec.y = (uint32_t)mine[i].w;
            rec.z = (uint32_t)mine[i].z;
            rec.w = (cnt > sat ? sat : cnt) | ((cnt > sat ? 1u : 0u) << 16);
            *(uint4 *)(a.clusters + r[i]) = rec;
        }
    }
}

__global__ void k_renumber(ExtractArgs a) {
    if (!lists_fit(a)) return;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += stride) {
        const int32_t c = a.cluster_of[i];
        if (c >= 0) a.cluster_of[i] = a.perm[c];
    }
}

}  // namespace

hipError_t launch_extract(const ExtractArgs &a, hipStream_t stream) {
    const unsigned init_blocks = (unsigned)std::min<int64_t>(
        (std::max(a.n + 1, a.n_cand) + 255) / 256, 4096);
    hipLaunchKernelGGL(k_extract_init, dim3(init_blocks), dim3(256), 0, stream, a);
    const unsigned cell_blocks =
        (unsigned)std::max<int64_t>(1, std::min<int64_t>((a.n_cand + CT / 64 - 1) / (CT / 64),
                                                         65536));
    if (a.n_cand > 0) {
        hipLaunchKernelGGL(k_contrib, dim3(cell_blocks), dim3(CT), 0, stream, a);
        for (int r = 1; r <= a.rounds; ++r) {
            hipLaunchKernelGGL(k_round_best, dim3(cell_blocks), dim3(CT), 0, stream, a, r);
            hipLaunchKernelGGL(k_round_take, dim3(cell_blocks), dim3(CT), 0, stream, a, r);
            hipLaunchKernelGGL(k_round_recount, dim3(cell_blocks), dim3(CT), 0, stream, a, r);
        }
        hipLaunchKernelGGL(k_inv_zero, dim3(init_blocks), dim3(256), 0, stream, a);
        hipLaunchKernelGGL(k_inv_count, dim3(2048), dim3(256), 0, stream, a);
        hipError_t e = launch_scan_exclusive(a.inv_first, a.n + 1, a.inv_blocksum, stream,
                                             a.counters + 2 + a.rounds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_inv_fill, dim3(2048), dim3(256), 0, stream, a);
    }
    hipLaunchKernelGGL(k_greedy, dim3(1), dim3(GT), 0, stream, a);
    const unsigned rank_blocks =
        (unsigned)std::max<int64_t>(1, std::min<int64_t>((a.n_cand + 15) / 16, 4096));
    hipLaunchKernelGGL(k_rank, dim3(rank_blocks), dim3(256), 0, stream, a);
    hipLaunchKernelGGL(k_renumber, dim3(init_blocks), dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace sas
