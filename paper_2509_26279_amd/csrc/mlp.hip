// Vetting MLP 32 -> 128 -> 128 -> 1 on gfx950: bf16 operands on the matrix
// cores (v_mfma_f32_16x16x32_bf16), FP32 accumulation.
//
// Forward:   a0 = q((x - mu) / sd);  h1 = q(relu(a0 q(W1) + b1));
//            h2 = q(relu(h1 q(W2) + b2));  z = h2 q(W3) + b3
// Backward:  dz = (sigmoid(z) (pw y + 1 - y) - pw y) / B;  g3 = q(dz)
//            dW3 = h2^T g3;  d2 = q((g3 q(W3)^T) [h2 > 0]);  dW2 = h1^T d2
//            d1 = q((d2 q(W2)^T) [h1 > 0]);  dW1 = a0^T d1;  db = column sums
// with q = round to bfloat16 (nearest even).  Weight gradients reduce over
// the batch in two stages (per-chunk partials, then a fixed-order sum), so
// the result is the same on every run.  AdamW keeps FP32 master weights and
// refreshes the bf16 working copies.
//
// The network is 20865 parameters: the time of a pass is launches and trips
// to memory, not products.  So a pass over the rows is one kernel that keeps
// the weights of a wave in registers and the activations in registers and
// LDS: k_mlp_forward reads x and writes logits; a training step is
// k_mlp_rows (forward, loss and backward of the rows, activations stored for
// the weight gradients), k_mlp_wgrad (all partial products and column sums)
// and k_mlp_update (fixed-order sums and AdamW).
// As 25 launches of one 64 x 64 tiled product, element-wise passes and
// reductions, a step on 4096 rows took 284 us and 2.3e5 logits 2350 us; now
// 19 us (8.8 us k_mlp_rows, 6.1 us k_mlp_wgrad, 3.3 us k_mlp_update) and
// 21 us.  A step is bound by the latency of its three launches, the logits
// by the LDS reads of the fragments and their products (30 MB of input at
// 1.4 TB/s, 0.45 PFLOP/s); results are bit for bit those of the older form.
//
// Matrix fragments.  A lane of the 16 x 16 x 32 product holds, of either
// operand, 8 consecutive k (8 (lane / 16) + j) of one row or column
// (lane % 16); of the result, rows 4 (lane / 16) + i of column lane % 16.
// The working copies of the weights and the stored activations are kept in
// fragment order ([tile][lane][8]), so that every load is 16 bytes a lane
// and contiguous over the wave.  The products over k of every output run
// in steps of 32 in ascending k.
#include <type_traits>

#include "internal.h"

namespace sas {
namespace {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
// rows of the caller's matrix: 4-byte aligned (global loads of any width are)
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));

constexpr int H = kMlpHidden;
constexpr int NT = H / 16;       // 16-column tiles of a hidden layer
constexpr int KT = H / 32;       // steps of 32 over a hidden layer
constexpr int MT = 256;          // threads: 4 waves, each 32 columns of a hidden layer
constexpr int MWAVES = MT / 64;
constexpr int LD = H + 8;        // LDS row of a hidden layer, in bf16 (16-byte multiple;
                                 // rows 4 banks apart)
constexpr int LD0 = kMlpIn + 8;  // LDS row of the inputs

__device__ inline __bf16 to_bf(float f) { return (__bf16)f; }
__device__ inline v8bf load8(const uint16_t *p) { return *(const v8bf *)p; }
__device__ inline v4f mma(v8bf a, v8bf b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Place of element (k, n) of a K x 128 matrix in fragment order.
__host__ __device__ inline int frag_index(int k, int n) {
    return (((k >> 5) * NT + (n >> 4)) * 64 + ((k & 31) >> 3) * 16 + (n & 15)) * 8 + (k & 7);
}

// Store parameter i (packed index) into the bf16 working copies.
__device__ inline void mlp_store_working(const MlpWeights &w, int i, float v) {
    const uint16_t q = __builtin_bit_cast(uint16_t, to_bf(v));
    if (i < kMlpOffB1) {
        w.w1[frag_index(i / H, i % H)] = q;
    } else if (i >= kMlpOffW2 && i < kMlpOffB2) {
        const int k = (i - kMlpOffW2) / H, n = (i - kMlpOffW2) % H;
        w.w2[frag_index(k, n)] = q;
        w.w2t[frag_index(n, k)] = q;
    } else if (i >= kMlpOffW3 && i < kMlpOffB3) {
        w.w3[i - kMlpOffW3] = q;
    }
}

// Weights of wave w: columns 32 w .. 32 w + 31 of the hidden layers, W3 whole.
struct FwdWeights {
    v8bf w1[2], w2[KT][2], w3[KT];
    float b1[2], b2[2], b3;
    __device__ FwdWeights(const MlpBuffers &b, int wave, int lane) {
        const int r16 = lane & 15, q4 = lane >> 4;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int nt = 2 * wave + t;
            w1[t] = load8(b.w.w1 + (nt * 64 + lane) * 8);
#pragma unroll
            for (int k = 0; k < KT; ++k) w2[k][t] = load8(b.w.w2 + ((k * NT + nt) * 64 + lane) * 8);
            b1[t] = b.p[kMlpOffB1 + 16 * nt + r16];
            b2[t] = b.p[kMlpOffB2 + 16 * nt + r16];
        }
        const v8bf zero = {};
#pragma unroll
        for (int k = 0; k < KT; ++k) {  // column 0 of a 16-column tile, the rest 0
            const v8bf c = load8(b.w.w3 + 32 * k + 8 * q4);
            w3[k] = r16 == 0 ? c : zero;
        }
        b3 = b.p[kMlpOffB3];
    }
};

// Standardised inputs of row m as the lane's fragment (zero past the end).
struct Norm {
    float mu[8], sd[8];
    __device__ Norm(const MlpBuffers &b, int lane) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            mu[j] = b.mu[8 * (lane >> 4) + j];
            const float s = b.sd[8 * (lane >> 4) + j];
            sd[j] = s == 0.0f ? 1.0f : s;
        }
    }
    __device__ v8bf row(const float *x, int64_t m, int64_t n, int lane) const {
        v8bf a = {};
        if (m < n) {
            const float *p = x + m * kMlpIn + 8 * (lane >> 4);
            const v4f_any u = *(const v4f_any *)p, v = *(const v4f_any *)(p + 4);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                a[j] = to_bf((u[j] - mu[j]) / sd[j]);
                a[4 + j] = to_bf((v[j] - mu[4 + j]) / sd[4 + j]);
            }
        }
        return a;
    }
};

// Hidden-layer epilogue of a 16-row tile: q(relu(acc + bias)) of the lane's
// 4 rows into LDS and back to the caller.
__device__ inline v4bf relu_store(v4f acc, float bias, __bf16 *tile, int q4, int col) {
    v4bf h;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        h[i] = to_bf(fmaxf(acc[i] + bias, 0.0f));
        tile[(4 * q4 + i) * LD + col] = h[i];
    }
    return h;
}

// Logits of rows [0, n).  A workgroup takes 16 R rows at a time; its 4 waves
// split the columns of the hidden layers.  R = 4 (large n): the weights and
// each A fragment serve 4 times the products, and each wave standardises and
// finishes one 16-row tile; R = 1 (small n): 4 times as many workgroups.
template <int R>
__global__ void __launch_bounds__(MT) k_mlp_forward(MlpBuffers b, const float *__restrict__ x,
                                                    int64_t n, float *__restrict__ out) {
    __shared__ __attribute__((aligned(16))) __bf16 a0s[16 * R * LD0];
    __shared__ __attribute__((aligned(16))) __bf16 h1s[16 * R * LD], h2s[16 * R * LD];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, q4 = lane >> 4;
    const FwdWeights w(b, wave, lane);
    const Norm norm(b, lane);
    const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
    const int64_t tiles = (n + 16 * R - 1) / (16 * R);
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int64_t m0 = t * (16 * R);
        v8bf a[R];
        if (R == 1) {  // every wave standardises the tile
            a[0] = norm.row(x, m0 + r16, n, lane);
        } else {       // wave r standardises row tile r
            *(v8bf *)(a0s + (16 * wave + r16) * LD0 + 8 * q4) =
                norm.row(x, m0 + 16 * wave + r16, n, lane);
            __syncthreads();
#pragma unroll
            for (int r = 0; r < R; ++r) a[r] = *(const v8bf *)(a0s + (16 * r + r16) * LD0 + 8 * q4);
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int c = 0; c < 2; ++c)
                relu_store(mma(a[r], w.w1[c], zero4), w.b1[c], h1s + 16 * r * LD, q4,
                           32 * wave + 16 * c + r16);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            v4f acc[2] = {zero4, zero4};
#pragma unroll
            for (int k = 0; k < KT; ++k) {
                const v8bf f = *(const v8bf *)(h1s + (16 * r + r16) * LD + 32 * k + 8 * q4);
                acc[0] = mma(f, w.w2[k][0], acc[0]);
                acc[1] = mma(f, w.w2[k][1], acc[1]);
            }
#pragma unroll
            for (int c = 0; c < 2; ++c)
                relu_store(acc[c], w.b2[c], h2s + 16 * r * LD, q4, 32 * wave + 16 * c + r16);
        }
        __syncthreads();
        if (R == MWAVES || wave == 0) {
            const int r = R == MWAVES ? wave : 0;
            v4f z = zero4;
#pragma unroll
            for (int k = 0; k < KT; ++k)
                z = mma(*(const v8bf *)(h2s + (16 * r + r16) * LD + 32 * k + 8 * q4), w.w3[k], z);
            if (r16 == 0)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int64_t m = m0 + 16 * r + 4 * q4 + i;
                    if (m < n) out[m] = z[i] + w.b3;
                }
        }
        // the next tile writes h1s (R = 4: a0s) after every wave has read it, and
        // h2s after the barrier that follows h1s
    }
}

// Offset of the lane's 4 rows of a result tile (16-row tile rt, column tile
// ct of nct) in an activation stored in fragment order over its rows:
// [row / 32][ct][(row % 32) / 8 * 16 + column][row % 8].
__device__ inline int64_t act_offset(int64_t rt, int nct, int ct, int lane) {
    const int q4 = lane >> 4;
    return ((rt >> 1) * nct + ct) * 512 +
           ((2 * (int)(rt & 1) + (q4 >> 1)) * 16 + (lane & 15)) * 8 + 4 * (q4 & 1);
}

// Forward, loss and backward of 16 rows per workgroup and pass, with the
// activations and their gradients stored for k_mlp_wgrad.  Rows past the
// batch (up to a multiple of 32) are stored as zeros.
__global__ void __launch_bounds__(MT) k_mlp_rows(MlpBuffers b, const float *__restrict__ x,
                                                 const float *__restrict__ y, int64_t B,
                                                 float pw) {
    __shared__ __attribute__((aligned(16))) __bf16 a0s[16 * LD0], h1s[16 * LD], h2s[16 * LD],
        d2s[16 * LD];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, q4 = lane >> 4;
    const FwdWeights w(b, wave, lane);
    const Norm norm(b, lane);
    v8bf w3r[2], w2t[KT][2];  // W3 as one row (k = 0), W2 transposed
    const v8bf zero8 = {};
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int nt = 2 * wave + c;
        w3r[c] = zero8;
        if (q4 == 0) w3r[c][0] = __builtin_bit_cast(__bf16, b.w.w3[16 * nt + r16]);
#pragma unroll
        for (int k = 0; k < KT; ++k) w2t[k][c] = load8(b.w.w2t + ((k * NT + nt) * 64 + lane) * 8);
    }
    const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
    const int64_t tiles = 2 * ((B + 31) / 32);
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int64_t m0 = t * 16;
        const v8bf a = norm.row(x, m0 + r16, B, lane);
        if (wave == 0) *(v8bf *)(a0s + r16 * LD0 + 8 * q4) = a;
        bool in[4];  // the lane's result rows are rows of the batch
#pragma unroll
        for (int i = 0; i < 4; ++i) in[i] = m0 + 4 * q4 + i < B;
        const __bf16 zb = to_bf(0.0f);
        v4bf h1[2], h2[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int col = 32 * wave + 16 * c + r16;
            h1[c] = relu_store(mma(a, w.w1[c], zero4), w.b1[c], h1s, q4, col);
            // no activation past the batch: its gradients are masked with it, also
            // where a zero meets an infinite weight
#pragma unroll
            for (int i = 0; i < 4; ++i) h1[c][i] = in[i] ? h1[c][i] : zb;
            *(v4bf *)(b.h1 + act_offset(t, NT, 2 * wave + c, lane)) = h1[c];
        }
        __syncthreads();
        if (wave < kMlpIn / 16) {  // the inputs by column
            v4bf s;
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = a0s[(4 * q4 + i) * LD0 + 16 * wave + r16];
            *(v4bf *)(b.a0 + act_offset(t, kMlpIn / 16, wave, lane)) = s;
        }
        v4f acc[2] = {zero4, zero4};
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            const v8bf f = *(const v8bf *)(h1s + r16 * LD + 32 * k + 8 * q4);
            acc[0] = mma(f, w.w2[k][0], acc[0]);
            acc[1] = mma(f, w.w2[k][1], acc[1]);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            h2[c] = relu_store(acc[c], w.b2[c], h2s, q4, 32 * wave + 16 * c + r16);
#pragma unroll
            for (int i = 0; i < 4; ++i) h2[c][i] = in[i] ? h2[c][i] : zb;
            *(v4bf *)(b.h2 + act_offset(t, NT, 2 * wave + c, lane)) = h2[c];
        }
        __syncthreads();
        v4f z = zero4;  // every wave: column 0 holds the logits, less b3
#pragma unroll
        for (int k = 0; k < KT; ++k)
            z = mma(*(const v8bf *)(h2s + r16 * LD + 32 * k + 8 * q4), w.w3[k], z);
        // loss and logit gradient of row r16, by every lane of the row
        float zr = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = __shfl(z[i], 16 * (r16 >> 2), 64);
            zr = (r16 & 3) == i ? v : zr;
        }
        zr += w.b3;
        const int64_t m = m0 + r16;
        __bf16 g = zb;
        if (m < B) {
            const float yi = y[m];
            const float sp_pos = fmaxf(zr, 0.0f) + log1pf(expf(-fabsf(zr)));   // softplus(z)
            const float sp_neg = fmaxf(-zr, 0.0f) + log1pf(expf(-fabsf(zr)));  // softplus(-z)
            const float sig = 1.0f / (1.0f + expf(-zr));
            g = to_bf((sig * (pw * yi + 1.0f - yi) - pw * yi) / (float)B);
            if (wave == 0 && q4 == 0) b.row_loss[m] = pw * yi * sp_neg + (1.0f - yi) * sp_pos;
        }
        if (wave == 0 && q4 == 0) b.g3[m] = __builtin_bit_cast(uint16_t, g);
        v8bf ga = zero8;
        if (q4 == 0) ga[0] = g;
        // d2 = q((g3 w3^T) [h2 > 0])
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const v4f d = mma(ga, w3r[c], zero4);
            v4bf s;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s[i] = to_bf((float)h2[c][i] > 0.0f ? d[i] : 0.0f);
                d2s[(4 * q4 + i) * LD + 32 * wave + 16 * c + r16] = s[i];
            }
            *(v4bf *)(b.d2 + act_offset(t, NT, 2 * wave + c, lane)) = s;
        }
        __syncthreads();
        // d1 = q((d2 W2^T) [h1 > 0])
        acc[0] = zero4;
        acc[1] = zero4;
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            const v8bf f = *(const v8bf *)(d2s + r16 * LD + 32 * k + 8 * q4);
            acc[0] = mma(f, w2t[k][0], acc[0]);
            acc[1] = mma(f, w2t[k][1], acc[1]);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            v4bf s;
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = to_bf((float)h1[c][i] > 0.0f ? acc[c][i] : 0.0f);
            *(v4bf *)(b.d1 + act_offset(t, NT, 2 * wave + c, lane)) = s;
        }
        // the next tile writes h1s and a0s, last read before the second barrier
        // above, and h2s and d2s after two barriers more
    }
}

// Partial weight gradients of one chunk of kMlpSplitK rows: [W1 | W2 | W3].
constexpr int kPartW2 = kMlpIn * H, kPartW3 = kPartW2 + H * H;
static_assert(kMlpPart == kPartW3 + H, "partials of W1, W2 and W3");
// Tasks of a chunk, one wave each: 16 x 32 blocks of dW2 and dW1, 32 of dW3.
constexpr int kTasksW2 = NT * (NT / 2), kTasksW1 = (kMlpIn / 16) * (NT / 2), kTasksW3 = NT / 2;
constexpr int kChunkTasks = kTasksW2 + kTasksW1 + kTasksW3;
constexpr int kSumTasks = (2 * H + 2) / 2 + 1;  // column sums, two a wave, and the loss

// f over the row blocks [rb0, rb1): blocks of kInFlight, then single ones.  A
// wave issues the loads of kInFlight row blocks before it uses the first:
// its tasks are serial chains, and the rows were written by other XCDs, so
// every load is a trip past the L2.  With the compiler's order of loads
// k_mlp_wgrad took 12.9 us on 4096 rows, now 6.1 us.
constexpr int kInFlight = 8;
template <class F>
__device__ __attribute__((always_inline)) inline void for_row_blocks(int64_t rb0, int64_t rb1,
                                                                     const F &f) {
    int64_t rb = rb0;
    for (; rb + kInFlight <= rb1; rb += kInFlight) f(std::integral_constant<int, kInFlight>{});
    for (; rb < rb1; ++rb) f(std::integral_constant<int, 1>{});
}

// Two 16 x 16 blocks A^T B of row blocks [rb0, rb1): operands in fragment order.
__device__ inline void partial_pair(const uint16_t *A, int nca, int ca, const uint16_t *Bm,
                                    int ncb, int cb, int64_t rb0, int64_t rb1, float *out, int ldo,
                                    int lane) {
    v4f acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    const uint16_t *pa = A + (rb0 * nca + ca) * 512 + lane * 8;
    const uint16_t *pb = Bm + (rb0 * ncb + cb) * 512 + lane * 8;
    for_row_blocks(rb0, rb1, [&](auto u) __attribute__((always_inline)) {
        constexpr int U = decltype(u)::value;
        v8bf fa[U], f0[U], f1[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            fa[k] = load8(pa + k * nca * 512);
            f0[k] = load8(pb + k * ncb * 512);
            f1[k] = load8(pb + k * ncb * 512 + 512);
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            acc[0] = mma(fa[k], f0[k], acc[0]);
            acc[1] = mma(fa[k], f1[k], acc[1]);
        }
        pa += U * nca * 512;
        pb += U * ncb * 512;
    });
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            out[(int64_t)(16 * ca + 4 * (lane >> 4) + i) * ldo + 16 * (cb + c) + (lane & 15)] =
                acc[c][i];
}

// Every reduction over the rows, one task a wave: the partial weight
// gradients of each chunk of kMlpSplitK rows, the column sums and the loss.
// The sums keep one fixed order: residue r of the rows modulo 256 is summed
// over its rows, then the 256 residues by a halving tree.
__global__ void __launch_bounds__(MT) k_mlp_wgrad(MlpBuffers b, int64_t B, int nz,
                                                  float *__restrict__ loss) {
    const int lane = threadIdx.x & 63;
    const int64_t task = (int64_t)blockIdx.x * MWAVES + (threadIdx.x >> 6);
    const int64_t nb = (B + 31) / 32;  // row blocks of 32
    if (task < kSumTasks) {
        if (task == kSumTasks - 1) {  // mean loss; lane: residues 4 lane + j
            float s[4] = {0.f, 0.f, 0.f, 0.f};
            const float *p = b.row_loss + 4 * lane;
            const int64_t full = max((B - 4 * lane) >> 2 << 2, (int64_t)0);  // whole quads
            const int64_t n = (full + 255) / 256;
            for_row_blocks(0, n, [&](auto uu) __attribute__((always_inline)) {
                constexpr int U = decltype(uu)::value;
                v4f v[U];
#pragma unroll
                for (int k = 0; k < U; ++k) v[k] = *(const v4f *)(p + 256 * k);
#pragma unroll
                for (int k = 0; k < U; ++k)
#pragma unroll
                    for (int j = 0; j < 4; ++j) s[j] += v[k][j];
                p += 256 * U;
            });
            for (int j = 0; j < 3; ++j)  // the rows of a last partial quad
                if (4 * lane + 256 * n + j < B) s[j] += p[j];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1)
#pragma unroll
                for (int j = 0; j < 4; ++j) s[j] += __shfl_down(s[j], o, 64);
            if (lane == 0) *loss = ((s[0] + s[2]) + (s[1] + s[3])) * (1.0f / (float)B);
            return;
        }
        // columns 2 task and 2 task + 1 of [d1 | d2 | g3]; half a wave each, lane
        // u of it: residues 8 u + j
        const int col = 2 * (int)task + (lane >> 5), u = lane & 31;
        float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (col <= 2 * H) {
            // rows r .. r + 7 of the column, then 256 rows on (8 row blocks)
            const int c = col & (H - 1);
            const uint16_t *p = b.g3 + 8 * u;
            int64_t step = 256;
            if (col < 2 * H) {
                p = (col < H ? b.d1 : b.d2) + ((int64_t)(u >> 2) * NT + (c >> 4)) * 512 +
                    ((u & 3) * 16 + (c & 15)) * 8;
                step = 8 * NT * 512;
            }
            const int64_t n = (32 * nb - 8 * u + 255) / 256;  // steps that hold rows
            for_row_blocks(0, max(n, (int64_t)0), [&](auto uu) __attribute__((always_inline)) {
                constexpr int U = decltype(uu)::value;
                v8bf v[U];
#pragma unroll
                for (int k = 0; k < U; ++k) v[k] = load8(p + k * step);
#pragma unroll
                for (int k = 0; k < U; ++k)
#pragma unroll
                    for (int j = 0; j < 8; ++j) s[j] += (float)v[k][j];
                p += U * step;
            });
        }
#pragma unroll
        for (int o = 16; o > 0; o >>= 1)
#pragma unroll
            for (int j = 0; j < 8; ++j) s[j] += __shfl_down(s[j], o, 32);
#pragma unroll
        for (int o = 4; o > 0; o >>= 1)
#pragma unroll
            for (int j = 0; j < o; ++j) s[j] += s[j + o];
        if (u == 0 && col <= 2 * H) b.bsum[col] = s[0];
        return;
    }
    const int64_t q = task - kSumTasks, z = q / kChunkTasks;
    if (z >= nz) return;
    int k = (int)(q - z * kChunkTasks);
    const int64_t rb0 = z * (kMlpSplitK / 32), rb1 = min(nb, rb0 + kMlpSplitK / 32);
    float *part = b.part + z * kMlpPart;
    if (k < kTasksW2) {
        partial_pair(b.h1, NT, k / (NT / 2), b.d2, NT, 2 * (k % (NT / 2)), rb0, rb1,
                     part + kPartW2, H, lane);
        return;
    }
    k -= kTasksW2;
    if (k < kTasksW1) {
        partial_pair(b.a0, kMlpIn / 16, k / (NT / 2), b.d1, NT, 2 * (k % (NT / 2)), rb0, rb1, part,
                     H, lane);
        return;
    }
    k -= kTasksW1;
    // dW3: two 16-row blocks of h2^T g3, in column 0
    const v8bf zero8 = {};
    v4f acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    const uint16_t *pg = b.g3 + rb0 * 32 + 8 * (lane >> 4);
    const uint16_t *ph = b.h2 + (rb0 * NT + 2 * k) * 512 + lane * 8;
    for_row_blocks(rb0, rb1, [&](auto u) __attribute__((always_inline)) {
        constexpr int U = decltype(u)::value;
        v8bf g[U], f0[U], f1[U];
#pragma unroll
        for (int r = 0; r < U; ++r) {
            g[r] = load8(pg + r * 32);
            f0[r] = load8(ph + r * NT * 512);
            f1[r] = load8(ph + r * NT * 512 + 512);
        }
#pragma unroll
        for (int r = 0; r < U; ++r) {
            const v8bf f = (lane & 15) == 0 ? g[r] : zero8;
            acc[0] = mma(f0[r], f, acc[0]);
            acc[1] = mma(f1[r], f, acc[1]);
        }
        pg += U * 32;
        ph += U * NT * 512;
    });
    if ((lane & 15) == 0)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                part[kPartW3 + 16 * (2 * k + c) + 4 * (lane >> 4) + i] = acc[c][i];
}

// Gradient of parameter i: its partials in chunk order, or its column sum.
__device__ inline float gradient_of(const MlpBuffers &b, int i, int nz) {
    if (i >= kMlpOffB1 && i < kMlpOffW2) return b.bsum[i - kMlpOffB1];
    if (i >= kMlpOffB2 && i < kMlpOffW3) return b.bsum[H + i - kMlpOffB2];
    if (i == kMlpOffB3) return b.bsum[2 * H];
    const int o = i < kMlpOffB1   ? i
                  : i < kMlpOffB2 ? kPartW2 + i - kMlpOffW2
                                  : kPartW3 + i - kMlpOffW3;
    float s = 0.0f;
#pragma unroll 8
    for (int z = 0; z < nz; ++z) s += b.part[(int64_t)z * kMlpPart + o];
    return s;
}

__global__ void k_mlp_gradient(MlpBuffers b, int nz, float *__restrict__ grad) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kMlpParams) grad[i] = gradient_of(b, i, nz);
}

// Gradient and AdamW over the packed FP32 parameters; refreshes the bf16
// working copies.
__global__ void k_mlp_update(MlpBuffers b, int nz, float lr, float b1, float b2, float eps,
                             float wd, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= kMlpParams) return;
    const float gi = gradient_of(b, i, nz);
    const float mi = b1 * b.m[i] + (1.0f - b1) * gi;
    const float vi = b2 * b.v[i] + (1.0f - b2) * gi * gi;
    b.m[i] = mi;
    b.v[i] = vi;
    const float p0 = b.p[i];
    const float pi = p0 - lr * ((mi * c1) / (sqrtf(vi * c2) + eps) + wd * p0);
    b.p[i] = pi;
    mlp_store_working(b.w, i, pi);
}

__global__ void k_refresh(MlpBuffers b) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kMlpParams) mlp_store_working(b.w, i, b.p[i]);
}

__global__ void k_mlp_copy(const float *__restrict__ from, int64_t n, float *__restrict__ to) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) to[i] = from[i];
}

inline unsigned nblk(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

constexpr int64_t kMaxRowBlocks = 2048;  // workgroups of a pass over rows (they stride)

hipError_t launch_rows(const MlpBuffers &b, const float *x, const float *y, int64_t B, float pw,
                       float *loss, hipStream_t s) {
    const unsigned grid = (unsigned)min((int64_t)nblk(B, 32) * 2, kMaxRowBlocks);
    hipLaunchKernelGGL(k_mlp_rows, dim3(grid), dim3(MT), 0, s, b, x, y, B, pw);
    const int nz = (int)nblk(B, kMlpSplitK);
    hipLaunchKernelGGL(k_mlp_wgrad, dim3(nblk((int64_t)nz * kChunkTasks + kSumTasks, MWAVES)),
                       dim3(MT), 0, s, b, B, nz, loss);
    return hipGetLastError();
}

}  // namespace

hipError_t mlp_logits(const MlpBuffers &b, const float *x, int64_t n, float *out, hipStream_t s) {
    // 64-row workgroups once there is one for every CU: up to 3e4 rows either
    // form takes the 8.7 us of a launch; 65536 rows 8.8 us against 15.9 us,
    // 2.3e5 rows 21 us against 46 us
    if (n >= 64 * 256)
        hipLaunchKernelGGL(k_mlp_forward<4>, dim3((unsigned)min((int64_t)(n + 63) / 64, (int64_t)768)),
                           dim3(MT), 0, s, b, x, n, out);
    else
        hipLaunchKernelGGL(k_mlp_forward<1>, dim3(nblk(n, 16)), dim3(MT), 0, s, b, x, n, out);
    return hipGetLastError();
}

hipError_t mlp_copy(const float *from, int64_t n, float *to, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_copy, dim3(nblk(n, 256)), dim3(256), 0, s, from, n, to);
    return hipGetLastError();
}

// Loss (mean) and gradient (packed like the parameters) of a batch of B rows.
hipError_t mlp_grad(const MlpBuffers &b, const float *x, const float *y, int64_t B, float pw,
                    float *loss, float *grad, hipStream_t s) {
    hipError_t e = launch_rows(b, x, y, B, pw, loss, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mlp_gradient, dim3(nblk(kMlpParams, 256)), dim3(256), 0, s, b,
                       (int)nblk(B, kMlpSplitK), grad);
    return hipGetLastError();
}

hipError_t mlp_step(const MlpBuffers &b, const float *x, const float *y, int64_t B, float pw,
                    float *loss, float lr, float b1, float b2, float eps, float wd, float c1,
                    float c2, hipStream_t s) {
    hipError_t e = launch_rows(b, x, y, B, pw, loss, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mlp_update, dim3(nblk(kMlpParams, 256)), dim3(256), 0, s, b,
                       (int)nblk(B, kMlpSplitK), lr, b1, b2, eps, wd, c1, c2);
    return hipGetLastError();
}

hipError_t mlp_refresh(const MlpBuffers &b, hipStream_t s) {
    hipLaunchKernelGGL(k_refresh, dim3(nblk(kMlpParams, 256)), dim3(256), 0, s, b);
    return hipGetLastError();
}

}  // namespace sas
