// The learned l(t) surrogate of lbcap: an MLP 19 -> 256 -> 256 -> 256 -> 64
// with GELU activations, trained by mean-squared error and Adam, all on the
// device in FP32.
//
// Two kernels (and mlp_row, a forward pass of few rows).  mlp_rows takes a few rows through all four layers (and, for the
// gradient, back again): the activations of the rows stay in LDS and registers,
// the weights stream through once per direction.  mlp_wgrad forms every weight
// and bias gradient from the activations and output gradients that mlp_rows left
// and, in training, applies Adam to them at once.  So a forward pass is one
// launch and a training step two.
//
// Every product runs on FP32 matrix instructions whose accumulation is a chain of
// fused multiply-adds in the order of k, one rounding each (v_mfma_f32_4x4x1 and
// 16x16x4 alike), so the results do not depend on how rows are tiled.  Reductions
// (bias gradients, the loss) are sequential per output element or a fixed tree:
// a training run is bitwise reproducible.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "lbcap.h"
#include "lb_barrier.h"
#include "lb_internal.h"

namespace {

constexpr int NLAYER = 4;
constexpr int DIMS[NLAYER + 1] = {19, 256, 256, 256, 64};
constexpr int WMAX = 256;               // widest layer

typedef float f4 __attribute__((ext_vector_type(4)));

// Packed copies of the weights, kept in step with the parameters: what a lane of
// mlp_rows multiplies next lies in one 16-byte word, 1 KB per wavefront load.
//   forward   Wf[l][c / 64][k / 4][c % 64][k % 4] = W_l[c][k]   (c: output, k: input)
//   backward  Wb[l][c / 64][k / 4][c % 64][k % 4] = W_l[k][c]   (c: input, k: output; l >= 1)
// The first layer's 19 inputs are padded to 32 with zeros.
constexpr int KPAD[NLAYER] = {32, 256, 256, 256};
constexpr int WF_OFF[NLAYER + 1] = {0, 8192, 8192 + 65536, 8192 + 2 * 65536, 8192 + 2 * 65536 + 16384};
constexpr int WB_OFF[NLAYER + 1] = {0, 0, 65536, 2 * 65536, 2 * 65536 + 16384};
constexpr int PACKED = WF_OFF[NLAYER] + WB_OFF[NLAYER];

__host__ __device__ constexpr int w_off(int l) {
    int n = 0;
    for (int i = 0; i < l; ++i) n += DIMS[i + 1] * DIMS[i] + DIMS[i + 1];
    return n;
}
__host__ __device__ constexpr int b_off(int l) { return w_off(l) + DIMS[l + 1] * DIMS[l]; }

// gelu(z) and its derivative from e1 = 1 + erf(z / sqrt(2)).
__device__ __forceinline__ float gelu_e1(float z) { return 1.f + erff(z * 0.70710678118654752f); }
__device__ __forceinline__ float gelu(float z, float e1) { return 0.5f * z * e1; }
__device__ __forceinline__ float gelu_grad(float z, float e1) {
    return 0.5f * e1 + z * 0.39894228040143268f * expf(-0.5f * z * z);
}

// Weight (o, i) of layer l into its packed places.
__device__ __forceinline__ void pack_weight(float* packed, int l, int o, int i, float w) {
    packed[WF_OFF[l] + (((o >> 6) * (KPAD[l] >> 2) + (i >> 2)) * 64 + (o & 63)) * 4 + (i & 3)] = w;
    if (l > 0)
        packed[WF_OFF[NLAYER] + WB_OFF[l] + (((i >> 6) * (DIMS[l + 1] >> 2) + (o >> 2)) * 64 + (i & 63)) * 4 +
               (o & 3)] = w;
}

__global__ void __launch_bounds__(256) mlp_pack(const float* __restrict__ P, float* __restrict__ packed) {
    const int e = blockIdx.x * 256 + threadIdx.x;
#pragma unroll
    for (int l = 0; l < NLAYER; ++l) {
        const int k = e - w_off(l);
        if (k >= 0 && k < DIMS[l + 1] * DIMS[l]) pack_weight(packed, l, k / DIMS[l], k % DIMS[l], P[e]);
    }
}

// What mlp_rows leaves for mlp_wgrad, in the order in which that kernel's lanes
// multiply: rows in groups of 16, columns in tiles of 16, and per group and tile
// [row % 4][column % 16][row / 4 % 4].  Rows past the last one of the pass up to a
// multiple of 16 are zero.
__device__ __forceinline__ long grad_at(int ntile, int group, int tile, int r4, int c) {
    return ((long)(group * ntile + tile) * 64 + r4 * 16 + c) * 4;
}

struct RowsArgs {
    const float* P;         // parameters (the biases are read)
    const float* packed;
    const float* X;         // n x 19
    const int* idx;         // rows of X and Y that the pass takes, null: 0 .. n-1
    int n;
    float* out;             // n x 64, or null
    // gradient pass only
    const float* Y;         // n x 64 targets
    float inv;              // 1 / (64 n)
    float* act[NLAYER];     // layer inputs, packed (grad_at)
    float* dz[NLAYER];      // gradients of the pre-activations, packed
    float* loss;            // sum of squared errors, one per workgroup
};

// (the weights requested ahead stay in flight over it, and nothing that a kernel of
// this file stores is read by the same kernel)
using lbk::lds_barrier;

// The stream of weights of one wavefront: chunks of 16 k x 64 columns, four 16-byte
// words per lane, through the four layers and (gradient) back through the last
// three.  Chunk g is requested AHEAD chunks before it is multiplied, across layers:
// with one or two wavefronts per SIMD it has to cover the L2's latency by itself
// (about 1000 cycles; a chunk's arithmetic takes 128 MT, or 256 for MT = 1, whose
// single chain of products waits for itself).  Left to the compiler, one chunk
// ahead: 2.5 times as long.
constexpr int CHUNK0[8] = {0, 2, 18, 34, 50, 54, 70, 86};   // first chunk of each product
template <bool GRAD, int AHEAD>
struct Stream {
    static constexpr int RING = AHEAD + 1;
    const f4* base[GRAD ? 7 : 4];
    f4 w[RING][4];
    __device__ __forceinline__ void init(const float* packed, int wv, int lane) {
#pragma unroll
        for (int l = 0; l < NLAYER; ++l)   // (the 64 outputs are one tile)
            base[l] = (const f4*)(packed + WF_OFF[l]) + (l < NLAYER - 1 ? wv * (KPAD[l] >> 2) * 64 : 0) + lane;
        if constexpr (GRAD) {
#pragma unroll
            for (int l = NLAYER - 1; l > 0; --l)
                base[NLAYER + (NLAYER - 1 - l)] =
                    (const f4*)(packed + WF_OFF[NLAYER] + WB_OFF[l]) + wv * (DIMS[l + 1] >> 2) * 64 + lane;
        }
#pragma unroll
        for (int g = 0; g < AHEAD; ++g) request(g);
    }
    // (g is a constant wherever this is called)
    __device__ __forceinline__ void request(int g) {
        constexpr int NP = GRAD ? 7 : 4;
#pragma unroll
        for (int p = 0; p < NP; ++p)
            if (g >= CHUNK0[p] && g < CHUNK0[p + 1]) {
#pragma unroll
                for (int q = 0; q < 4; ++q) w[g % RING][q] = base[p][((g - CHUNK0[p]) * 4 + q) * 64];
            }
    }
};

// acc[m][v] += sum over k of H(4 m + v, k) W(column of the lane, k), in the order of k:
// product P of the stream.  Hs: [m][k][4 rows] in LDS, WMAX k apart.  The 4x4x1
// instruction works on 16 blocks of 4 rows x 4 columns; with the first operand
// broadcast from block k % 16, one LDS word per lane holds 4 rows of 16 k.
template <int MT, int P, bool GRAD, int AHEAD>
__device__ __forceinline__ void rows_product(Stream<GRAD, AHEAD>& s, const float* Hs, int lane, f4 (&acc)[MT]) {
    constexpr int NC = CHUNK0[P + 1] - CHUNK0[P];
    float a[2][MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) a[0][m] = Hs[m * WMAX * 4 + lane];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int g = CHUNK0[P] + c;
        s.request(g + AHEAD);
        if (c + 1 < NC) {
#pragma unroll
            for (int m = 0; m < MT; ++m) a[(c + 1) & 1][m] = Hs[(m * WMAX + (c + 1) * 16) * 4 + lane];
        }
        // (the requests stay ahead of the arithmetic)
        __builtin_amdgcn_sched_barrier(0);
#define MLP_STEP(k)                                                                                       \
    _Pragma("unroll") for (int m = 0; m < MT; ++m) acc[m] =                                               \
        __builtin_amdgcn_mfma_f32_4x4x1f32(a[c & 1][m], s.w[g % (AHEAD + 1)][(k) / 4][(k) % 4], acc[m], 4, k, 0);
        MLP_STEP(0) MLP_STEP(1) MLP_STEP(2) MLP_STEP(3) MLP_STEP(4) MLP_STEP(5) MLP_STEP(6) MLP_STEP(7)
        MLP_STEP(8) MLP_STEP(9) MLP_STEP(10) MLP_STEP(11) MLP_STEP(12) MLP_STEP(13) MLP_STEP(14) MLP_STEP(15)
#undef MLP_STEP
        __builtin_amdgcn_sched_barrier(0);
    }
}

// 4 MT rows through the network: four wavefronts, each 64 of the 256 columns of a
// hidden layer (the 64 outputs: one wavefront per 4 rows).  GRAD: and back again.
// Bound by the chain of products per column (787 forward, 1363 with the gradient) and
// the weights' way through the CU (0.6 and 1.2 MB per workgroup), both about 10 us a
// gradient pass; the activation functions add a third.  A training step of 512 rows takes
// 28 us (22 launches took 860), the gradient of 3675 rows 63 us (5800).
template <int MT, bool GRAD>
__global__ void __launch_bounds__(256, GRAD && MT == 2 ? 2 : 1) mlp_rows(RowsArgs a) {
    constexpr int R = 4 * MT;
    __shared__ float Hb[2][MT * WMAX * 4];   // activations of the rows, [m][k][4 rows], two layers in turn
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6), col = t;
    const int r0 = blockIdx.x * R;
    // group of 16 rows and this workgroup's first fours of it, for the packed outputs
    const int group = r0 >> 4, f0 = (r0 & 15) >> 2;
    auto row_of = [&](int r) { return a.idx ? a.idx[r] : r; };
    // the rows of X, zero past the last row and the last input (before the weights, or
    // they wait for all of those requested ahead)
    constexpr int XN = (R * 32 + 255) / 256;
    float xv[XN];
#pragma unroll
    for (int j = 0; j < XN; ++j) {
        const int e = t + 256 * j, r = e >> 5, k = e & 31;
        xv[j] = (r < R && k < DIMS[0] && r0 + r < a.n) ? a.X[(long)row_of(r0 + r) * DIMS[0] + k] : 0.f;
    }
    Stream<GRAD, GRAD && MT == 2 ? 4 : 7> ws;
    ws.init(a.packed, wv, lane);
#pragma unroll
    for (int j = 0; j < XN; ++j) {
        const int e = t + 256 * j, r = e >> 5, k = e & 31;
        if (r < R) {
            Hb[0][((r >> 2) * WMAX + k) * 4 + (r & 3)] = xv[j];
            if (GRAD) a.act[0][grad_at(2, group, k >> 4, r & 3, k & 15) + f0 + (r >> 2)] = xv[j];
        }
    }
    lds_barrier();

    // values of the lane's column and the workgroup's rows to a packed matrix of ntile tiles
    auto put = [&](float* dst, int ntile, int c, const f4 (&v)[MT]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float* p = dst + grad_at(ntile, group, c >> 4, r, c & 15) + f0;
#pragma unroll
            for (int m = 0; m < MT; ++m) p[m] = v[m][r];
        }
    };
    f4 gp[GRAD ? NLAYER - 1 : 1][MT];   // gelu' of the hidden pre-activations
    int cur = 0;
#pragma unroll
    for (int l = 0; l < NLAYER - 1; ++l) {
        f4 acc[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m] = f4{0.f, 0.f, 0.f, 0.f};
        const float bias = a.P[b_off(l) + col];
        if (l == 0)
            rows_product<MT, 0>(ws, Hb[cur], lane, acc);
        else if (l == 1)
            rows_product<MT, 1>(ws, Hb[cur], lane, acc);
        else
            rows_product<MT, 2>(ws, Hb[cur], lane, acc);
        f4 h[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float z = acc[m][v] + bias;
                const float e1 = gelu_e1(z);
                h[m][v] = gelu(z, e1);
                if (GRAD) {
                    // a row past the last one ends here, or its biases alone could take it
                    // to an infinity, which times its zero gradient is no zero
                    const bool row = r0 + 4 * m + v < a.n;
                    h[m][v] = row ? h[m][v] : 0.f;
                    gp[l][m][v] = row ? gelu_grad(z, e1) : 0.f;
                }
            }
            *(f4*)&Hb[cur ^ 1][(m * WMAX + col) * 4] = h[m];
        }
        if (GRAD) put(a.act[l + 1], 16, col, h);
        lds_barrier();
        cur ^= 1;
    }
    // outputs, 64 columns: wavefront w takes the four rows w % MT (with fewer fours than
    // wavefronts the others do the same work and leave no result)
    float se = 0.f;
    {
        constexpr int L3 = NLAYER - 1;
        const int m = wv % MT;
        f4 acc[1] = {f4{0.f, 0.f, 0.f, 0.f}};
        const float bias = a.P[b_off(L3) + lane];
        float y[4] = {0.f, 0.f, 0.f, 0.f};
        if (GRAD) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = r0 + 4 * m + v;
                if (r < a.n) y[v] = a.Y[(long)row_of(r) * DIMS[NLAYER] + lane];
            }
        }
        rows_product<1, 3>(ws, &Hb[cur][m * WMAX * 4], lane, acc);
        if (wv < MT) {
            f4 dz;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = r0 + 4 * m + v;
                const float o = acc[0][v] + bias;
                if (a.out && r < a.n) a.out[(long)r * DIMS[NLAYER] + lane] = o;
                if (GRAD) {
                    const float d = r < a.n ? o - y[v] : 0.f;
                    dz[v] = 2.f * d * a.inv;
                    se += d * d;
                    a.dz[L3][grad_at(4, group, lane >> 4, v, lane & 15) + f0 + m] = dz[v];
                }
            }
            if (GRAD) *(f4*)&Hb[cur ^ 1][(m * WMAX + lane) * 4] = dz;
        }
    }
    if constexpr (GRAD) {
        // squared errors: a fixed tree over the lanes, then the wavefronts in order
        __shared__ float red[4];
        for (int s = 32; s > 0; s >>= 1) se += __shfl_down(se, s);
        if (lane == 0) red[wv] = se;
        lds_barrier();
        if (t == 0) a.loss[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
        cur ^= 1;
#pragma unroll
        for (int l = NLAYER - 1; l > 0; --l) {
            // d act = dz W, times gelu' of the layer below
            f4 acc[MT];
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m] = f4{0.f, 0.f, 0.f, 0.f};
            if (l == 3)
                rows_product<MT, 4>(ws, Hb[cur], lane, acc);
            else if (l == 2)
                rows_product<MT, 5>(ws, Hb[cur], lane, acc);
            else
                rows_product<MT, 6>(ws, Hb[cur], lane, acc);
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                acc[m] *= gp[l - 1][m];
                if (l > 1) *(f4*)&Hb[cur ^ 1][(m * WMAX + col) * 4] = acc[m];
            }
            put(a.dz[l - 1], 16, col, acc);
            if (l > 1) lds_barrier();
            cur ^= 1;
        }
    }
}

// acc = sum over k of h[k] W(column of the lane, k), in the order of k: product P of the
// stream for one row h in LDS, by vector FMAs.
template <int P, int AHEAD>
__device__ __forceinline__ float row_product(Stream<false, AHEAD>& s, const float* h) {
    constexpr int NC = CHUNK0[P + 1] - CHUNK0[P];
    float acc = 0.f;
    f4 a[2][4];
    auto read = [&](f4 (&to)[4], int c) {
        int at = 16 * c;
        asm volatile("" : "+v"(at));   // (or the reads of all chunks come first)
#pragma unroll
        for (int q = 0; q < 4; ++q) to[q] = *(const f4*)&h[at + 4 * q];
    };
    read(a[0], 0);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int g = CHUNK0[P] + c;
        s.request(g + AHEAD);
        if (c + 1 < NC) read(a[(c + 1) & 1], c + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 16; ++k)
            acc = __builtin_fmaf(a[c & 1][k / 4][k % 4], s.w[g % (AHEAD + 1)][k / 4][k % 4], acc);
        asm volatile("" : "+v"(acc));   // (or the sums come after all requests)
        __builtin_amdgcn_sched_barrier(0);
    }
    return acc;
}

// The forward pass with one row per workgroup, as long as every row has a CU.  The
// matrix instruction takes four rows at a time, 16 cycles a link of the chain of
// products; a vector FMA takes 4, with the same sums (one rounding per product, in the
// order of k), and each lane has one activation to evaluate instead of four.  What is
// left is the weights' way into the CU (0.6 MB at 64 bytes a cycle, 4 us).  One row
// 8.3 -> 7.3 us a call, 256 rows 8.8 -> 8.0, 300 rows (two rounds) 8.8 -> 13.3; the
// gradient pass gains nothing (256 rows 102 us either way).
__global__ void __launch_bounds__(256, 1) mlp_row(RowsArgs a) {
    __shared__ float H[2][WMAX];   // activations, two layers in turn
    const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
    // (the row before the weights, as in mlp_rows)
    const float xv = t < DIMS[0] ? a.X[(long)blockIdx.x * DIMS[0] + t] : 0.f;
    Stream<false, 7> ws;
    ws.init(a.packed, wv, lane);
    if (t < KPAD[0]) H[0][t] = xv;
    lds_barrier();
#pragma unroll
    for (int l = 0; l < NLAYER - 1; ++l) {
        const float bias = a.P[b_off(l) + t];
        const float* h = H[l & 1];
        const float z =
            (l == 0 ? row_product<0>(ws, h) : l == 1 ? row_product<1>(ws, h) : row_product<2>(ws, h)) + bias;
        H[(l & 1) ^ 1][t] = gelu(z, gelu_e1(z));
        lds_barrier();
    }
    // the 64 outputs: every wavefront does the same work, the first one keeps the result
    const float bias = a.P[b_off(NLAYER - 1) + lane];
    const float o = row_product<3>(ws, H[(NLAYER - 1) & 1]) + bias;
    if (wv == 0) a.out[(long)blockIdx.x * DIMS[NLAYER] + lane] = o;
}

// Adam (Kingma & Ba 2015, Algorithm 1); bc1 = 1 - beta1^t, bc2 = 1 - beta2^t.
struct AdamArgs {
    float *P, *m, *v, *packed;
    float lr, b1, b2, eps, bc1, bc2;
};

// One parameter: its value and moments before the step, and the gradient.  (Written
// as fused operations, so that the trained weights do not depend on which products
// a compiler contracts.)
struct AdamState {
    float p, m, v;
};
__device__ __forceinline__ AdamState adam_state(const AdamArgs& a, int i) { return AdamState{a.P[i], a.m[i], a.v[i]}; }
__device__ __forceinline__ float adam(const AdamArgs& a, int i, const AdamState& s, float gi) {
    const float mi = __builtin_fmaf(1.f - a.b1, gi, a.b1 * s.m);
    const float vi = __builtin_fmaf(gi, (1.f - a.b2) * gi, a.b2 * s.v);
    a.m[i] = mi;
    a.v[i] = vi;
    const float p = s.p - a.lr * (mi / a.bc1) / (sqrtf(vi / a.bc2) + a.eps);
    a.P[i] = p;
    return p;
}

struct WgradArgs {
    const float* act[NLAYER];
    const float* dz[NLAYER];
    int groups;             // groups of 16 rows
    const float* part;      // squared errors of the workgroups of mlp_rows
    int nparts;
    float inv;
    float* loss;
    float* G;               // gradients (null in training)
    AdamArgs adam;
};

constexpr int WG_TILES[NLAYER] = {8, 64, 64, 16};   // 32 x 32 tiles of weight gradients per layer
constexpr int WG_WEIGHTS = 8 + 64 + 64 + 16;
constexpr int WG_BIAS = (3 * 16 + 4) / 4;           // workgroups of the bias gradients
constexpr int WG_GRID = WG_WEIGHTS + WG_BIAS + 1;   // and one for the loss

// Sum over the rows of A(row, o) B(row, i) of one 16 x 16 tile, rows in order; ONES: of
// A(row, o).  16 groups of rows are requested ahead: one wavefront per SIMD, and what
// mlp_rows wrote comes from beyond the L2 for most of the XCDs.
template <bool ONES>
__device__ __forceinline__ f4 wgrad_sum(const f4* __restrict__ A, int sa, const f4* __restrict__ B, int sb,
                                        int groups) {
    constexpr int DEPTH = 16;
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    f4 x[DEPTH], y[DEPTH];
    auto request = [&](int d, int g) {
        const int gg = min(g, groups - 1);   // (past the end: a repeat, unused)
        x[d] = A[(long)gg * sa];
        if (!ONES) y[d] = B[(long)gg * sb];
    };
    auto add = [&](int d) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[d][q], ONES ? 1.f : y[d][q], acc, 0, 0, 0);
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) request(d, d);
    int g = 0;
    for (; g + DEPTH <= groups; g += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            add(d);
            request(d, g + DEPTH + d);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        if (g + d < groups) add(d);
    return acc;
}

// Gradient of one 16 x 16 tile of dW[o][i] = sum over the rows of dz[r][o] act[r][i] per
// wavefront, rows in order; the bias gradients are the same sums against ones.
// A chain of 8 cycles a row per tile, and no more than 660 tiles: bound by that chain.
// TRAIN: Adam on the finished gradients.
template <bool TRAIN>
__global__ void __launch_bounds__(256) mlp_wgrad(WgradArgs a) {
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int b = blockIdx.x, l, ot, it = 0, ni = 0;
    bool bias = false;
    if (b >= WG_WEIGHTS + WG_BIAS) {   // the loss
        float s = 0.f;
        __shared__ float red[256];
        for (int e = threadIdx.x; e < a.nparts; e += 256) s += a.part[e];
        red[threadIdx.x] = s;
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
            __syncthreads();
        }
        if (threadIdx.x == 0) *a.loss = red[0] * a.inv;
        return;
    }
    if (b >= WG_WEIGHTS) {
        bias = true;
        const int k = (b - WG_WEIGHTS) * 4 + wv;
        l = k >> 4;
        ot = k & 15;
    } else {
        l = 0;
#pragma unroll
        for (int q = 0; q < NLAYER - 1; ++q)
            if (l == q && b >= WG_TILES[q]) {
                b -= WG_TILES[q];
                l = q + 1;
            }
        ni = l == 0 ? 2 : 16;               // tiles of 16 inputs
        const int bi = ni >> 1;
        ot = (b / bi) * 2 + (wv >> 1);
        it = (b % bi) * 2 + (wv & 1);
    }
    const int no = l == NLAYER - 1 ? 4 : 16;
    // 16 x 16 result tile: lane holds rows 4 (lane / 16) + v, column lane % 16; a bias
    // gradient is in every column
    const int in = DIMS[l], i = it * 16 + (lane & 15), o0 = ot * 16 + 4 * (lane >> 4);
    const bool mine = bias ? (lane & 15) == 0 : i < in;
    const int e0 = bias ? b_off(l) + o0 : w_off(l) + o0 * in + i, es = bias ? 1 : in;
    AdamState state[4];
    if (TRAIN && mine) {   // (before the sums, which cover the latency)
#pragma unroll
        for (int v = 0; v < 4; ++v) state[v] = adam_state(a.adam, e0 + v * es);
    }
    const f4* A = (const f4*)a.dz[l] + ot * 64 + lane;
    const int sa = no * 64;
    f4 acc;
    if (bias)
        acc = wgrad_sum<true>(A, sa, A, sa, a.groups);
    else
        acc = wgrad_sum<false>(A, sa, (const f4*)a.act[l] + it * 64 + lane, ni * 64, a.groups);
    if (!mine) return;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int e = e0 + v * es;
        if (TRAIN) {
            const float p = adam(a.adam, e, state[v], acc[v]);
            if (!bias) pack_weight(a.adam.packed, l, o0 + v, i, p);
        } else {
            a.G[e] = acc[v];
        }
    }
}

// ---- host side -----------------------------------------------------------------

long param_count() { return w_off(NLAYER); }

uint64_t splitmix64(uint64_t x) {
    x += 0x9E3779B97F4A7C15ull;
    x = (x ^ (x >> 30)) * 0xBF58476D1CE4E5B9ull;
    x = (x ^ (x >> 27)) * 0x94D049BB133111EBull;
    return x ^ (x >> 31);
}

double uniform01(uint64_t seed, uint64_t i) {
    return (double)(splitmix64(seed * 0x100000001B3ull + i) >> 11) * (1.0 / 9007199254740992.0);
}

#define MLP_TRY(call)                                                                          \
    do {                                                                                       \
        hipError_t e_ = (call);                                                                \
        if (e_ != hipSuccess)                                                                  \
            return lbk::set_error(LB_EDEVICE, (std::string(#call) + ": " + hipGetErrorString(e_)).c_str()); \
    } while (0)

}  // namespace

// Rows that mlp_predict passes through pinned memory, which the kernel reads and writes
// itself (507 rows: 29 us, with copies to and from pageable memory 45).
constexpr int PIN_ROWS = 1024;
static_assert(sizeof(float) * PIN_ROWS * (DIMS[0] + DIMS[NLAYER]) <= lbk::PIN_BYTES, "rows fit");

struct mlp_net {
    int device = -1;           // the GPU the parameters live on
    hipStream_t stream = nullptr;
    float* P = nullptr;        // parameters, mlp_get_params layout
    float* packed = nullptr;   // the weights as mlp_rows reads them
    float* G = nullptr;        // gradients, mlp_get_params layout
    float* Mo = nullptr;       // Adam first moments
    float* Vo = nullptr;       // Adam second moments
    float* pin = nullptr;      // pinned host memory, PIN_ROWS rows of inputs and outputs (pin_take)
    float* xcopy = nullptr;    // MLP_NOALLOC_MAX_ROWS rows of X (see mlp_predict_device_noalloc)
    long adam_t = 0;           // Adam steps taken
    int cap = 0;               // rows that x and y hold
    float* x = nullptr;        // inputs, cap x 19
    float* y = nullptr;        // outputs or targets, cap x 64
    int gcap = 0;              // groups of 16 rows that the packed matrices hold
    float* act[NLAYER] = {};   // layer inputs, packed
    float* dz[NLAYER] = {};    // gradients of the pre-activations, packed
    float* part = nullptr;     // squared errors per workgroup of mlp_rows
    float* loss = nullptr;     // device scalars, one per minibatch
    int loss_cap = 0;
    float* Xall = nullptr;     // training set on the device
    float* Yall = nullptr;
    int* idx = nullptr;
    long data_cap = 0;
};

namespace {

void free_rows(mlp_net* n) {
    (void)hipFree(n->x);
    (void)hipFree(n->y);
    n->x = n->y = nullptr;
    n->cap = 0;
}

void free_groups(mlp_net* n) {
    for (int l = 0; l < NLAYER; ++l) {
        (void)hipFree(n->act[l]);
        (void)hipFree(n->dz[l]);
        n->act[l] = n->dz[l] = nullptr;
    }
    (void)hipFree(n->part);
    n->part = nullptr;
    n->gcap = 0;
}

lb_status ensure_rows(mlp_net* n, int rows) {
    if (rows <= n->cap) return LB_OK;
    MLP_TRY(hipStreamSynchronize(n->stream));
    free_rows(n);
    MLP_TRY(hipMalloc(&n->x, sizeof(float) * (size_t)rows * DIMS[0]));
    MLP_TRY(hipMalloc(&n->y, sizeof(float) * (size_t)rows * DIMS[NLAYER]));
    n->cap = rows;
    return LB_OK;
}

// Packed matrices of a gradient pass over `rows` rows.
lb_status ensure_groups(mlp_net* n, int rows) {
    const int groups = rows / 16 + (rows % 16 != 0);
    if (groups <= n->gcap) return LB_OK;
    MLP_TRY(hipStreamSynchronize(n->stream));
    free_groups(n);
    for (int l = 0; l < NLAYER; ++l) {
        MLP_TRY(hipMalloc(&n->act[l], sizeof(float) * 16 * (size_t)groups * KPAD[l]));
        MLP_TRY(hipMalloc(&n->dz[l], sizeof(float) * 16 * (size_t)groups * DIMS[l + 1]));
    }
    MLP_TRY(hipMalloc(&n->part, sizeof(float) * 4 * (size_t)groups));
    n->gcap = groups;
    return LB_OK;
}

template <int MT, bool GRAD>
void launch_rows(const mlp_net* net, const RowsArgs& a, int work) {
    hipLaunchKernelGGL((mlp_rows<MT, GRAD>), dim3(work), dim3(256), 0, net->stream, a);
}

// Forward pass of n rows of X into out.  One row per workgroup while there is a CU for
// each (mlp_row).  Rows per workgroup beyond: 4 are the matrix instruction's least and
// leave every product a single chain (10 us, of which 4 are the launch's), 8 run two
// chains in the same time per workgroup, 16 share each weight among most rows.  Measured, us, with 4 / 8 / 16 rows: 17.7 / 13.6 / 19.6 at
// 1100 rows, 19.4 / 14.4 / 19.3 at 2048, 35.2 / 23.4 / 21.2 at 4096, 128 / 80 / 66 at
// 16384 (four products as launches of their own: 22 us each at 507 rows).
lb_status forward(const mlp_net* net, const float* X, int n, float* out) {
    RowsArgs a{};
    a.P = net->P;
    a.packed = net->packed;
    a.X = X;
    a.n = n;
    a.out = out;
    if (n <= 256)
        hipLaunchKernelGGL(mlp_row, dim3(n), dim3(256), 0, net->stream, a);
    else if (n <= 1024)
        launch_rows<1, false>(net, a, (n + 3) / 4);
    else if (n <= 2048)
        launch_rows<2, false>(net, a, (n + 7) / 8);
    else
        launch_rows<4, false>(net, a, n / 16 + (n % 16 != 0));
    MLP_TRY(hipGetLastError());
    return LB_OK;
}

// Loss and gradient of n rows (idx: those rows of X and Y); train: and one Adam
// step with its result, else the gradient into G.
lb_status gradient(mlp_net* net, const float* X, const float* Y, const int* idx, int n, float* loss, bool train,
                   float lr) {
    RowsArgs a{};
    a.P = net->P;
    a.packed = net->packed;
    a.X = X;
    a.Y = Y;
    a.idx = idx;
    a.n = n;
    a.inv = 1.f / (float)((long)n * DIMS[NLAYER]);
    WgradArgs w{};
    for (int l = 0; l < NLAYER; ++l) {
        w.act[l] = a.act[l] = net->act[l];
        w.dz[l] = a.dz[l] = net->dz[l];
    }
    a.loss = net->part;
    w.groups = n / 16 + (n % 16 != 0);
    w.part = net->part;
    w.inv = a.inv;
    w.loss = loss;
    // Whole groups of 16 rows, as the packed matrices.  4 rows per workgroup while they
    // leave CUs idle (512 rows: 19.6 against 20.3 us), else 8, two workgroups per CU
    // (3675 rows: 39.7 us; 64 with 4 rows, 39.9 with 16).
    if (n <= 1024) {
        w.nparts = 4 * w.groups;
        launch_rows<1, true>(net, a, w.nparts);
    } else {
        w.nparts = 2 * w.groups;
        launch_rows<2, true>(net, a, w.nparts);
    }
    MLP_TRY(hipGetLastError());
    if (train) {
        net->adam_t += 1;
        const float bc1 = 1.f - (float)std::pow(0.9, (double)net->adam_t);
        const float bc2 = 1.f - (float)std::pow(0.999, (double)net->adam_t);
        w.adam = AdamArgs{net->P, net->Mo, net->Vo, net->packed, lr, 0.9f, 0.999f, 1e-8f, bc1, bc2};
        hipLaunchKernelGGL(mlp_wgrad<true>, dim3(WG_GRID), dim3(256), 0, net->stream, w);
    } else {
        w.G = net->G;
        hipLaunchKernelGGL(mlp_wgrad<false>, dim3(WG_GRID), dim3(256), 0, net->stream, w);
    }
    MLP_TRY(hipGetLastError());
    return LB_OK;
}

// The packed weights from the parameters.
lb_status pack(mlp_net* n) {
    hipLaunchKernelGGL(mlp_pack, dim3((unsigned)((param_count() + 255) / 256)), dim3(256), 0, n->stream, n->P,
                       n->packed);
    MLP_TRY(hipGetLastError());
    return LB_OK;
}

lb_status ensure_loss(mlp_net* n, int count) {
    if (count <= n->loss_cap) return LB_OK;
    MLP_TRY(hipStreamSynchronize(n->stream));
    (void)hipFree(n->loss);
    n->loss = nullptr;
    n->loss_cap = 0;
    MLP_TRY(hipMalloc(&n->loss, sizeof(float) * (size_t)count));
    n->loss_cap = count;
    return LB_OK;
}

lb_status check_net(const mlp_net* n) {
    if (!n) return lbk::set_error(LB_EINVAL, "null network");
    return LB_OK;
}

}  // namespace

extern "C" {

lb_status mlp_init(mlp_net** out, int seed, void* hip_stream) {
    if (!out) return lbk::set_error(LB_EINVAL, "null output pointer");
    *out = nullptr;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev == 0) return lbk::set_error(LB_EDEVICE, "no HIP device");
    mlp_net* n = new mlp_net();
    n->stream = (hipStream_t)hip_stream;
    if (hipGetDevice(&n->device) != hipSuccess) {
        delete n;
        return lbk::set_error(LB_EDEVICE, "no current HIP device");
    }
    const long np = param_count();
    auto bail = [&](lb_status st) {
        mlp_free(n);
        return st;
    };
    // one allocation: parameters, gradients, moments, packed weights, the copy of X (sizes
    // in whole 256-byte lines)
    static_assert(w_off(NLAYER) % 64 == 0 && PACKED % 64 == 0, "aligned parts");
    if (hipMalloc(&n->P, sizeof(float) * (4 * np + PACKED + MLP_NOALLOC_MAX_ROWS * DIMS[0])) != hipSuccess)
        return bail(lbk::set_error(LB_ENOMEM, "device allocation of the network failed"));
    n->G = n->P + np;
    n->Mo = n->G + np;
    n->Vo = n->Mo + np;
    n->packed = n->Vo + np;
    n->xcopy = n->packed + PACKED;
    // uniform(-1/sqrt(fan_in), 1/sqrt(fan_in)) for weights and biases
    std::vector<float> h(np);
    for (int l = 0; l < NLAYER; ++l) {
        const double bound = 1.0 / std::sqrt((double)DIMS[l]);
        const long a = w_off(l), b = b_off(l) + DIMS[l + 1];
        for (long i = a; i < b; ++i) h[i] = (float)((2.0 * uniform01((uint64_t)seed, (uint64_t)i) - 1.0) * bound);
    }
    if (hipMemsetAsync(n->G, 0, sizeof(float) * (3 * np + PACKED), n->stream) != hipSuccess ||
        hipMemcpyAsync(n->P, h.data(), sizeof(float) * np, hipMemcpyHostToDevice, n->stream) != hipSuccess)
        return bail(lbk::set_error(LB_EDEVICE, "network initialisation failed"));
    if (lb_status st = pack(n)) return bail(st);
    if (hipStreamSynchronize(n->stream) != hipSuccess)
        return bail(lbk::set_error(LB_EDEVICE, "network initialisation failed"));
    *out = n;
    return LB_OK;
}

void mlp_free(mlp_net* n) {
    if (!n) return;
    if (n->stream) (void)hipStreamSynchronize(n->stream);
    else (void)hipDeviceSynchronize();
    free_rows(n);
    free_groups(n);
    if (n->pin) lbk::pin_give((char*)n->pin);
    (void)hipFree(n->P);
    (void)hipFree(n->loss);
    (void)hipFree(n->Xall);
    (void)hipFree(n->Yall);
    (void)hipFree(n->idx);
    delete n;
}

long mlp_param_count(const mlp_net* n) { return n ? param_count() : 0; }

lb_status mlp_get_params(mlp_net* n, float* host, long count) {
    if (lb_status st = check_net(n)) return st;
    if (!host || count != param_count()) return lbk::set_error(LB_EINVAL, "parameter buffer size mismatch");
    MLP_TRY(hipMemcpyAsync(host, n->P, sizeof(float) * count, hipMemcpyDeviceToHost, n->stream));
    MLP_TRY(hipStreamSynchronize(n->stream));
    return LB_OK;
}

lb_status mlp_set_params(mlp_net* n, const float* host, long count) {
    if (lb_status st = check_net(n)) return st;
    if (!host || count != param_count()) return lbk::set_error(LB_EINVAL, "parameter buffer size mismatch");
    MLP_TRY(hipMemcpyAsync(n->P, host, sizeof(float) * count, hipMemcpyHostToDevice, n->stream));
    MLP_TRY(hipMemsetAsync(n->Mo, 0, sizeof(float) * count, n->stream));
    MLP_TRY(hipMemsetAsync(n->Vo, 0, sizeof(float) * count, n->stream));
    if (lb_status st = pack(n)) return st;
    MLP_TRY(hipStreamSynchronize(n->stream));
    n->adam_t = 0;
    return LB_OK;
}

lb_status mlp_predict(mlp_net* n, const float* X, int rows, float* Y) {
    if (lb_status st = check_net(n)) return st;
    if (rows < 0 || (rows > 0 && (!X || !Y))) return lbk::set_error(LB_EINVAL, "bad rows or null arrays");
    if (rows == 0) return LB_OK;
    if (rows <= PIN_ROWS) {
        if (!n->pin) n->pin = (float*)lbk::pin_take();
        if (!n->pin) return lbk::set_error(LB_ENOMEM, "allocation of pinned host memory failed");
        float *hx = n->pin, *hy = n->pin + PIN_ROWS * DIMS[0];
        std::memcpy(hx, X, sizeof(float) * (size_t)rows * DIMS[0]);
        if (lb_status st = forward(n, hx, rows, hy)) return st;
        MLP_TRY(hipStreamSynchronize(n->stream));
        std::memcpy(Y, hy, sizeof(float) * (size_t)rows * DIMS[NLAYER]);
        return LB_OK;
    }
    if (lb_status st = ensure_rows(n, rows)) return st;
    MLP_TRY(hipMemcpyAsync(n->x, X, sizeof(float) * (size_t)rows * DIMS[0], hipMemcpyHostToDevice, n->stream));
    if (lb_status st = forward(n, n->x, rows, n->y)) return st;
    MLP_TRY(hipMemcpyAsync(Y, n->y, sizeof(float) * (size_t)rows * DIMS[NLAYER], hipMemcpyDeviceToHost, n->stream));
    MLP_TRY(hipStreamSynchronize(n->stream));
    return LB_OK;
}

lb_status mlp_predict_device_noalloc(mlp_net* n, const float* dX, int rows, float* dY) {
    if (lb_status st = check_net(n)) return st;
    if (rows < 0 || rows > MLP_NOALLOC_MAX_ROWS)
        return lbk::set_error(LB_EINVAL, "mlp_predict_device_noalloc: rows must be in 0..MLP_NOALLOC_MAX_ROWS (1024)");
    if (rows > 0 && (!dX || !dY)) return lbk::set_error(LB_EINVAL, "null device arrays");
    if (rows == 0) return LB_OK;
    // rows are finished in any order: an output that overlaps the inputs needs a copy of them
    const uintptr_t x0 = (uintptr_t)dX, x1 = x0 + sizeof(float) * (size_t)rows * DIMS[0];
    const uintptr_t y0 = (uintptr_t)dY, y1 = y0 + sizeof(float) * (size_t)rows * DIMS[NLAYER];
    if (x0 < y1 && y0 < x1) {
        MLP_TRY(hipMemcpyAsync(n->xcopy, dX, x1 - x0, hipMemcpyDeviceToDevice, n->stream));
        dX = n->xcopy;
    }
    return forward(n, dX, rows, dY);
}

lb_status mlp_loss_grad(mlp_net* n, const float* X, const float* Y, int rows, float* loss, float* grads) {
    if (lb_status st = check_net(n)) return st;
    if (rows <= 0 || !X || !Y) return lbk::set_error(LB_EINVAL, "bad rows or null arrays");
    if (lb_status st = ensure_rows(n, rows)) return st;
    if (lb_status st = ensure_groups(n, rows)) return st;
    if (lb_status st = ensure_loss(n, 1)) return st;
    MLP_TRY(hipMemcpyAsync(n->x, X, sizeof(float) * (size_t)rows * DIMS[0], hipMemcpyHostToDevice, n->stream));
    MLP_TRY(hipMemcpyAsync(n->y, Y, sizeof(float) * (size_t)rows * DIMS[NLAYER], hipMemcpyHostToDevice, n->stream));
    if (lb_status st = gradient(n, n->x, n->y, nullptr, rows, n->loss, false, 0.f)) return st;
    float l = 0.f;
    MLP_TRY(hipMemcpyAsync(&l, n->loss, sizeof(float), hipMemcpyDeviceToHost, n->stream));
    if (grads)
        MLP_TRY(hipMemcpyAsync(grads, n->G, sizeof(float) * param_count(), hipMemcpyDeviceToHost, n->stream));
    MLP_TRY(hipStreamSynchronize(n->stream));
    if (loss) *loss = l;
    return LB_OK;
}

lb_status mlp_train(mlp_net* n, const float* X, const float* Y, int rows, int epochs, int batch, float lr, int seed,
                    float* last_loss) {
    if (lb_status st = check_net(n)) return st;
    if (rows <= 0 || !X || !Y || epochs < 0 || batch <= 0 || !(lr > 0.f))
        return lbk::set_error(LB_EINVAL, "bad training arguments");
    const int nb = (rows + batch - 1) / batch;   // minibatches per epoch, the last one may be short
    const int bmax = std::min(batch, rows);
    if (lb_status st = ensure_groups(n, bmax)) return st;
    if (lb_status st = ensure_loss(n, nb)) return st;
    if (rows > n->data_cap) {
        MLP_TRY(hipStreamSynchronize(n->stream));
        (void)hipFree(n->Xall);
        (void)hipFree(n->Yall);
        (void)hipFree(n->idx);
        n->Xall = n->Yall = nullptr;
        n->idx = nullptr;
        n->data_cap = 0;
        MLP_TRY(hipMalloc(&n->Xall, sizeof(float) * (size_t)rows * DIMS[0]));
        MLP_TRY(hipMalloc(&n->Yall, sizeof(float) * (size_t)rows * DIMS[NLAYER]));
        MLP_TRY(hipMalloc(&n->idx, sizeof(int) * (size_t)rows));
        n->data_cap = rows;
    }
    MLP_TRY(hipMemcpyAsync(n->Xall, X, sizeof(float) * (size_t)rows * DIMS[0], hipMemcpyHostToDevice, n->stream));
    MLP_TRY(hipMemcpyAsync(n->Yall, Y, sizeof(float) * (size_t)rows * DIMS[NLAYER], hipMemcpyHostToDevice, n->stream));
    std::vector<int> perm(rows);
    for (int e = 0; e < epochs; ++e) {
        // seeded Fisher-Yates shuffle of the rows
        for (int i = 0; i < rows; ++i) perm[i] = i;
        for (int i = rows - 1; i > 0; --i) {
            const uint64_t r = splitmix64(((uint64_t)seed << 32) ^ ((uint64_t)e * 0x9E3779B97F4A7C15ull) ^ (uint64_t)i);
            std::swap(perm[i], perm[(int)(r % (uint64_t)(i + 1))]);
        }
        MLP_TRY(hipStreamSynchronize(n->stream));   // the previous epoch's index upload has been consumed
        MLP_TRY(hipMemcpy(n->idx, perm.data(), sizeof(int) * (size_t)rows, hipMemcpyHostToDevice));
        for (int b = 0; b < nb; ++b) {
            const int r0 = b * batch, nr = std::min(batch, rows - r0);
            if (lb_status st = gradient(n, n->Xall, n->Yall, n->idx + r0, nr, n->loss + b, true, lr)) return st;
        }
    }
    if (last_loss) {
        *last_loss = 0.f;
        if (epochs > 0) {
            std::vector<float> l(nb);
            MLP_TRY(hipMemcpyAsync(l.data(), n->loss, sizeof(float) * nb, hipMemcpyDeviceToHost, n->stream));
            MLP_TRY(hipStreamSynchronize(n->stream));
            double s = 0.0;
            for (int b = 0; b < nb; ++b) s += (double)l[b] * std::min(batch, rows - b * batch);
            *last_loss = (float)(s / rows);
        }
    }
    MLP_TRY(hipStreamSynchronize(n->stream));
    return LB_OK;
}

}  // extern "C"
