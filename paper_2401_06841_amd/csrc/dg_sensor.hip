// dg_sensor.hip -- learned shock sensor: per-cell features, plain-sensor labels, the
// 20-64-64-1 GELU network on the bf16 matrix cores (forward, gradient, Adam) and the
// judge that sends cells back to the plain sensor.  The network is not in the paper; it
// stands in for the compression sensor of Sec. 3.1 and is trained on that sensor's output.
//
// Matrix-core mapping (v_mfma_f32_16x16x32_bf16, one wave64 per 16-row tile): lane
// 16 g + i holds A[i][8g .. 8g+7], B[8g .. 8g+7][i] and accumulates D[4g .. 4g+3][i].
// Activations are rounded to bf16 only where they feed a matrix instruction; bias, GELU,
// the last layer and all accumulations are FP32.  Gradients are reduced per wave, then
// summed over waves and blocks in a fixed order (deterministic).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>

#include "dg.h"
#include "dg_ctx.hpp"
#include "dg_kernels.hpp"

namespace dg {

constexpr int NIN = DG_MLP_NIN, NH = DG_MLP_NHID, NPARAM = DG_MLP_NPARAM;
constexpr int OFF_W1 = 0, OFF_B1 = NH * NIN, OFF_W2 = OFF_B1 + NH, OFF_B2 = OFF_W2 + NH * NH,
              OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NH;
constexpr int MLP_BLOCKS = MLP_PART_ROWS / 4;   // blocks of the gradient kernel: its 4 waves are one per SIMD
constexpr double NU0 = 1e-3;            // nu scale of the target t = log(1 + nu/nu0)

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }

// GELU and its derivative from one exponential: gelu = z Phi(z), gelu' = Phi(z) + z phi(z).  The
// tail q = Phi(-|z|) = exp(-z^2/2) erfcx(|z|/sqrt 2)/2 is the same exponential times 1/2 plus a
// polynomial of degree 9 without a constant term in w = 0.36 |z|/(1 + 0.36 |z|), a weighted fit of that
// quotient on 0 <= |z| <= 14 (largest relative error 2.4e-7, times the exponential 2.4e-9; the
// reciprocal is the hardware's, to 1 ulp, which counts for little in w).  Largest errors against
// 64 bits over |z| <= 8, measured: 3.8e-7 (gelu) and 1.1e-7 (gelu', rms 2.4e-8); with the library's erff
// and expf 4.4e-7 and 1.3e-7 (rms 2.6e-8) at three times the instructions, and the relative error of
// gelu's negative tail (4e-6) there is 1, from 1 + erf.  (A polynomial in 1 - w, whose terms have to
// add up to 1/2 at z = 0: 2.0e-7 in gelu' there, at the same speed.)
__device__ __forceinline__ void gelu_both(float z, float &f, float &d)
{
    const float b = 0.36f * fabsf(z);
    const float e = __builtin_amdgcn_exp2f(z * z * -0.72134752044448170f);
    const float w = b * __builtin_amdgcn_rcpf(1.0f + b);
    float p = 0.0159039553f;
    p = fmaf(p, w, -0.0774657652f);
    p = fmaf(p, w, 0.107688867f);
    p = fmaf(p, w, -0.0153067438f);
    p = fmaf(p, w, 0.011065728f);
    p = fmaf(p, w, -0.154588133f);
    p = fmaf(p, w, -0.0999606401f);
    p = fmaf(p, w, 0.820816517f);
    p = fmaf(p, w, -1.10817254f);
    const float q = fmaf(p, w, 0.5f) * e;
    const float cdf = z < 0.0f ? q : 1.0f - q;
    f = z * cdf;
    d = fmaf(z, 0.39894228040143268f * e, cdf);
}

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// the 16-slot form: lane 16 g + i holds A[i][4g .. 4g+3], B[4g .. 4g+3][i]
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 mfma(bf16x4 a, bf16x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b), c, 0, 0, 0);
}

__device__ __forceinline__ void wave_fence() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

// sum over the 16 lanes of a lane group (same g), in pairs at distance 1, 2, 4, 8: the group is a
// row of the data-parallel moves, so nothing goes through LDS (lanes that already hold equal sums
// may be paired in mirrored order)
template <int CTRL>
__device__ __forceinline__ float row_move(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}

__device__ __forceinline__ float group_sum(float v)
{
    v += row_move<0xB1>(v);     // quad_perm [1, 0, 3, 2]
    v += row_move<0x4E>(v);     // quad_perm [2, 3, 0, 1]
    v += row_move<0x141>(v);    // row_half_mirror
    v += row_move<0x140>(v);    // row_mirror
    return v;
}

// sum over the 4 lane groups (same i)
__device__ __forceinline__ float across_groups(float v)
{
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    return v;
}

// network weights of one wave in matrix-operand form
struct Net {
    bf16x8 b1[4];        // layer 1, tile t: W1[16t+i][8g+j] (k >= 20: 0)
    bf16x8 b2[2][4];     // layer 2, (k-step s, tile t): W2[16t+i][32s+8g+j]
    float bias1[4], bias2[4], w3[4];
    float b3;
};

__device__ __forceinline__ void load_net(const float *__restrict__ P, Net &w)
{
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int k = 8 * g + j;
            const float v = P[OFF_W1 + (16 * t + i) * NIN + (k < NIN ? k : 0)];   // (no branch per load)
            w.b1[t][j] = (__bf16)(k < NIN ? v : 0.0f);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int j = 0; j < 8; ++j) w.b2[s][t][j] = (__bf16)P[OFF_W2 + (16 * t + i) * NH + 32 * s + 8 * g + j];
        w.bias1[t] = P[OFF_B1 + 16 * t + i];
        w.bias2[t] = P[OFF_B2 + 16 * t + i];
        w.w3[t] = P[OFF_W3 + 16 * t + i];
    }
    w.b3 = P[OFF_B3];
}

// per-wave LDS scratch of one tile (bf16)
struct alignas(16) TileLds {
    __bf16 h1[16 * NH];     // H1 row-major [row][n]
};

// the features 8g .. 8g+7 of row r as a matrix operand (rows past n and features past 20: zeros);
// a row is 80 bytes, of which only 4-byte alignment is known
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
struct Row {
    f32x4 lo, hi;
};
__device__ __forceinline__ Row load_row(const float *__restrict__ x, long r, int n)
{
    const int g = (threadIdx.x & 63) >> 4;
    Row v = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
    if (r < n && g < 3) {
        const f4u *p = (const f4u *)(x + (size_t)r * NIN + 8 * g);
        v.lo = p[0];
        if (g < 2) v.hi = p[1];
    }
    return v;
}

// forward pass of a 16-row tile from the lane's row of inputs (row i of the tile).  y[j]: output of
// row 4g+j (valid in every lane of the group).
__device__ __forceinline__ void forward_tile(const Row &xr, const Net &w, TileLds &L, float (&y)[4])
{
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    bf16x8 a;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        a[j] = (__bf16)xr.lo[j];
        a[4 + j] = (__bf16)xr.hi[j];
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        f32x4 d = mfma(a, w.b1[t], f32x4{0.0f, 0.0f, 0.0f, 0.0f});
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            L.h1[(4 * g + j) * NH + 16 * t + i] = (__bf16)gelu(d[j] + w.bias1[t]);
        }
    }
    wave_fence();
    bf16x8 a2[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) a2[s] = *(const bf16x8 *)&L.h1[i * NH + 32 * s + 8 * g];
    float p[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        f32x4 d = mfma(a2[0], w.b2[0][t], f32x4{0.0f, 0.0f, 0.0f, 0.0f});
        d = mfma(a2[1], w.b2[1][t], d);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            p[j] += gelu(d[j] + w.bias2[t]) * w.w3[t];
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] = group_sum(p[j]) + w.b3;
    wave_fence();
}

// ------------------------------------------------------------------ forward
// y[n] from x[n][20]; with nu != nullptr the output is the viscosity
// nu = nu0 (exp(y) - 1), clipped at zero, stored in the state's element type.  With vmax
// != nullptr each block also writes vmax[block] = the largest stored viscosity of its cells
// whose fallback flag fb is 0 (0 if none): the learned cells' part of the viscous time-step
// bound.
template <typename T>
__global__ void __launch_bounds__(256) k_mlp_forward(const float *__restrict__ P, const float *__restrict__ x, int n,
                                                     float *__restrict__ y, T *__restrict__ nu,
                                                     const int *__restrict__ fb, double *__restrict__ vmax)
{
    __shared__ double bmax[4];
    double vm = 0.0;
    __shared__ TileLds lds[4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    Net w;
    load_net(P, w);
    const int ntile = (n + 15) / 16;
    const int nw = gridDim.x * 4;
    Row next = load_row(x, (long)(blockIdx.x * 4 + wave) * 16 + i, n);
    for (int tile = blockIdx.x * 4 + wave; tile < ntile; tile += nw) {
        float yy[4];
        const Row xr = next;
        next = load_row(x, ((long)tile + nw) * 16 + i, n);      // in flight while this tile is worked on
        forward_tile(xr, w, lds[wave], yy);
        // lane i < 4 of each group finishes row 4g + i (one exponential for all 16 rows; four in a row in
        // lane 0 were a tenth of the pass: 398 -> 348 us for 128^3 cells, 315 us with the sums over the
        // groups in data-parallel moves and the inputs loaded a tile ahead)
        const int r = tile * 16 + 4 * g + i;
        if (i < 4 && r < n) {
            const float yr = i == 0 ? yy[0] : (i == 1 ? yy[1] : (i == 2 ? yy[2] : yy[3]));
            if (y) y[r] = yr;
            if (nu) {
                const T v = (T)fmax(NU0 * expm1((double)yr), 0.0);
                nu[r] = v;
                if (vmax && fb[r] == 0) vm = fmax(vm, fmax((double)v, 0.0));
            }
        }
    }
    if (vmax) {
        vm = wave_max(vm);
        if (lane == 0) bmax[wave] = vm;
        __syncthreads();
        if (threadIdx.x == 0) vmax[blockIdx.x] = fmax(fmax(bmax[0], bmax[1]), fmax(bmax[2], bmax[3]));
    }
}

// --------------------------------------------------------------- gradient
// four FP32 values as bf16, into half HALF of a matrix operand
template <int HALF>
__device__ __forceinline__ void pack4(const f32x4 &v, bf16x8 &o)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) o[4 * HALF + j] = (__bf16)v[j];
}

__device__ __forceinline__ bf16x4 to_bf16(const f32x4 &v)
{
    bf16x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = (__bf16)v[j];
    return o;
}

// Mean-squared-error loss L = (1/n) sum (y - t)^2 and dL/dparams; each block writes the sums of
// its rows to part[block][NPARAM + 1] (the last entry is the loss sum).
//
// A wave takes a 16-row tile at a time and keeps it in registers throughout.  The layers run
// transposed, D[neuron][row] = W X^T: lane (g, i) then holds, for row i, the neurons 16t + 4g + j
// (t, j < 4), which is an operand of the next layer's product as it is when slot (s, g, jj) of the
// contraction stands for neuron 16(2s + (jj >> 2)) + 4g + (jj & 3) on both sides.  The weight
// gradients contract over rows: their operands need a neuron per lane and rows in the slots, the
// transpose, which the matrix cores give too: the held values as the left operand times a 0/1
// matrix that picks the neurons 16t + i is D[row][16t + i], exactly (one product per 16 neurons
// instead of 16-bit stores and loads through LDS, 88 per tile before).  Every lane needs GELU and
// its derivative of 32 values per tile, which bounds the kernel: both come from one exponential
// (gelu_both).  One wave per SIMD: the weights in operand form (80 registers) and the gradient
// accumulators (144) beside the tile (32 rows at a time spilled 14-51 registers).  One gradient and
// update, before and after: 197 -> 61 us at 262,144 rows, 45 -> 25 us at 16,000, 25 -> 17 us at
// 1,000, 675 -> 180 us at 1,000,000.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1)))
k_mlp_grad(const float *__restrict__ P, const float *__restrict__ x, const float *__restrict__ tgt, int n,
           float *__restrict__ part)
{
    // the parameters on entry (a wave's operands are built from here: one coalesced read of them per
    // block), the waves' gradient sums at the end
    constexpr int ROW = (NPARAM + 1 + 3) / 4 * 4;
    __shared__ alignas(16) float red[4][ROW];
    // the FP32 vectors of the network: biases and last layer (a lane's four neurons are one 16-byte
    // read; in registers they made the kernel spill)
    __shared__ f32x4 vec[3][NH / 4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int nw = gridDim.x * 4;
    Row next = load_row(x, (long)(blockIdx.x * 4 + wave) * 16 + i, n);
    float *Q = red[0];
#pragma unroll
    for (int j = 0; j < (NPARAM + 255) / 256; ++j) {
        const int p = 256 * j + threadIdx.x;
        if (p < NPARAM) Q[p] = P[p];
    }
    __syncthreads();
    if (threadIdx.x < NH) {
        ((float *)vec[0])[threadIdx.x] = Q[OFF_B1 + threadIdx.x];
        ((float *)vec[1])[threadIdx.x] = Q[OFF_B2 + threadIdx.x];
        ((float *)vec[2])[threadIdx.x] = Q[OFF_W3 + threadIdx.x];
    }
    // neuron of contraction slot (s, g, jj)
    auto neuron = [&](int s, int jj) { return 16 * (2 * s + (jj >> 2)) + 4 * g + (jj & 3); };
    bf16x8 w1[4], w2[2][4], w2t[2][4], sel[2];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            const int k = 8 * g + jj;
            const float w = Q[OFF_W1 + (16 * t + i) * NIN + (k < NIN ? k : 0)];   // (no branch per load)
            w1[t][jj] = (__bf16)(k < NIN ? w : 0.0f);
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) {
                w2[s][t][jj] = (__bf16)Q[OFF_W2 + (16 * t + i) * NH + neuron(s, jj)];
                w2t[s][t][jj] = (__bf16)Q[OFF_W2 + neuron(s, jj) * NH + 16 * t + i];
            }
    }
    const float b3 = Q[OFF_B3];
    __syncthreads();
    // sel[p]: picks, of the 8 values of a slot group, the one of half p that belongs to lane i
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) sel[p][jj] = (__bf16)((jj >> 2) == p && 4 * g + (jj & 3) == i ? 1.0f : 0.0f);

    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 aw2[4][4], aw1[4][2], gb1[4], gb2[4], gw3[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
#pragma unroll
        for (int b = 0; b < 4; ++b) aw2[a][b] = zero;
        aw1[a][0] = aw1[a][1] = zero;
        gb1[a] = gb2[a] = gw3[a] = zero;
    }
    float gb3 = 0.0f, loss = 0.0f;
    const float inv_n = 1.0f / (float)n;
    const int ntile = (int)(((long)n + 15) / 16);
    for (int tile = blockIdx.x * 4 + wave; tile < ntile; tile += nw) {
        const f32x4 *b1 = vec[0] + g, *b2 = vec[1] + g, *w3 = vec[2] + g;
        const int r = tile * 16 + i;
        const bool in = r < n;
        bf16x8 xb, hb[2], gb[2], gc[2];
        pack4<0>(next.lo, xb);
        pack4<1>(next.hi, xb);
        next = load_row(x, ((long)tile + nw) * 16 + i, n);      // in flight while this tile is worked on
        const float target = in ? tgt[r] : 0.0f;
        f32x4 d1[4], d2[4], h2[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const f32x4 z = mfma(w1[t], xb, zero) + b1[4 * t];
            f32x4 h;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float f, d;
                gelu_both(z[j], f, d);
                h[j] = f;
                d1[t][j] = d;
            }
            if (t & 1) pack4<1>(h, hb[t >> 1]);
            else pack4<0>(h, hb[t >> 1]);
        }
        // layer 2 and the output of row i, summed over the neurons of the lane, then over g
        float y = 0.0f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            f32x4 z = mfma(w2[0][t], hb[0], zero);
            z = mfma(w2[1][t], hb[1], z) + b2[4 * t];
            const f32x4 w3t = w3[4 * t];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float f, d;
                gelu_both(z[j], f, d);
                h2[t][j] = f;
                d2[t][j] = d;
                y = fmaf(f, w3t[j], y);
            }
        }
        y = across_groups(y) + b3;
        const float e = in ? y - target : 0.0f;
        const float g3 = 2.0f * inv_n * e;
        if (g == 0) {
            loss += e * e;
            gb3 += g3;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            gw3[t] += g3 * h2[t];
            const f32x4 v = (g3 * w3[4 * t]) * d2[t];
            gb2[t] += v;
            if (t & 1) pack4<1>(v, gb[t >> 1]);
            else pack4<0>(v, gb[t >> 1]);
        }
        // rows into the slots, a neuron per lane: dW2[m][k] += sum_rows G2[row][m] H1[row][k]
        bf16x4 ta[4], tb[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            ta[t] = to_bf16(mfma(gb[t >> 1], sel[t & 1], zero));
            tb[t] = to_bf16(mfma(hb[t >> 1], sel[t & 1], zero));
        }
#pragma unroll
        for (int tn = 0; tn < 4; ++tn)
#pragma unroll
            for (int tk = 0; tk < 4; ++tk) aw2[tn][tk] = mfma(ta[tn], tb[tk], aw2[tn][tk]);
        // G1 = (W2^T G2) gelu'(z1)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            f32x4 z = mfma(w2t[0][t], gb[0], zero);
            z = mfma(w2t[1][t], gb[1], z) * d1[t];
            gb1[t] += z;
            if (t & 1) pack4<1>(z, gc[t >> 1]);
            else pack4<0>(z, gc[t >> 1]);
        }
        // dW1[k][f] += sum_rows G1[row][k] X[row][f]
#pragma unroll
        for (int p = 0; p < 2; ++p) tb[p] = to_bf16(mfma(xb, sel[p], zero));
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            ta[t] = to_bf16(mfma(gc[t >> 1], sel[t & 1], zero));
#pragma unroll
            for (int p = 0; p < 2; ++p) aw1[t][p] = mfma(ta[t], tb[p], aw1[t][p]);
        }
    }
    // the neurons' sums over the 16 lanes (rows) of a group, all waves at once
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            gb1[t][j] = group_sum(gb1[t][j]);
            gb2[t][j] = group_sum(gb2[t][j]);
            gw3[t][j] = group_sum(gw3[t][j]);
        }
    gb3 = group_sum(gb3);
    loss = group_sum(loss);
    // every wave's sums into its own row, then the block's in wave order
    float *own = red[wave];
#pragma unroll
    for (int tn = 0; tn < 4; ++tn) {
#pragma unroll
        for (int tk = 0; tk < 4; ++tk)
#pragma unroll
            for (int j = 0; j < 4; ++j) own[OFF_W2 + (16 * tn + 4 * g + j) * NH + 16 * tk + i] = aw2[tn][tk][j];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int f = 8 * (i >> 2) + 4 * p + (i & 3);      // input feature of column i of half p
            if (f < NIN)
#pragma unroll
                for (int j = 0; j < 4; ++j) own[OFF_W1 + (16 * tn + 4 * g + j) * NIN + f] = aw1[tn][p][j];
        }
        if (i == 0)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                own[OFF_B1 + 16 * tn + 4 * g + j] = gb1[tn][j];
                own[OFF_B2 + 16 * tn + 4 * g + j] = gb2[tn][j];
                own[OFF_W3 + 16 * tn + 4 * g + j] = gw3[tn][j];
            }
    }
    if (lane == 0) {
        own[OFF_B3] = gb3;
        own[NPARAM] = loss;
    }
    __syncthreads();
    float *pw = part + (size_t)blockIdx.x * (NPARAM + 1);
    for (int p = threadIdx.x; p <= NPARAM; p += 256) pw[p] = ((red[0][p] + red[1][p]) + red[2][p]) + red[3][p];
}

// fixed-order sum of the per-block partials: grad[p] and loss = sum / n.  A block takes 16
// entries; its 16 lane groups sum the rows r, r+16, r+32, ... in order, and the group sums are
// added in order.
__global__ void __launch_bounds__(256) k_mlp_reduce(const float *__restrict__ part, int nrows, int n,
                                                    float *__restrict__ grad, float *__restrict__ loss)
{
    __shared__ float lds[16][16];
    const int r = threadIdx.x >> 4, e = threadIdx.x & 15;
    const int p = blockIdx.x * 16 + e;
    float s = 0.0f;
    if (p <= NPARAM)
#pragma unroll 16
        for (int row = r; row < nrows; row += 16) s += part[(size_t)row * (NPARAM + 1) + p];
    lds[r][e] = s;
    __syncthreads();
    if (r == 0 && p <= NPARAM) {
        float t = lds[0][e];
#pragma unroll
        for (int k = 1; k < 16; ++k) t += lds[k][e];
        if (p < NPARAM) grad[p] = t;
        else loss[0] = t / (float)n;
    }
}

// Adam (Kingma & Ba 2015), beta1 0.9, beta2 0.999, eps 1e-8
__global__ void __launch_bounds__(256) k_mlp_adam(float *__restrict__ P, const float *__restrict__ G,
                                                  float *__restrict__ m, float *__restrict__ v, int step, float lr)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= NPARAM) return;
    const float b1 = 0.9f, b2 = 0.999f;
    const float gg = G[p];
    const float mm = b1 * m[p] + (1.0f - b1) * gg;
    const float vv = b2 * v[p] + (1.0f - b2) * gg * gg;
    m[p] = mm;
    v[p] = vv;
    const float mh = mm / (1.0f - powf(b1, (float)step));
    const float vh = vv / (1.0f - powf(b2, (float)step));
    P[p] -= lr * mh / (sqrtf(vh) + 1e-8f);
}

// ------------------------------------------------------------ features
// x[cell][20] (degree 2, modes in graded order 0:(000) 1:(100) 2:(010) 3:(001) 4:(200)
// 5:(110) 6:(101) 7:(020) 8:(011) 9:(002)):
//   [0..5]   density shape W_rho,l/W_rho,0 for l = 1, 2, 3, 4, 7, 9
//   [6]      log10 W_rho,0
//   [7..15]  cell-mean velocity gradient (2 sqrt(3)/h) vhat_{d,(e)}, scaled by (h/3)/cs
//   [16..18] slopes of div vhat across the cell: with d/dxi Lt_1 = sqrt(3) and
//            d/dxi Lt_2 = 3 sqrt(5) xi the divergence is D0 + sum_i D_i xi_i with
//            D_1 = 3 sqrt(5) V_x,(200) + 3 V_y,(110) + 3 V_z,(101) (and cyclic), times 2/h,
//            scaled by (h/3)/cs
//   [19]     |mean velocity|/cs
// vhat: the projected velocity of u already at hand (same arithmetic as project_lines), used
// unless *fail is raised (then u is not the state vhat belongs to); NULL: project here.
template <typename T>
__global__ void __launch_bounds__(BLOCK) k_features(const void *u_, float *__restrict__ x, const void *tab_, Mesh g,
                                                    double cs, const void *vhat, const int *fail)
{
    constexpr int K = 2, NB = Shape<K>::NB;
    const int nc = g.nc;
    const int c0 = blockIdx.x * BLOCK + threadIdx.x;
    const bool active = c0 < nc;
    const int c = active ? c0 : 0;
    const unsigned bo = (unsigned)c * sizeof(T);
    T W[4][NB];
    T V[3][NB];
    if (vhat && !*fail) {
#pragma unroll
        for (int l = 0; l < NB; ++l) W[0][l] = Field<T, 1>(u_, NB, nc).get(0, l, bo);
        load_field<T, K, 3>(Field<T, 3>(vhat, NB, nc), bo, V);
    } else {
        load_field<T, K, 4>(Field<T, 4>(u_, NB, nc), bo, W);
        double sm = 0.0;
        project_lines<T, K, 0, 3, false>(W, as_tab<T>(tab_), V, 0.0, sm);
    }
    if (!active) return;
    const double r0 = (double)W[0][0];
    float *xc = x + (size_t)c * NIN;
    constexpr int dmode[6] = {1, 2, 3, 4, 7, 9};
#pragma unroll
    for (int i = 0; i < 6; ++i) xc[i] = (float)((double)W[0][dmode[i]] / r0);
    xc[6] = (float)log10(r0);
    const double fac = 2.0 * 1.7320508075688772 / (3.0 * cs);
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int e = 0; e < 3; ++e) xc[7 + 3 * d + e] = (float)(fac * (double)V[d][1 + e]);
    const double r5 = 3.0 * 2.23606797749979;     // 3 sqrt(5)
    const double sfac = 2.0 / (3.0 * cs);         // (h/3)/cs * 2/h
    xc[16] = (float)(sfac * (r5 * (double)V[0][4] + 3.0 * (double)V[1][5] + 3.0 * (double)V[2][6]));
    xc[17] = (float)(sfac * (3.0 * (double)V[0][5] + r5 * (double)V[1][7] + 3.0 * (double)V[2][8]));
    xc[18] = (float)(sfac * (3.0 * (double)V[0][6] + 3.0 * (double)V[1][8] + r5 * (double)V[2][9]));
    const double vm = sqrt((double)V[0][0] * V[0][0] + (double)V[1][0] * V[1][0] + (double)V[2][0] * V[2][0]);
    xc[19] = (float)(vm / cs);
}

// plain-sensor label: the vNR bulk viscosity nu(s) = alpha (h/p)^2 s + beta cs (h/p)
// (Pi = rho nu s without the cap, Sec. 3.1) averaged over the compressed interior points
// (s = -div v > 0) with weights omega s: nu = alpha (h/p)^2 sum(w s^2)/sum(w s) + beta cs h/p
// OUT = double: the label nu itself; OUT = float: the training target log(1 + nu/nu0)
template <typename T, int K, typename OUT>
__global__ void __launch_bounds__(BLOCK) k_labels(const void *u_, OUT *__restrict__ nu, const void *tab_, Mesh g,
                                                  double h, double cs, double alpha, double beta)
{
    using S = Shape<K>;
    using TL = TabLayout<K>;
    constexpr int NB = S::NB;
    const int nc = g.nc;
    const int c0 = blockIdx.x * BLOCK + threadIdx.x;
    const bool active = c0 < nc;
    const int c = active ? c0 : 0;
    const unsigned bo = (unsigned)c * sizeof(T);
    ctab<T> *tab = as_tab<T>(tab_);
    T W[4][NB];
    load_field<T, K, 4>(Field<T, 4>(u_, NB, nc), bo, W);
    T V[3][NB];
    double sm = 0.0;
    project_lines<T, K, 0, 3, false>(W, tab, V, 0.0, sm);
    // modal coefficients of the divergence of the projected velocity, then its values line by line
    constexpr DivMap<K> DM = make_divmap<K>();
    T Dv[DivMap<K>::NDIV];
#pragma unroll
    for (int m = 0; m < DivMap<K>::NDIV; ++m) Dv[m] = T(0);
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int l = 0; l < NB; ++l)
#pragma unroll
            for (int t = 0; t < DivMap<K>::MAXT; ++t)
                if (DM.m[d][l][t] >= 0) Dv[DM.m[d][l][t]] += V[d][l] * T(__builtin_sqrt(double(DM.f[d][l][t])));
    double s1 = 0.0, s2 = 0.0;
#pragma unroll 1
    for (int r = 0; r < S::NF; ++r) {
        T cd[K], div[S::N1];
        line_coefficients<T, K, K>(Dv, tab + TL::F2 + r * S::NB2, cd);
        line_eval<K>(cd, div);
#pragma unroll
        for (int t = 0; t < S::N1; ++t) {
            const double sq = -(double)div[t] * (2.0 / h);
            if (sq > 0.0) {
                const double w = (double)tab[TL::VW + r + S::NF * t];
                s1 += w * sq;
                s2 += w * sq * sq;
            }
        }
    }
    if (!active) return;
    const double hp = h / (K + 1);
    const double v = s1 > 0.0 ? alpha * hp * hp * (s2 / s1) + beta * cs * hp : 0.0;
    if (sizeof(OUT) == 8) nu[c] = (OUT)v;
    else nu[c] = (OUT)log1p(v / NU0);
}

// judge: fallback flag where |nu_learned - nu_plain| / (nu_plain + nu0) > tau; counts the flags
template <typename T>
__global__ void __launch_bounds__(BLOCK) k_judge(const T *__restrict__ nul, const double *__restrict__ nup, int nc,
                                                 double tau, int *__restrict__ fb, unsigned long long *__restrict__ count)
{
    __shared__ double lds[4];
    const int c = blockIdx.x * BLOCK + threadIdx.x;
    int flag = 0;
    if (c < nc) {
        const double a = (double)nul[c], b = nup[c];
        flag = fabs(a - b) / (b + NU0) > tau ? 1 : 0;
        fb[c] = flag;
    }
    double v[1] = {(double)flag};
    block_sum<1>(v, lds);
    if (threadIdx.x == 0 && v[0] > 0.0) atomicAdd(count, (unsigned long long)v[0]);
}

__global__ void k_fill_int(int *__restrict__ p, int n, int value)
{
    const int c = blockIdx.x * BLOCK + threadIdx.x;
    if (c < n) p[c] = value;
}

}  // namespace dg

using namespace dg;

// gradient: at most MLP_BLOCKS blocks, one partial-sum row each
static int mlp_blocks(int n)
{
    const int ntile = (int)(((long)n + 15) / 16);
    return ntile < 4 * MLP_BLOCKS ? (ntile + 3) / 4 : MLP_BLOCKS;
}

// forward: one full round of waves at the kernel's occupancy (3 waves per SIMD), each wave
// looping over its share of the 16-row tiles (the network is loaded into registers once per
// wave, and no wave waits for a second round)
static int fwd_blocks(const dg_ctx *c, int n)
{
    const long ntile = ((long)n + 15) / 16;
    const long round = (long)c->ncu * 4 * 3;
    const long nw = ntile < round ? ntile : round;
    return (int)((nw + 3) / 4);
}

static float *mlp_part(dg_ctx *c) { return (float *)c->wp(c->off.mlp); }

static int need_k2(dg_ctx *c)
{
    if (c->k != 2) return dg_fail(c, DG_EUNSUPPORTED, "the learned sensor is defined for degree 2");
    if (!c->ws) return dg_fail(c, DG_ENOMEM, "no workspace set (dg_set_workspace)");
    return DG_OK;
}

int dg_mlp_forward(dg_ctx *c, const float *P, const float *x, int n, float *y)
{
    if (!c) return DG_EINVAL;
    if (!P || !x || !y || n < 0) return dg_fail(c, DG_EINVAL, "bad network arguments");
    if (n == 0) return DG_OK;
    int rc;
    if ((rc = dg_check_array(c, P, sizeof(float) * NPARAM, sizeof(float), "params")) ||
        (rc = dg_check_array(c, x, sizeof(float) * NIN * (size_t)n, sizeof(float), "x")) ||
        (rc = dg_check_array(c, y, sizeof(float) * (size_t)n, sizeof(float), "y")))
        return rc;
    hipLaunchKernelGGL((k_mlp_forward<float>), dim3(fwd_blocks(c, n)), dim3(256), 0, c->stream, P, x, n, y,
                       (float *)nullptr, (const int *)nullptr, (double *)nullptr);
    LAUNCHCHK(c);
    return DG_OK;
}

int dg_mlp_grad(dg_ctx *c, const float *P, const float *x, const float *t, int n, float *grad, float *loss)
{
    if (!c) return DG_EINVAL;
    if (!P || !x || !t || !grad || !loss || n <= 0) return dg_fail(c, DG_EINVAL, "bad network arguments");
    if (dg_check_array(c, P, sizeof(float) * NPARAM, sizeof(float), "params") ||
        dg_check_array(c, x, sizeof(float) * NIN * (size_t)n, sizeof(float), "x") ||
        dg_check_array(c, t, sizeof(float) * (size_t)n, sizeof(float), "t") ||
        dg_check_array(c, grad, sizeof(float) * NPARAM, sizeof(float), "grad") ||
        dg_check_array(c, loss, sizeof(float), sizeof(float), "loss"))
        return DG_EINVAL;
    if (!c->ws) return dg_fail(c, DG_ENOMEM, "no workspace set (dg_set_workspace)");
    const int nb = mlp_blocks(n);
    hipLaunchKernelGGL(k_mlp_grad, dim3(nb), dim3(256), 0, c->stream, P, x, t, n, mlp_part(c));
    LAUNCHCHK(c);
    hipLaunchKernelGGL(k_mlp_reduce, dim3((NPARAM + 1 + 15) / 16), dim3(256), 0, c->stream, (const float *)mlp_part(c),
                       nb, n, grad, loss);
    LAUNCHCHK(c);
    return DG_OK;
}

int dg_mlp_adam(dg_ctx *c, float *P, const float *G, float *m, float *v, int step, float lr)
{
    if (!c) return DG_EINVAL;
    if (!P || !G || !m || !v || step < 1 || !(lr > 0.0f)) return dg_fail(c, DG_EINVAL, "bad Adam arguments");
    if (dg_check_array(c, P, sizeof(float) * NPARAM, sizeof(float), "params") ||
        dg_check_array(c, G, sizeof(float) * NPARAM, sizeof(float), "grad") ||
        dg_check_array(c, m, sizeof(float) * NPARAM, sizeof(float), "m") ||
        dg_check_array(c, v, sizeof(float) * NPARAM, sizeof(float), "v"))
        return DG_EINVAL;
    hipLaunchKernelGGL(k_mlp_adam, dim3((NPARAM + 255) / 256), dim3(256), 0, c->stream, P, G, m, v, step, lr);
    LAUNCHCHK(c);
    return DG_OK;
}

int dg_sensor_set_params(dg_ctx *c, const float *P)
{
    if (!c) return DG_EINVAL;
    c->spec_valid = false;          // the viscosity or flags a launched next stage used change
    if (int rc = dg_check_array(c, P, sizeof(float) * NPARAM, sizeof(float), "params")) return rc;
    HIPCHK(c, hipMemcpyAsync(c->mlp_bf16, P, sizeof(float) * NPARAM, hipMemcpyDeviceToDevice, c->stream));
    c->have_params = true;
    return DG_OK;
}

static int launch_features(dg_ctx *c, const void *u, float *x, const void *vhat)
{
    const Mesh g{c->cfg.nx, c->cfg.ny, c->cfg.nz, c->nc};
    const int *fail = (const int *)c->fail();
    if (c->es == 8)
        hipLaunchKernelGGL((k_features<double>), dim3(c->nblk), dim3(BLOCK), 0, c->stream, u, x, c->tab, g, c->cfg.cs,
                           vhat, fail);
    else
        hipLaunchKernelGGL((k_features<float>), dim3(c->nblk), dim3(BLOCK), 0, c->stream, u, x, c->tab, g, c->cfg.cs,
                           vhat, fail);
    LAUNCHCHK(c);
    return DG_OK;
}

int dg_sensor_features(dg_ctx *c, const void *u, float *x)
{
    if (!c) return DG_EINVAL;
    int rc = need_k2(c);
    if (rc) return rc;
    if ((rc = dg_check_array(c, u, dg_state_bytes(c), c->es, "u")) ||
        (rc = dg_check_array(c, x, sizeof(float) * NIN * (size_t)c->nc, sizeof(float), "x")))
        return rc;
    return launch_features(c, u, x, nullptr);
}

template <typename T, int K, typename OUT>
static void launch_labels(dg_ctx *c, const void *u, OUT *nu)
{
    const Mesh g{c->cfg.nx, c->cfg.ny, c->cfg.nz, c->nc};
    hipLaunchKernelGGL((k_labels<T, K, OUT>), dim3(c->nblk), dim3(BLOCK), 0, c->stream, u, nu, c->tab, g, c->cfg.h,
                       c->cfg.cs, c->cfg.alpha_visc, c->cfg.beta_visc);
}

template <typename OUT>
static int labels_any(dg_ctx *c, const void *u, OUT *nu)
{
    if (!c) return DG_EINVAL;
    if (int rc = dg_check_array(c, u, dg_state_bytes(c), c->es, "u")) return rc;
    if (int rc = dg_check_array(c, nu, sizeof(OUT) * (size_t)c->nc, sizeof(OUT), "output")) return rc;
    if (c->es == 8) {
        if (c->k == 1) launch_labels<double, 1>(c, u, nu);
        else if (c->k == 2) launch_labels<double, 2>(c, u, nu);
        else launch_labels<double, 3>(c, u, nu);
    } else {
        if (c->k == 1) launch_labels<float, 1>(c, u, nu);
        else if (c->k == 2) launch_labels<float, 2>(c, u, nu);
        else launch_labels<float, 3>(c, u, nu);
    }
    LAUNCHCHK(c);
    return DG_OK;
}

int dg_sensor_labels(dg_ctx *c, const void *u, double *nu) { return labels_any(c, u, nu); }

int dg_sensor_targets(dg_ctx *c, const void *u, float *t)
{
    if (!c) return DG_EINVAL;
    int rc = need_k2(c);
    if (rc) return rc;
    return labels_any(c, u, t);
}

int sensor_infer_impl(dg_ctx *c, const void *u, int *nvmax, const void *vhat)
{
    int rc = need_k2(c);
    if (rc) return rc;
    if (!c->have_params) return dg_fail(c, DG_ESTATE, "no network parameters (dg_sensor_set_params)");
    float *x = (float *)c->wp(c->off.feat);
    if ((rc = dg_check_array(c, u, dg_state_bytes(c), c->es, "u"))) return rc;
    rc = launch_features(c, u, x, vhat);
    if (rc) return rc;
    const int nblk = fwd_blocks(c, c->nc);
    const int *fb = nvmax ? (const int *)c->wp(c->off.fb) : nullptr;
    double *vmax = nvmax ? (double *)c->wp(c->off.mlp) : nullptr;
    if (c->es == 8)
        hipLaunchKernelGGL((k_mlp_forward<double>), dim3(nblk), dim3(256), 0, c->stream, (const float *)c->mlp_bf16,
                           (const float *)x, c->nc, (float *)nullptr, (double *)c->wp(c->off.nu), fb, vmax);
    else
        hipLaunchKernelGGL((k_mlp_forward<float>), dim3(nblk), dim3(256), 0, c->stream, (const float *)c->mlp_bf16,
                           (const float *)x, c->nc, (float *)nullptr, (float *)c->wp(c->off.nu), fb, vmax);
    LAUNCHCHK(c);
    if (nvmax) *nvmax = nblk;
    c->have_nu = true;
    return DG_OK;
}

int dg_sensor_infer(dg_ctx *c, const void *u)
{
    if (!c) return DG_EINVAL;
    c->spec_valid = false;          // the viscosity or flags a launched next stage used change
    if (int rc = dg_check_array(c, u, dg_state_bytes(c), c->es, "u")) return rc;
    return sensor_infer_impl(c, u);
}

int dg_sensor_judge(dg_ctx *c, const void *u, double tau, long *nfallback)
{
    if (!c) return DG_EINVAL;
    c->spec_valid = false;          // the viscosity or flags a launched next stage used change
    if (!u || !(tau >= 0.0)) return dg_fail(c, DG_EINVAL, "bad judge arguments");
    if (int rc = dg_check_array(c, u, dg_state_bytes(c), c->es, "u")) return rc;
    int rc = sensor_infer_impl(c, u);
    if (rc) return rc;
    double *lab = (double *)c->wp(c->off.lab);
    rc = dg_sensor_labels(c, u, lab);
    if (rc) return rc;
    unsigned long long *cnt = (unsigned long long *)(c->scal() + 32);
    std::memset(c->pinned + 8, 0, 8);
    HIPCHK(c, hipMemcpyAsync(cnt, c->pinned + 8, 8, hipMemcpyHostToDevice, c->stream));
    int *fb = (int *)c->wp(c->off.fb);
    if (c->es == 8)
        hipLaunchKernelGGL((k_judge<double>), dim3(c->nblk), dim3(BLOCK), 0, c->stream,
                           (const double *)c->wp(c->off.nu), (const double *)lab, c->nc, tau, fb, cnt);
    else
        hipLaunchKernelGGL((k_judge<float>), dim3(c->nblk), dim3(BLOCK), 0, c->stream,
                           (const float *)c->wp(c->off.nu), (const double *)lab, c->nc, tau, fb, cnt);
    LAUNCHCHK(c);
    HIPCHK(c, hipMemcpyAsync(c->pinned, cnt, 8, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if (nfallback) *nfallback = (long)((volatile unsigned long long *)c->pinned)[0];
    return DG_OK;
}

int dg_sensor_set_nu(dg_ctx *c, const void *nu, const int32_t *fb)
{
    if (!c) return DG_EINVAL;
    c->spec_valid = false;          // the viscosity or flags a launched next stage used change
    int rc = need_k2(c);
    if (rc) return rc;
    if (nu && (rc = dg_check_array(c, nu, c->es * (size_t)c->nc, c->es, "nu"))) return rc;
    if (fb && (rc = dg_check_array(c, fb, 4 * (size_t)c->nc, 4, "fallback"))) return rc;
    if (nu) {
        HIPCHK(c, hipMemcpyAsync(c->wp(c->off.nu), nu, c->es * (size_t)c->nc, hipMemcpyDeviceToDevice, c->stream));
        c->have_nu = true;
    }
    if (fb) HIPCHK(c, hipMemcpyAsync(c->wp(c->off.fb), fb, 4 * (size_t)c->nc, hipMemcpyDeviceToDevice, c->stream));
    return DG_OK;
}

// clear the fallback flags of a fresh workspace (every cell starts on the learned sensor)
int sensor_reset_flags(dg_ctx *c)
{
    hipLaunchKernelGGL(k_fill_int, dim3(c->nblk), dim3(BLOCK), 0, c->stream, (int *)c->wp(c->off.fb), c->nc, 0);
    LAUNCHCHK(c);
    return DG_OK;
}
