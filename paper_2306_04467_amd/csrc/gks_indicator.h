// Learned smoothness indicator: a small MLP (44 -> 64 -> 64 -> 1, ReLU) predicts from a cell's
// compact stencil whether the nonlinear weights of the reconstruction may be skipped (the linear
// P^3 reconstruction is then used, which the nonlinear one reproduces on smooth data).
//
//   features  per cell, for the interface level eta1 = h1 + B and then h2: the 9 stencil differences
//             (Q_l - Q_0)/s and the 8 scaled gradients hs grad Q_l / s of the cell and its face
//             neighbours, s = max_l |Q_l - Q_0| + 1e-12 |Q_0|; the size of the variation,
//             log10(s / h)/4, and of the layer's momentum variation against h sqrt(G h); then the
//             face neighbours' area ratios and the cell's edge lengths over hs (static, from the mesh)
//   inference BF16 MFMA (v_mfma_f32_32x32x16_bf16), FP32 accumulation, 32 cells per wave; the
//             44 inputs are padded with zeros to 48 (three K-steps of 16)
//   training  FP32 on the matrix cores: tiles of 32 samples forward, backward and into block-wise
//             weight-gradient sums, added in a fixed order (deterministic) by the Adam step
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gks_kernels.h"
#include "gks_mlp.h"

namespace gks {

// Features of field f of cell c (f = 0: eta1 with the lower layer's momenta, f = 1: h2 with the
// upper layer's): x[0..16] the stencil differences and scaled gradients, x[17] the size of the
// variation, x[18] the size of the momentum variation.  Computed from the reconstruction's own
// right-hand sides, with the arithmetic of the reconstruction kernel's fused indicator.
template <typename R>
__device__ inline void field_features(const MeshDev &m, double G, const LayerW<R> *__restrict__ W,
                                      const LayerG<R> *__restrict__ gW, int f, int64_t c, float *x)
{
    double Q0h;
    R rhs[3][17];
    recon_rhs<R>(m, W, gW, 1 - f, c, Q0h, rhs);
    const double h = f == 0 ? Q0h - m.Bbar[c] : Q0h;
    thick_features<R>(rhs[0], Q0h, h, x);
    x[18] = mom_feature(fmax(max_diff<R>(rhs[1]), max_diff<R>(rhs[2])), h, G);
}

// all 44 features of cell c (training export), 256 threads a block: without the bound the compiler keeps to
// the 128 registers of a block of 1024, and the three variables' right-hand sides spill in FP64
template <typename R>
__global__ void __launch_bounds__(256) k_features(MeshDev m, double G, const LayerW<R> *__restrict__ W,
                           const LayerG<R> *__restrict__ gW, float *__restrict__ X)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= m.T) return;
    float *x = X + c * MLP_IN;
#pragma unroll
    for (int f = 0; f < 2; f++) {
        float y[19];
        field_features<R>(m, G, W, gW, f, c, y);
#pragma unroll
        for (int k = 0; k < 17; k++) x[17 * f + k] = y[k];
        x[34 + f] = y[17];
        x[36 + f] = y[18];
    }
#pragma unroll
    for (int k = 0; k < 6; k++) x[38 + k] = m.igeo[k * m.T + c];
}

// ---------------------------------------------------------------------------------------------
// inference: 4 waves per block, one wave per 32 cells (the network itself is in gks_mlp.h)

// W1b, W2b: the weight matrices in operand order (k_weights_bf16); P: FP32 parameters (biases and
// the output layer).
// Writes mask[c] = (logit > thr) and, when logit is not null, the logit.
template <typename R>
__global__ void __launch_bounds__(64 * IND_WAVES) k_indicator(MeshDev m, double G, const LayerW<R> *__restrict__ W,
                                                               const LayerG<R> *__restrict__ gW,
                                                               const short *__restrict__ W1b,
                                                               const short *__restrict__ W2b,
                                                               const float *__restrict__ P, float thr,
                                                               uint8_t *__restrict__ mask, float *__restrict__ logit)
{
    __shared__ __align__(16) short feat[IND_WAVES][32][FB];
    __shared__ __align__(16) short hid[IND_WAVES][32][HB];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, row = lane & 31, half = lane >> 5;
    const int64_t T = m.T;
    const int64_t base = ((int64_t)blockIdx.x * IND_WAVES + wv) * 32;
    const int64_t c = base + row;
    // features: lanes 0..31 the interface level (and the geometry), lanes 32..63 h2 (and the
    // zero padding of the inputs)
    {
        float x[19];
        if (c < T) {
            field_features<R>(m, G, W, gW, half, c, x);
        } else {
#pragma unroll
            for (int k = 0; k < 19; k++) x[k] = 0.f;
        }
#pragma unroll
        for (int k = 0; k < 17; k++) feat[wv][row][17 * half + k] = to_bf16(x[k]);
        feat[wv][row][34 + half] = to_bf16(x[17]);
        feat[wv][row][36 + half] = to_bf16(x[18]);
        if (!half) {
#pragma unroll
            for (int k = 0; k < 6; k++) feat[wv][row][38 + k] = to_bf16(c < T ? m.igeo[k * T + c] : 0.f);
        } else {
#pragma unroll
            for (int k = MLP_IN; k < MLP_K; k++) feat[wv][row][k] = 0;
        }
    }
    __syncthreads();
    mlp_layer1(feat[wv], hid[wv], lane, 0, W1b, P);
    mlp_layer1(feat[wv], hid[wv], lane, 1, W1b, P);
    __syncthreads();
    float z[16];
    mlp_layer2_out(hid[wv], lane, W2b, P, z);
    if (row == 0) {
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const int64_t ci = base + 8 * (r / 4) + 4 * half + (r % 4);
            if (ci < T) {
                mask[ci] = z[r] > thr ? 1 : 0;
                if (logit) logit[ci] = z[r];
            }
        }
    }
}

// the same network on stored feature rows X[n][44] (threshold selection on training samples)
__global__ void __launch_bounds__(64 * IND_WAVES) k_mlp_infer(const float *__restrict__ X, int64_t n,
                                                               const short *__restrict__ W1b,
                                                               const short *__restrict__ W2b,
                                                               const float *__restrict__ P, float *__restrict__ logit)
{
    __shared__ __align__(16) short feat[IND_WAVES][32][FB];
    __shared__ __align__(16) short hid[IND_WAVES][32][HB];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, row = lane & 31, half = lane >> 5;
    const int64_t base = ((int64_t)blockIdx.x * IND_WAVES + wv) * 32;
    for (int k = half; k < MLP_K; k += 2)
        feat[wv][row][k] = to_bf16((base + row < n && k < MLP_IN) ? X[(base + row) * MLP_IN + k] : 0.f);
    __syncthreads();
    mlp_layer1(feat[wv], hid[wv], lane, 0, W1b, P);
    mlp_layer1(feat[wv], hid[wv], lane, 1, W1b, P);
    __syncthreads();
    float z[16];
    mlp_layer2_out(hid[wv], lane, W2b, P, z);
    if (row == 0) {
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const int64_t i = base + 8 * (r / 4) + 4 * half + (r % 4);
            if (i < n) logit[i] = z[r];
        }
    }
}

// ---------------------------------------------------------------------------------------------
// labels: 1 where the nonlinear and the linear reconstructions agree at every Gauss point within
// tol times the variable's scale (layer thickness, or h sqrt(G h) for momenta)

template <typename R>
__global__ void k_label(MeshDev m, double G, double tol, const LayerW<R> *__restrict__ W,
                        const GpHead<R> *__restrict__ rec_nl, const GpHead<R> *__restrict__ rec_li, uint8_t *__restrict__ y)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= m.T) return;
    const double h2 = W[2 * c].h, h1 = W[2 * c + 1].h - m.Bbar[c];
    const double sh[2] = {h2, h1}, sm[2] = {h2 * sqrt(G * h2), h1 * sqrt(G * h1)};
    bool ok = true;
    for (int slot = 0; slot < 6; slot++) {
        const int64_t at = rec_at(m.T, c, slot / 2, slot % 2);
        const GpHead<R> &a = rec_nl[at], &b = rec_li[at];
        for (int q = 0; q < 2; q++) ok = ok && fabs(a.h[q] - b.h[q]) <= tol * sh[q];
        for (int q = 0; q < 4; q++) ok = ok && fabs((double)a.q[q] - (double)b.q[q]) <= tol * sm[q / 2];
    }
    y[c] = ok ? 1 : 0;
}

__global__ void k_u8_to_f32(const uint8_t *__restrict__ a, int64_t n, float *__restrict__ b)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = (float)a[i];
}

// ---------------------------------------------------------------------------------------------
// training (FP32)

constexpr int TRAIN_TILE = 32;          // samples a block takes through the network at a time
constexpr int TRAIN_MAX_BLOCKS = 512;   // a larger batch loops over its tiles (bounds the partial sums)
// LDS row strides of the tile's matrices: multiples of 4 whose sixteen first multiples are distinct
// modulo the 64 banks, so that a 16 x 4 matrix-core operand (row * stride + 0..3) is conflict free
constexpr int TX = 52, TH = MLP_H + 4;

typedef float f32x4 __attribute__((ext_vector_type(4)));

// acc[r] += A[i][k] B[k][j] over k = 0 .. 4 steps - 1 on one wave (v_mfma_f32_16x16x4_f32: lane l
// supplies A row l % 16 and B column l % 16 at k = 4 step + l / 16, register r holds row
// 4 (l / 16) + r, column l % 16).  Element strides: A (ai, ak), B (bk, bj).
__device__ inline f32x4 tile_product(const float *A, int ai, int ak, const float *Bm, int bk, int bj, int steps,
                                     int lane, f32x4 acc)
{
    const int i = lane & 15, k = lane >> 4;
    A += i * ai + k * ak;
    Bm += i * bj + k * bk;
    for (int s = 0; s < steps; s++) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(A[4 * s * ak], Bm[4 * s * bk], acc, 0, 0, 0);
    return acc;
}

// One minibatch (rows idx[0 .. B) of X, Y): forward pass, logistic loss, back-propagation and the
// weight gradients of the mean loss, tile by tile of 32 samples held in LDS; each block leaves its
// sums over its tiles in part[block][MLP_NP] and its loss sum in lpart[block], and k_mlp_reduce
// adds the blocks in order (no atomics, the same bits every time).  All products run on the matrix
// cores in FP32, column block w of every matrix on wave w.
// What bounds it: a batch of 2048 is 86 MFLOP on 64 blocks, about 2 us of matrix work a block, so
// launch and memory latency: with the weights, the indices, the rows and the labels read one after the
// other 19.5 us a batch of 2048, 11.3 with all of it under way at once.  One thread per parameter summing the batch serially (111 waves on the whole chip)
// and a forward pass on 16 blocks took 526 + 79 us for 2048 samples.
__global__ void __launch_bounds__(256) k_mlp_batch(const float *__restrict__ P, const float *__restrict__ X,
                                                   const float *__restrict__ Y, const int32_t *__restrict__ idx, int B,
                                                   float *__restrict__ part, float *__restrict__ lpart)
{
    __shared__ alignas(16) float w1[MLP_IN * TH], w2[MLP_H * TH], xs[TRAIN_TILE * TX];
    __shared__ float b1[MLP_H], b2[MLP_H], w3[MLP_H];
    __shared__ float h1[TRAIN_TILE * TH], h2[TRAIN_TILE * TH], d1[TRAIN_TILE * TH],
        d2[TRAIN_TILE * TH], dz[TRAIN_TILE], ls[TRAIN_TILE];
    const int t = threadIdx.x, w = t >> 6, lane = t & 63, j0 = 16 * w;
    const int col = lane & 15, row4 = 4 * (lane >> 4);
    // everything the block reads is under way before any of it is stored: the tile's rows and labels (whose
    // indices come first) and the weights, in 16-byte words
    constexpr int XV = TRAIN_TILE * 12, V1 = MLP_IN * MLP_H / 4, V2 = MLP_H * MLP_H / 4;  // words (12 a row, the last 0)
    static_assert(MLP_IN % 4 == 0 && MLP_H % 4 == 0 && OFF_W2 % 4 == 0 && TX % 4 == 0 && TH % 4 == 0, "16-byte words");
    f32x4 xv[(XV + 255) / 256];
    float yv = 0.f;
    auto load_tile = [&](int tile) {
        const int s0 = tile * TRAIN_TILE, ns = B - s0 < TRAIN_TILE ? B - s0 : TRAIN_TILE;
        int row[(XV + 255) / 256];
#pragma unroll
        for (int j = 0; j < (XV + 255) / 256; j++) {
            const int r = (t + 256 * j) / 12, k = (t + 256 * j) % 12;
            row[j] = r < ns && k < MLP_IN / 4 ? idx[s0 + r] : -1;
        }
        const int ry = (t >> 3) < ns ? idx[s0 + (t >> 3)] : -1;
#pragma unroll
        for (int j = 0; j < (XV + 255) / 256; j++)
            xv[j] = row[j] >= 0 ? reinterpret_cast<const f32x4 *>(X + (int64_t)row[j] * MLP_IN)[(t + 256 * j) % 12] : f32x4{0};
        yv = ry >= 0 ? Y[ry] : 0.f;
    };
    f32x4 v1[(V1 + 255) / 256], v2[V2 / 256];
#pragma unroll
    for (int j = 0; j < (V1 + 255) / 256; j++)
        if (t + 256 * j < V1) v1[j] = reinterpret_cast<const f32x4 *>(P)[t + 256 * j];
#pragma unroll
    for (int j = 0; j < V2 / 256; j++) v2[j] = reinterpret_cast<const f32x4 *>(P + OFF_W2)[t + 256 * j];
    const float b3 = P[OFF_B3];
    const float p1 = P[OFF_B1 + (t & 63)], p2 = P[OFF_B2 + (t & 63)], p3 = P[OFF_W3 + (t & 63)];
    load_tile(blockIdx.x);
#pragma unroll
    for (int j = 0; j < (V1 + 255) / 256; j++) {
        const int i = t + 256 * j;
        if (i < V1) *reinterpret_cast<f32x4 *>(w1 + (i / (MLP_H / 4)) * TH + 4 * (i % (MLP_H / 4))) = v1[j];
    }
#pragma unroll
    for (int j = 0; j < V2 / 256; j++) {
        const int i = t + 256 * j;
        *reinterpret_cast<f32x4 *>(w2 + (i / (MLP_H / 4)) * TH + 4 * (i % (MLP_H / 4))) = v2[j];
    }
    if (t < MLP_H) {
        b1[t] = p1;
        b2[t] = p2;
        w3[t] = p3;
    }
    f32x4 g1[3] = {}, g2[4] = {};  // column block w of dW1 (44 rows padded to 48) and dW2
    float gb = 0.f;                // threads 0..63 db1, 64..127 db2, 128..191 dw3, 192 db3, 193 the loss
    for (int tile = blockIdx.x; tile * TRAIN_TILE < B; tile += gridDim.x) {
        const int s0 = tile * TRAIN_TILE, ns = B - s0 < TRAIN_TILE ? B - s0 : TRAIN_TILE;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < (XV + 255) / 256; j++) {
            const int i = t + 256 * j;
            if (i < XV) *reinterpret_cast<f32x4 *>(xs + (i / 12) * TX + 4 * (i % 12)) = xv[j];
        }
        const float y = yv;
        if ((tile + gridDim.x) * TRAIN_TILE < B) load_tile(tile + gridDim.x);
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < 2; rb++) {
            const f32x4 a = tile_product(xs + 16 * rb * TX, TX, 1, w1 + j0, TH, 1, MLP_IN / 4, lane, f32x4{0});
#pragma unroll
            for (int r = 0; r < 4; r++) h1[(16 * rb + row4 + r) * TH + j0 + col] = fmaxf(a[r] + b1[j0 + col], 0.f);
        }
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < 2; rb++) {
            const f32x4 a = tile_product(h1 + 16 * rb * TH, TH, 1, w2 + j0, TH, 1, MLP_H / 4, lane, f32x4{0});
#pragma unroll
            for (int r = 0; r < 4; r++) h2[(16 * rb + row4 + r) * TH + j0 + col] = fmaxf(a[r] + b2[j0 + col], 0.f);
        }
        __syncthreads();
        {  // output unit: eight threads a sample
            const int s = t >> 3, q = t & 7;
            float z = 0.f;
#pragma unroll
            for (int k = 0; k < 8; k++) z = fmaf(h2[s * TH + 8 * k + q], w3[8 * k + q], z);
            z += __shfl_xor(z, 1);
            z += __shfl_xor(z, 2);
            z += __shfl_xor(z, 4);
            z += b3;
            // softplus(z) - y z, evaluated without overflow
            const float L = fmaxf(z, 0.f) + log1pf(expf(-fabsf(z))) - y * z;
            const float e = s < ns ? (1.f / (1.f + expf(-z)) - y) / (float)B : 0.f;
            if (q == 0) {
                dz[s] = e;
                ls[s] = s < ns ? L : 0.f;
            }
#pragma unroll
            for (int k = 0; k < 8; k++) {
                const int j = 8 * k + q;
                d2[s * TH + j] = h2[s * TH + j] > 0.f ? e * w3[j] : 0.f;
            }
        }
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < 2; rb++) {  // D2 W2^T
            const f32x4 a = tile_product(d2 + 16 * rb * TH, TH, 1, w2 + j0 * TH, 1, TH, MLP_H / 4, lane, f32x4{0});
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int i = (16 * rb + row4 + r) * TH + j0 + col;
                d1[i] = h1[i] > 0.f ? a[r] : 0.f;
            }
        }
        __syncthreads();
#pragma unroll
        for (int rb = 0; rb < 3; rb++)
            g1[rb] = tile_product(xs + 16 * rb, 1, TX, d1 + j0, TH, 1, TRAIN_TILE / 4, lane, g1[rb]);
#pragma unroll
        for (int rb = 0; rb < 4; rb++)
            g2[rb] = tile_product(h1 + 16 * rb, 1, TH, d2 + j0, TH, 1, TRAIN_TILE / 4, lane, g2[rb]);
        if (t < 192) {
            const int j = t & 63;
            for (int s = 0; s < TRAIN_TILE; s++)
                gb += t < 64 ? d1[s * TH + j] : t < 128 ? d2[s * TH + j] : dz[s] * h2[s * TH + j];
        } else if (t < 194) {
            for (int s = 0; s < TRAIN_TILE; s++) gb += t == 192 ? dz[s] : ls[s];
        }
    }
    float *g = part + (int64_t)blockIdx.x * MLP_NP;
#pragma unroll
    for (int rb = 0; rb < 3; rb++)
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int i = 16 * rb + row4 + r;
            if (i < MLP_IN) g[i * MLP_H + j0 + col] = g1[rb][r];
        }
#pragma unroll
    for (int rb = 0; rb < 4; rb++)
#pragma unroll
        for (int r = 0; r < 4; r++) g[OFF_W2 + (16 * rb + row4 + r) * MLP_H + j0 + col] = g2[rb][r];
    if (t < 193) g[t < 64 ? OFF_B1 + t : t < 128 ? OFF_B2 + t - 64 : t < 192 ? OFF_W3 + t - 128 : OFF_B3] = gb;
    if (t == 193) lpart[blockIdx.x] = gb;
}

struct AdamArgs {
    float *P, *mo, *ve;
    float lr, b1, b2, eps, c1, c2;  // c1, c2: 1 - b1^t, 1 - b2^t
};

// the blocks' partial sums in a fixed order: the mean loss, and the gradient (grad not null) or the
// Adam step with it.  One thread per parameter, thread MLP_NP the loss.
// Bound by latency: 64 blocks' sums with 8 reads under way 5.1 us, with 32 3.9.
__global__ void __launch_bounds__(64) k_mlp_reduce(const float *__restrict__ part, const float *__restrict__ lpart, int nb,
                                                   int B, float *__restrict__ loss, float *__restrict__ grad, AdamArgs o)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p > MLP_NP) return;
    const float *q = p < MLP_NP ? part + p : lpart;
    const int64_t st = p < MLP_NP ? MLP_NP : 1;
    float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int b = 0;
    for (; b + 32 <= nb; b += 32) {  // 32 reads ahead of their sums
        float x[32];
#pragma unroll
        for (int k = 0; k < 32; k++) x[k] = q[(b + k) * st];
#pragma unroll
        for (int k = 0; k < 32; k++) s[k & 7] += x[k];
    }
    for (; b + 8 <= nb; b += 8)
#pragma unroll
        for (int k = 0; k < 8; k++) s[k] += q[(b + k) * st];
    for (; b < nb; b++) s[0] += q[b * st];
    const float g = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    if (p == MLP_NP) {
        loss[0] = g / (float)B;
        return;
    }
    if (grad) {
        grad[p] = g;
        return;
    }
    const float m = o.b1 * o.mo[p] + (1.f - o.b1) * g;
    const float v = o.b2 * o.ve[p] + (1.f - o.b2) * g * g;
    o.mo[p] = m;
    o.ve[p] = v;
    o.P[p] -= o.lr * (m / o.c1) / (sqrtf(v / o.c2) + o.eps);
}

}  // namespace gks
