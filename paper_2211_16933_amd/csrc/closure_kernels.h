// Device kernels of the learned closure (gfx950): the MLP 12 -> 64 -> 64 -> 64 -> Q_s with
// SiLU on bfloat16 matrix cores (v_mfma_f32_16x16x32_bf16, FP32 accumulation), its
// backward pass and Adam, and the per-cell closure: moments of every row, the 12 inputs,
// the correction added to the student's L[phi], and the training samples.  Included by
// elb.hip only.  The parameter layout and the normalisation block are those of
// mlp_device.h.  The stage kernel carries a fused form of k_closure_rows and
// k_closure_apply (elb_set_closure with enabled = 1); these two kernels are the separate
// form (enabled = 2).
#pragma once
#include <hip/hip_runtime.h>

#include "elb_kernels.h"
#include "mlp_device.h"
#include "state_kernels.h"

namespace elb {

// acc[t] (t < NT) = A[16][K] x B^T for the 16-column block t of B, where A is a bf16 tile
// with row stride as and B is [N][K] bf16 with row stride bs (both in LDS).  Operand lane
// layout of v_mfma_f32_16x16x32_bf16: lane l holds A[l % 16][8 (l / 16) + i] and
// B[8 (l / 16) + i][l % 16], i < 8; the result D[4 (l / 16) + r][l % 16] sits in acc[r].
template <int K, int NT>
__device__ inline void mma_rows16(const unsigned short *A, int as, const unsigned short *B, int bs,
                                  floatx4 acc[NT], int lane)
{
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int r = lane & 15, kq = 8 * (lane >> 4);
#pragma unroll
    for (int kk = 0; kk < K / 32; ++kk) {
        bf16x8 a = ld8(A + r * as + kk * 32 + kq);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            bf16x8 b = ld8(B + (t * 16 + r) * bs + kk * 32 + kq);
            acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[t], 0, 0, 0);
        }
    }
}

// Weights of the forward pass in LDS (bf16) and the biases (FP32).
struct alignas(16) MlpSmem {
    unsigned short w1[MLP_H * WS1];
    unsigned short w2[MLP_H * WSH];
    unsigned short w3[MLP_H * WSH];
    unsigned short w4[MLP_OUT * WSH];
    float bias[3 * MLP_H + MLP_OUT];
    unsigned short act[4][2][16 * AS];   // per wave: two activation tiles (ping-pong)
};

__device__ inline void mlp_stage_weights(MlpSmem &s, const unsigned short *wb, const float *params)
{
    for (int j = threadIdx.x; j < MLP_H * MLP_K1; j += blockDim.x)
        s.w1[(j / MLP_K1) * WS1 + j % MLP_K1] = wb[OFF_W1 + j];
    for (int j = threadIdx.x; j < MLP_H * MLP_H; j += blockDim.x) {
        s.w2[(j / MLP_H) * WSH + j % MLP_H] = wb[OFF_W2 + j];
        s.w3[(j / MLP_H) * WSH + j % MLP_H] = wb[OFF_W3 + j];
    }
    for (int j = threadIdx.x; j < MLP_OUT * MLP_H; j += blockDim.x)
        s.w4[(j / MLP_H) * WSH + j % MLP_H] = wb[OFF_W4 + j];
    for (int j = threadIdx.x; j < MLP_H; j += blockDim.x) {
        s.bias[j] = params[OFF_B1 + j];
        s.bias[MLP_H + j] = params[OFF_B2 + j];
        s.bias[2 * MLP_H + j] = params[OFF_B3 + j];
    }
    for (int j = threadIdx.x; j < MLP_OUT; j += blockDim.x) s.bias[3 * MLP_H + j] = params[OFF_B4 + j];
}

// Forward pass of the 16 rows whose bf16 inputs are in s.act[wave][0] (columns 0..31).
// Output y[16][16] (FP32) in the D layout of acc4.  Every wave of the block must call this (it
// synchronises the block between layers).
__device__ inline void mlp_forward_rows(MlpSmem &s, int wave, int lane, floatx4 &acc4)
{
    unsigned short *a0 = s.act[wave][0], *a1 = s.act[wave][1];
    floatx4 acc[4];
    const int col = lane & 15, rq = 4 * (lane >> 4);
    // layer 1: K = 32
    mma_rows16<MLP_K1, 4>(a0, AS, s.w1, WS1, acc, lane);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = rq + r, c = t * 16 + col;
            a1[row * AS + c] = f2bf(silu(acc[t][r] + s.bias[c]));
        }
    __syncthreads();
    // layers 2 and 3: K = 64
#pragma unroll
    for (int l = 0; l < 2; ++l) {
        const unsigned short *ain = l == 0 ? a1 : a0;
        unsigned short *aout = l == 0 ? a0 : a1;
        mma_rows16<MLP_H, 4>(ain, AS, l == 0 ? s.w2 : s.w3, WSH, acc, lane);
        __syncthreads();  // every lane has read ain / may overwrite aout (aliases a0 at l = 0)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = rq + r, c = t * 16 + col;
                aout[row * AS + c] = f2bf(silu(acc[t][r] + s.bias[(l + 1) * MLP_H + c]));
            }
        __syncthreads();
    }
    // layer 4: 16 outputs
    floatx4 o[1];
    mma_rows16<MLP_H, 1>(a1, AS, s.w4, WSH, o, lane);
#pragma unroll
    for (int r = 0; r < 4; ++r) o[0][r] += s.bias[3 * MLP_H + col];
    acc4 = o[0];
}

// --------------------------------------------------------------------------------------
// Training.  A minibatch of a few thousand rows is too small to fill the chip, so its kernels
// are bound by latency, and each is cut into as many short blocks as the shapes give: 16 rows
// per block forward and backward, the 64 columns of a layer spread over four waves, every
// weight a wave needs loaded from L2 at the start (no staging in LDS); weight gradients by
// (128-row chunk, layer), from operands that the backward kernel leaves in the layout the matrix
// cores read.  Batch 4096, us per launch before (64 rows per block with staged weights; gradients
// one block per chunk, transposing through LDS) and now: forward 17.8 / 5.4, backward 17.3 / 8.6,
// weight gradients 75.6 / 5.6, reduction 8.6 / 3.2.
//
// From about 2e5 rows on, the forward is bound by what it writes, 830 bytes per row (mostly the
// pre-activations, which stay FP32).  It is also all that an evaluation runs, so the transposed
// operands, another 450 bytes, are left to the backward kernel, which has the pre-activations in
// hand: 1048576 rows 325 us (625 with them in the forward, 2-byte stores 256 bytes apart; 365
// before), 4194304 rows 1241 (2638; 1407).  Backward and gradients there: 1.9 ms (5.7), 7.8 (22.6).
// --------------------------------------------------------------------------------------
constexpr int TRAIN_ROWS = 16;  // batch rows per block, forward and backward

// Transposed bf16 operands, by chunks of WGRAD_ROWS rows: [chunk][column][WGRAD_ROWS]; the
// place of (row b, column c) of a matrix of `cols` columns.
__device__ inline size_t chunk_at(int b, int c, int cols)
{
    return ((size_t)(b / WGRAD_ROWS) * cols + c) * WGRAD_ROWS + b % WGRAD_ROWS;
}

// Training forward: rows b < batch of x[index[b]] (or x[b]), normalised, through the MLP.
// y [batch][16] (normalised outputs).  Kept for the backward pass: z [3][batch][64]
// pre-activations and the bf16 inputs a0 [batch][32].  A block takes `tiles` tiles of 16 rows one
// after another with its weights in registers (forward_tiles).
__global__ __launch_bounds__(256) void k_mlp_forward(const unsigned short *wb, const float *params,
                                                     const float *norm, const float *x,
                                                     const int *index, int batch, int tiles, float *y,
                                                     unsigned short *a0, float *z)
{
    __shared__ __attribute__((aligned(16))) unsigned short act[2][TRAIN_ROWS * AS];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int col = lane & 15, rq = 4 * (lane >> 4), kq = 8 * (lane >> 4);
    const int c = wave * 16 + col;  // this lane's output column of the hidden layers
    const bf16x8 w1 = ld8(wb + OFF_W1 + c * MLP_K1 + kq);
    bf16x8 w2[2], w3[2], w4[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
        w2[kk] = ld8(wb + OFF_W2 + c * MLP_H + kk * 32 + kq);
        w3[kk] = ld8(wb + OFF_W3 + c * MLP_H + kk * 32 + kq);
        w4[kk] = ld8(wb + OFF_W4 + col * MLP_H + kk * 32 + kq);
    }
    const float bias[3] = {params[OFF_B1 + c], params[OFF_B2 + c], params[OFF_B3 + c]};
    const float bias4 = params[OFF_B4 + col];
    const size_t zstride = (size_t)batch * MLP_H;
    const int end = (int)min((long long)batch, ((long long)blockIdx.x + 1) * tiles * TRAIN_ROWS);
    for (int row0 = blockIdx.x * tiles * TRAIN_ROWS; row0 < end; row0 += TRAIN_ROWS) {
        // inputs: 16 rows of 32 columns, two neighbours per thread.  act[0] is free: what the tile
        // before read from it was read before its last barrier
        {
            const int r = threadIdx.x >> 4, k = 2 * (threadIdx.x & 15), b = row0 + r;
            ushort2 h = {0, 0};
            if (b < batch && k < MLP_IN) {
                const float *xr = x + (size_t)(index ? index[b] : b) * MLP_IN;
                h.x = f2bf((xr[k] - norm[NRM_IN_MEAN + k]) / norm[NRM_IN_STD + k]);
                h.y = f2bf((xr[k + 1] - norm[NRM_IN_MEAN + k + 1]) / norm[NRM_IN_STD + k + 1]);
            }
            *reinterpret_cast<ushort2 *>(act[0] + r * AS + k) = h;
            if (b < batch) *reinterpret_cast<ushort2 *>(a0 + (size_t)b * MLP_K1 + k) = h;
        }
        __syncthreads();
        floatx4 acc =
            __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(act[0] + col * AS + kq), w1, floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
        for (int l = 0; l < 3; ++l) {
            unsigned short *out = act[(l + 1) & 1];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float zz = acc[r] + bias[l];
                if (row0 + rq + r < batch) z[l * zstride + (size_t)(row0 + rq + r) * MLP_H + c] = zz;
                out[(rq + r) * AS + c] = f2bf(silu(zz));
            }
            __syncthreads();
            if (l == 2 && wave > 0) continue;  // 16 outputs: one wave
            const bf16x8 *w = l == 0 ? w2 : l == 1 ? w3 : w4;
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(out + col * AS + kq), w[0], floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(out + col * AS + 32 + kq), w[1], acc, 0, 0, 0);
        }
        if (wave == 0)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (row0 + rq + r < batch) y[(size_t)(row0 + rq + r) * MLP_OUT + col] = acc[r] + bias4;
    }
}

// Loss mean((y - t_norm)^2) over batch x q_out and its gradient dy (zero on padded outputs);
// t_norm = (t[index[b]] - out_mean) / out_std.  Per-block partial sums of the loss go to
// part[blockIdx.x] (summed by k_sum_partials).
__global__ __launch_bounds__(256) void k_mlp_loss(const float *y, const float *t, const int *index,
                                                  const float *norm, int batch, int q_out, float *dy,
                                                  double *part)
{
    __shared__ double red[256];
    double acc = 0.0;
    const double scale = 2.0 / ((double)batch * q_out);
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < batch * MLP_OUT; j += gridDim.x * blockDim.x) {
        const int b = j / MLP_OUT, o = j - b * MLP_OUT;
        float g = 0.f;
        if (o < q_out) {
            const int src = index ? index[b] : b;
            float tn = (t[(size_t)src * q_out + o] - norm[NRM_OUT_MEAN + o]) / norm[NRM_OUT_STD + o];
            float d = y[j] - tn;
            acc += (double)d * d;
            g = (float)(scale * d);
        }
        dy[j] = g;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// *out = scale * sum of n <= 256 partial sums, added in order; the loads are spread over the
// block first (one thread walking them in memory took 13 us).
__global__ __launch_bounds__(256) void k_sum_partials(const double *part, int n, double scale, double *out)
{
    __shared__ double sh[256];
    sh[threadIdx.x] = (int)threadIdx.x < n ? part[threadIdx.x] : 0.0;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
#pragma unroll 16
        for (int i = 0; i < n; ++i) s += sh[i];
        *out = s * scale;
    }
}

// Backward pass, per row: dz4 = dy; da_l = bf16(dz_{l+1}) W_{l+1}; dz_l = da_l SiLU'(z_l).
// dz [3][batch][64] (layers 1..3, FP32, for the bias gradients), and transposed by chunk in
// bf16 gt (64 columns, layers 1..3, tstride apart) and g4t (16 columns, dy), and the layer inputs
// at (64 columns, layers 2..4, tstride apart) and a0t (32 columns).
__global__ __launch_bounds__(256) void k_mlp_backward(const unsigned short *wb, const float *dy,
                                                      const float *z, const unsigned short *a0, int batch, float *dz,
                                                      unsigned short *gt, unsigned short *at, size_t tstride,
                                                      unsigned short *g4t, unsigned short *a0t)
{
    __shared__ __attribute__((aligned(16))) unsigned short act[2][TRAIN_ROWS * AS];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int row0 = blockIdx.x * TRAIN_ROWS;
    const int nvalid = batch - row0;
    const int col = lane & 15, rq = 4 * (lane >> 4), kq = 8 * (lane >> 4);
    const int c = wave * 16 + col;  // this lane's column (an input of layer l + 1)
    const size_t lstride = (size_t)batch * MLP_H;
    // W_{l+1} as B operands (row k of W is output k): layer 4 has 16 outputs, so only the lanes
    // of k < 16 hold any
    ushort8 w4 = {0, 0, 0, 0, 0, 0, 0, 0}, w3[2], w2[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (kq < MLP_OUT) w4[i] = wb[OFF_W4 + (kq + i) * MLP_H + c];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            w3[kk][i] = wb[OFF_W3 + (kk * 32 + kq + i) * MLP_H + c];
            w2[kk][i] = wb[OFF_W2 + (kk * 32 + kq + i) * MLP_H + c];
        }
    }
    float zv[3][4];
#pragma unroll
    for (int l = 0; l < 3; ++l)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            zv[l][r] = rq + r < nvalid ? z[l * lstride + (size_t)(row0 + rq + r) * MLP_H + c] : 0.f;
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        ushort4 h4;
        unsigned short *h = reinterpret_cast<unsigned short *>(&h4);
#pragma unroll
        for (int r = 0; r < 4; ++r) h[r] = f2bf(silu(zv[l][r]));
        *reinterpret_cast<ushort4 *>(at + l * tstride + chunk_at(row0 + rq, c, MLP_H)) = h4;
    }
    if (threadIdx.x < MLP_K1 * TRAIN_ROWS / 4) {  // four rows of a column
        const int k = threadIdx.x % MLP_K1, r0 = threadIdx.x / MLP_K1 * 4;
        ushort4 h4;
        unsigned short *h = reinterpret_cast<unsigned short *>(&h4);
#pragma unroll
        for (int r = 0; r < 4; ++r) h[r] = r0 + r < nvalid ? a0[(size_t)(row0 + r0 + r) * MLP_K1 + k] : (unsigned short)0;
        *reinterpret_cast<ushort4 *>(a0t + chunk_at(row0 + r0, k, MLP_K1)) = h4;
    }
    for (int j = threadIdx.x; j < TRAIN_ROWS * MLP_K1; j += 256) {
        const int r = j / MLP_K1, k = j % MLP_K1;
        const float v = (k < MLP_OUT && r < nvalid) ? dy[(size_t)(row0 + r) * MLP_OUT + k] : 0.f;
        const unsigned short h = f2bf(v);
        act[0][r * AS + k] = h;
        if (k < MLP_OUT) g4t[chunk_at(row0 + r, k, MLP_OUT)] = h;
    }
    __syncthreads();
#pragma unroll
    for (int l = 2; l >= 0; --l) {  // hidden layer l + 1
        const unsigned short *in = act[l & 1];  // l = 2 reads dy from act[0]
        unsigned short *out = act[(l + 1) & 1];
        floatx4 acc;
        if (l == 2) {
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(in + col * AS + kq), __builtin_bit_cast(bf16x8, w4),
                                                          floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        } else {
            const ushort8 *w = l == 1 ? w3 : w2;
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(in + col * AS + kq), __builtin_bit_cast(bf16x8, w[0]),
                                                          floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(in + col * AS + 32 + kq), __builtin_bit_cast(bf16x8, w[1]), acc,
                                                          0, 0, 0);
        }
        ushort4 h4;
        unsigned short *h = reinterpret_cast<unsigned short *>(&h4);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float d = 0.f;
            if (rq + r < nvalid) {
                d = acc[r] * dsilu(zv[l][r]);
                dz[l * lstride + (size_t)(row0 + rq + r) * MLP_H + c] = d;
            }
            h[r] = f2bf(d);
            out[(rq + r) * AS + c] = h[r];
        }
        *reinterpret_cast<ushort4 *>(gt + l * tstride + chunk_at(row0 + rq, c, MLP_H)) = h4;
        __syncthreads();
    }
}

// Weight gradients over a chunk of WGRAD_ROWS batch rows (blockIdx.x) of one layer
// (4 - blockIdx.y): partial dW_l = bf16(dz_l)^T a_{l-1} and db_l = sum dz_l, written to
// part[chunk][MLP_PARAMS].  Waves 0..3 take 16 outputs each (layer 4: 16 inputs each), wave 4
// the bias sums, in row order.  Rows past the batch: the operands of a 16-row block that was
// written are zero (g) there; blocks that were not written are not read.
constexpr int WGRAD_THREADS = 320;

__global__ __launch_bounds__(WGRAD_THREADS) void k_mlp_wgrad(const float *dy, const float *dz, const unsigned short *gt,
                                                             size_t gstride, const unsigned short *g4t,
                                                             const unsigned short *a0t, const unsigned short *at,
                                                             size_t astride, int batch, float *part)
{
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int chunk = blockIdx.x, b0 = chunk * WGRAD_ROWS, layer = 4 - blockIdx.y;
    const int nrow = min(WGRAD_ROWS, batch - b0);
    float *P = part + (size_t)chunk * MLP_PARAMS;
    if (wave == 4) {
        const int nout = layer == 4 ? MLP_OUT : MLP_H;
        const float *g = (layer == 4 ? dy : dz + (size_t)(layer - 1) * batch * MLP_H) + (size_t)b0 * nout;
        const int boff = layer == 1 ? OFF_B1 : layer == 2 ? OFF_B2 : layer == 3 ? OFF_B3 : OFF_B4;
        if (lane < nout) {
            float acc = 0.f;
            int b = 0;
            for (; b + 32 <= nrow; b += 32) {  // 32 loads in flight, added in row order
                float v[32];
#pragma unroll
                for (int i = 0; i < 32; ++i) v[i] = g[(size_t)(b + i) * nout + lane];
#pragma unroll
                for (int i = 0; i < 32; ++i) acc += v[i];
            }
            for (; b < nrow; ++b) acc += g[(size_t)b * nout + lane];
            P[boff + lane] = acc;
        }
        return;
    }
    const int r = lane & 15, kq = 8 * (lane >> 4), rq = 4 * (lane >> 4);
    const ushort8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
    // 8 rows of column c of a transposed operand, from row kk 32 + kq of the chunk
    auto op = [&](const unsigned short *m, int c, int cols, int kk) {
        const int row = kk * 32 + kq;
        const ushort8 v = row < nrow ? *reinterpret_cast<const ushort8 *>(m + ((size_t)chunk * cols + c) * WGRAD_ROWS + row) : zero;
        return __builtin_bit_cast(bf16x8, v);
    };
    auto tile = [&](const bf16x8 *A, const bf16x8 *B) {
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < WGRAD_ROWS / 32; ++kk) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[kk], B[kk], acc, 0, 0, 0);
        return acc;
    };
    constexpr int KK = WGRAD_ROWS / 32;
    bf16x8 A[KK], B[4][KK];
    if (layer == 4) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            A[kk] = op(g4t, r, MLP_OUT, kk);
            B[0][kk] = op(at + 2 * astride, wave * 16 + r, MLP_H, kk);
        }
        const floatx4 acc = tile(A, B[0]);
#pragma unroll
        for (int i = 0; i < 4; ++i) P[OFF_W4 + (rq + i) * MLP_H + wave * 16 + r] = acc[i];
        return;
    }
    const int kin = layer == 1 ? MLP_K1 : MLP_H;
    const int woff = layer == 1 ? OFF_W1 : layer == 2 ? OFF_W2 : OFF_W3;
    const unsigned short *am = layer == 1 ? a0t : at + (size_t)(layer - 2) * astride;
    const unsigned short *gm = gt + (size_t)(layer - 1) * gstride;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) A[kk] = op(gm, wave * 16 + r, MLP_H, kk);
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (t * 16 < kin)
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) B[t][kk] = op(am, t * 16 + r, kin, kk);
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (t * 16 < kin) {
            const floatx4 acc = tile(A, B[t]);
#pragma unroll
            for (int i = 0; i < 4; ++i) P[woff + (wave * 16 + rq + i) * kin + t * 16 + r] = acc[i];
        }
}

// grad[j] = sum over blocks of part[blk][j], in block order (deterministic)
__global__ __launch_bounds__(64) void k_mlp_reduce(const float *part, int nblk, float *grad)
{
    const int j = blockIdx.x * 64 + threadIdx.x;
    if (j >= MLP_PARAMS) return;
    float s = 0.f;
    int b = 0;
    for (; b + 16 <= nblk; b += 16) {  // 16 loads in flight, added in order
        float v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = part[(size_t)(b + i) * MLP_PARAMS + j];
#pragma unroll
        for (int i = 0; i < 16; ++i) s += v[i];
    }
    for (; b < nblk; ++b) s += part[(size_t)b * MLP_PARAMS + j];
    grad[j] = s;
}

// Adam (Kingma and Ba, 2015) on the FP32 master parameters; refreshes the bf16 copy.
__global__ void k_mlp_adam(float *w, unsigned short *wb, float *m, float *v, const float *g, int count,
                           float lr, float b1, float b2, float eps, float c1, float c2)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= count) return;
    float gj = g[j];
    float mj = b1 * m[j] + (1.f - b1) * gj;
    float vj = b2 * v[j] + (1.f - b2) * gj * gj;
    m[j] = mj;
    v[j] = vj;
    float wj = w[j] - lr * (mj / c1) / (sqrtf(vj / c2) + eps);
    w[j] = wj;
    wb[j] = f2bf(wj);
}

__global__ void k_round_bf16(const float *w, unsigned short *wb, int count)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < count) wb[j] = f2bf(w[j]);
}

// --------------------------------------------------------------------------------------
// Closure of a student context
// --------------------------------------------------------------------------------------
// (n, u, T, q, Pxx) of rows r < nx + 6 (cell r - 3; periodic problems wrap the cell index,
// others read the ghost rows).  Deviation storage adds ref; with U the density, velocity
// and temperature come from the conserved densities.
template <typename R>
__global__ void k_closure_rows(const R *psi, const double *ref, const double *U, const double *p,
                               int nx, int Q, int periodic, double *rows5)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nx + 2 * NG) return;
    const int sr = row_of(r - NG, nx, periodic);
    const R *ph = psi + (size_t)sr * 2 * Q;
    const R *th = ph + Q;
    double n = 0, j = 0, e2 = 0;
    for (int k = 0; k < Q; ++k) {
        double v = (double)ph[k] + ref[k];
        n += v;
        j += p[k] * v;
        e2 += 0.5 * (p[k] * p[k] * v + (double)th[k] + ref[Q + k]);
    }
    if (U) {
        const double *Ui = U + 3 * (size_t)sr;
        n = Ui[0];
        j = Ui[1];
        e2 = Ui[2];
    }
    double u = j / n, pxx = 0, e = 0, q = 0;
    for (int k = 0; k < Q; ++k) {
        double xi = p[k] - u;
        double vp = (double)ph[k] + ref[k], vt = (double)th[k] + ref[Q + k];
        double ek = 0.5 * xi * xi * vp + 0.5 * vt;
        pxx += xi * xi * vp;
        e += ek;
        q += xi * ek;
    }
    double T = U ? (2.0 * e2 / n - u * u) / 3.0 : e / (1.5 * n);
    double *o = rows5 + 5 * (size_t)r;
    o[0] = n; o[1] = u; o[2] = T; o[3] = q; o[4] = pxx;
}

struct ClosureConst {
    double dx, b, mu_ref, denseness, log10kn;
};

// The 12 inputs of cell i from the row moments, and n / tau.
__device__ inline void closure_features(const double *rows5, int i, const ClosureConst &cc,
                                        double x[MLP_IN], double *scale)
{
    const double *c = rows5 + 5 * (size_t)(i + NG);
    const double n = c[0], u = c[1], T = c[2], q = c[3], pxx = c[4];
    double d[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) {
        const double *m = rows5 + 5 * (size_t)i + f;  // row i = cell i - 3
        d[f] = (-m[0] + 9.0 * m[5] - 45.0 * m[10] + 45.0 * m[20] - 9.0 * m[25] + m[30]) / (60.0 * cc.dx);
    }
    const double eta = 0.25 * cc.b * n;
    const double chi = chi_set(eta);
    const double y = cc.b * n * chi;
    const double itau = inv_tau(cc.mu_ref, n, T, chi, y);
    const double sT = sqrt(T);
    const double lam = sT / itau;
    const double qs = n * T * sT;
    x[0] = n; x[1] = u; x[2] = T;
    x[3] = q / qs;
    x[4] = pxx / (n * T) - 1.0;
    x[5] = lam * d[0] / n;
    x[6] = lam * d[1] / sT;
    x[7] = lam * d[2] / T;
    x[8] = lam * d[3] / qs;
    x[9] = lam * d[4] / (n * T);
    x[10] = cc.denseness;
    x[11] = cc.log10kn;
    *scale = n * itau;
}

// Correction of the student's L[phi]: corr[i][k] (k < Q) = P (n / tau) (y * out_std +
// out_mean) on cells whose normalised inputs lie in [lo, hi]; zero (and counted in
// *outside) elsewhere.  The projection runs in FP64, so the mass, momentum and energy of
// the correction vanish to FP64 rounding before it is stored in the state's precision R.
// 64 cells per block.
template <typename R>
__global__ __launch_bounds__(256) void k_closure_apply(const unsigned short *wb, const float *params,
                                                       const float *norm, const double *Pc,
                                                       const double *rows5, ClosureConst cc, int nx,
                                                       int Q, R *corr,
                                                       unsigned long long *outside)
{
    __shared__ MlpSmem s;
    __shared__ float ys[4][16 * 17];
    __shared__ double sc[4][16];
    __shared__ int in_hull[4][16];
    __shared__ double pcs[MLP_OUT * MLP_OUT];
    mlp_stage_weights(s, wb, params);
    for (int j = threadIdx.x; j < MLP_OUT * MLP_OUT; j += blockDim.x) pcs[j] = Pc[j];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int cell0 = blockIdx.x * MLP_ROWS + wave * 16;
    for (int j = lane; j < 16 * MLP_K1; j += 64) s.act[wave][0][(j / MLP_K1) * AS + j % MLP_K1] = 0;
    __syncthreads();
    if (lane < 16) {
        const int i = cell0 + lane;
        int inside = 0;
        double scale = 0.0;
        if (i < nx) {
            double x[MLP_IN], sd;
            closure_features(rows5, i, cc, x, &sd);
            inside = 1;
            for (int c = 0; c < MLP_IN; ++c) {
                float v = ((float)x[c] - norm[NRM_IN_MEAN + c]) / norm[NRM_IN_STD + c];
                if (!(v >= norm[NRM_LO + c] && v <= norm[NRM_HI + c])) inside = 0;
                s.act[wave][0][lane * AS + c] = f2bf(v);
            }
            scale = sd;
        }
        sc[wave][lane] = scale;
        in_hull[wave][lane] = inside;
    }
    __syncthreads();
    floatx4 o;
    mlp_forward_rows(s, wave, lane, o);
    {
        const int col = lane & 15, rq = 4 * (lane >> 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) ys[wave][(rq + r) * 17 + col] = o[r];
    }
    __syncthreads();
    if (lane < 16) {
        const int i = cell0 + lane;
        if (i < nx) {
            const bool inside = in_hull[wave][lane] != 0;
            double v[MLP_OUT];
            for (int o2 = 0; o2 < MLP_OUT; ++o2)
                v[o2] = o2 < Q ? sc[wave][lane] * (double)(ys[wave][lane * 17 + o2] * norm[NRM_OUT_STD + o2] +
                                                           norm[NRM_OUT_MEAN + o2])
                               : 0.0;
            for (int k = 0; k < Q; ++k) {
                double acc = 0.0;
                for (int o2 = 0; o2 < Q; ++o2) acc += pcs[k * MLP_OUT + o2] * v[o2];
                corr[(size_t)i * Q + k] = inside ? (R)acc : R(0);
            }
            if (!inside) atomicAdd(outside, 1ull);
        }
    }
}

// Training sample of every cell: x[i] = the 12 inputs, y[i][j] = (Lt[i][j] - Ls[i][j]) tau / n
// for j < Q; Lt: the projected teacher right-hand side, Ls = psi1 - psi0 the student's (all
// rows of stride ls).
__global__ void k_closure_sample(const double *rows5, ClosureConst cc, int nx, int Q,
                                 const double *Lt, const double *psi1, const double *psi0, int ls, float *x_out,
                                 float *y_out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nx) return;
    double x[MLP_IN], sd;
    closure_features(rows5, i, cc, x, &sd);
    for (int c = 0; c < MLP_IN; ++c) x_out[(size_t)i * MLP_IN + c] = (float)x[c];
    for (int j = 0; j < Q; ++j) {
        const size_t o = (size_t)i * ls + j;
        y_out[(size_t)i * Q + j] = (float)((Lt[o] - (psi1[o] - psi0[o])) / sd);
    }
}

// Projection of a fine state onto QO <= 16 nodes: out[r][j] = sum_k P[k][j] in[r][k] for rows
// r < nrows (FP64), P [qi][MLP_OUT].  blockIdx.y: 0 phi, 1 theta of psi0, 2 the right-hand
// side of phi, psi1 - psi0 (rows of 2 qi values; out rows of 2 QO).  One thread per row, its QO
// sums in registers and P in scalar registers, so that a value read serves QO sums: bound by
// reading the rows.  65536 cells, 96 -> 12 nodes: the three fields 59 us; 3 x 198 us with a
// thread per sum, and 49 us for the difference as a pass of its own.
constexpr int PROJ_THREADS = 64;

template <int QO>
__global__ __launch_bounds__(PROJ_THREADS) void k_project_rows(const double *__restrict__ P, const double *__restrict__ psi0,
                                                               const double *__restrict__ psi1, int qi,
                                                               double *__restrict__ state, double *__restrict__ rhs, int nrows)
{
    const int r = blockIdx.x * PROJ_THREADS + threadIdx.x;
    if (r >= nrows) return;
    const int field = blockIdx.y;
    const double *in = psi0 + (size_t)r * 2 * qi + (field == 1 ? qi : 0);
    const double *in1 = psi1 + (size_t)r * 2 * qi;
    double acc[QO];
#pragma unroll
    for (int j = 0; j < QO; ++j) acc[j] = 0.0;
    for (int k = 0; k < qi; k += 4) {  // every compiled node count is a multiple of 4
        double v[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) v[d] = in[k + d];
        if (field == 2)
#pragma unroll
            for (int d = 0; d < 4; ++d) v[d] = in1[k + d] - v[d];
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int j = 0; j < QO; ++j) acc[j] = fma(P[(k + d) * MLP_OUT + j], v[d], acc[j]);
    }
    double *out = (field == 2 ? rhs : state) + (size_t)r * 2 * QO + (field == 1 ? QO : 0);
#pragma unroll
    for (int j = 0; j < QO; ++j) out[j] = acc[j];
}

// Lift of a state on QS <= 16 nodes onto qo: out[r][k] = sum_j Lam[k][j] in[r][j] for phi
// (blockIdx.y = 0) and theta (1), rows of 2 QS and 2 qo values.  One thread per node, its row
// of Lam in registers, over LIFT_ROWS rows whose inputs come in scalar registers: bound by
// writing the rows.  65536 cells, 12 -> 96 nodes: 59 us, 2 x 198 with a thread per sum.
constexpr int LIFT_ROWS = 32;

template <int QS>
__global__ __launch_bounds__(256) void k_lift_rows(const double *__restrict__ Lam, const double *__restrict__ in, int qo,
                                                   double *__restrict__ out, int nrows)
{
    const int k = threadIdx.x;
    const int r0 = blockIdx.x * LIFT_ROWS, r1 = min(r0 + LIFT_ROWS, nrows);
    double lam[QS];
#pragma unroll
    for (int j = 0; j < QS; ++j) lam[j] = Lam[min(k, qo - 1) * QS + j];
    const double *src = in + (blockIdx.y ? QS : 0);
    double *dst = out + (blockIdx.y ? qo : 0);
    for (int r = r0; r < r1; ++r) {
        double s = 0.0;
#pragma unroll
        for (int j = 0; j < QS; ++j) s = fma(lam[j], src[(size_t)r * 2 * QS + j], s);
        if (k < qo) dst[(size_t)r * 2 * qo + k] = s;
    }
}

// The right-hand side psi1 - psi0 of the interior rows as two planes, phi [nx][Q] and theta
// [nx][Q] (FP64).
__global__ __launch_bounds__(PLANE_THREADS) void k_rhs_planes(const double *psi1, const double *psi0, int nx, int Q, double *phi,
                                                              double *theta)
{
    for (size_t t = plane_first(); t < (size_t)nx * Q; t += plane_stride()) {
        const size_t i = t / Q, o = i * 2 * Q + (t - i * Q);
        phi[t] = psi1[o] - psi0[o];
        theta[t] = psi1[o + Q] - psi0[o + Q];
    }
}

}  // namespace elb
