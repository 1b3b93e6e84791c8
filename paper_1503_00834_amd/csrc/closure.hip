// Kernels of the learned subgrid closure that are not part of the SD
// residual: packing the network for the bfloat16 matrix cores, FP32
// training (forward, backward, Adam) and the per-element filter that makes
// training targets from a higher-order solution.  The fused inference
// lives with the residual kernels.
//
// Training is a sequence of small fixed-order kernels (no atomics), so a
// run is bitwise reproducible:
//   k_train      forward pass, loss, backward pass and weight gradients of
//                16-sample groups, every product on the FP32 matrix cores;
//                one partial sum of each gradient (and the loss) per block
//   k_wgrad_sum  the blocks' partials summed (the gradient alone)
//   k_wgrad_sum_adam  the partials summed and the Adam update (Kingma & Ba
//                2015, with bias correction) applied at once (training)
// (every sum in an order that the batch size alone fixes: the matrix-core
// products in their instruction order, the partials as eight interleaved
// running sums, then pairwise)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "launch.hpp"
#include "mlp_bf16.hpp"

namespace chorus {

// parameter vector offsets
constexpr int kW1 = 0, kB1 = 1280, kW2 = 1344, kB2 = 5440, kW3 = 5504, kB3 = 6464;
static_assert(kB3 + kMlpOut == kMlpParams, "parameter layout");

// ---------------------------------------------------------------------------
// packing
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_pack(const float *__restrict__ W, const float *__restrict__ norm,
                                             unsigned char *__restrict__ model) {
    const int lane = threadIdx.x, g = lane >> 4, r = lane & 15;
    bool ok = true;
    for (int q = lane; q < kMlpParams; q += 64) ok = ok && isfinite(W[q]);
    for (int q = lane; q < 70; q += 64) ok = ok && isfinite(norm[q]);
    uint32_t *fr = reinterpret_cast<uint32_t *>(model);
    for (int f = 0; f < kMlpFrags; ++f) {
        float a[8];
        for (int i = 0; i < 8; ++i) {
            float v = 0.0f;
            if (f < 4) {
                const int row = 16 * f + r, k = 8 * g + i;
                v = (k < kMlpIn) ? W[kW1 + row * kMlpIn + k] : 0.0f;
            } else if (f < 12) {
                const int mt = (f - 4) >> 1, ks = (f - 4) & 1;
                v = W[kW2 + (16 * mt + r) * kMlpHid + mlp_kperm(ks, g, i)];
            } else {
                const int ks = f - 12;
                v = (r < kMlpOut) ? W[kW3 + r * kMlpHid + mlp_kperm(ks, g, i)] : 0.0f;
            }
            a[i] = v;
        }
        uint32_t *dst = fr + (f * 64 + lane) * 4;
        for (int w = 0; w < 4; ++w) dst[w] = bf16_pair(a[2 * w], a[2 * w + 1]);
    }
    float *fl = reinterpret_cast<float *>(model + kMlpFloatOff);
    for (int q = lane; q < kMlpNFloat; q += 64) {
        float v = 0.0f;
        if (q < kMlpB2) v = W[kB1 + q];
        else if (q < kMlpB3) v = W[kB2 + q - kMlpB2];
        else if (q < kMlpXMean) v = (q - kMlpB3 < kMlpOut) ? W[kB3 + q - kMlpB3] : 0.0f;
        else if (q < kMlpXInv) v = norm[q - kMlpXMean];
        else if (q < kMlpYMean) v = norm[20 + q - kMlpXInv];
        else if (q < kMlpYStd) v = (q - kMlpYMean < kMlpOut) ? norm[40 + q - kMlpYMean] : 0.0f;
        else v = (q - kMlpYStd < kMlpOut) ? norm[55 + q - kMlpYStd] : 0.0f;
        fl[q] = v;
    }
    const bool all_ok = __all(ok);
    if (lane == 0) reinterpret_cast<int *>(model + kMlpFlagOff)[0] = all_ok ? 1 : 0;
}

// ---------------------------------------------------------------------------
// training
// ---------------------------------------------------------------------------
// GELU h = z Phi(z) and its derivative Phi(z) + z phi(z) in FP32, with
// erf by the rational approximation 7.1.26 of Abramowitz and Stegun (as in
// the inference; |error| <= 1.5e-7, the size of an FP32 rounding at these
// magnitudes; hardware reciprocal and exponential): with x = |z| / sqrt 2,
// 1 - erf(x) = t (a1 + a2 t + ... + a5 t^4) exp(-x^2), t = 1 / (1 + p x);
// exp(-x^2) = exp(-z^2 / 2) is also the normal density's factor, so one
// exponential serves both
__device__ __forceinline__ void gelu_and_prime(float z, float &h, float &gp) {
    const float az = fabsf(z);
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f * 0.70710678118654752f, az, 1.0f));
    float q = fmaf(1.061405429f, t, -1.453152027f);
    q = fmaf(q, t, 1.421413741f);
    q = fmaf(q, t, -0.284496736f);
    q = fmaf(q, t, 0.254829592f);
    const float e = __builtin_amdgcn_exp2f(z * z * (-0.5f * 1.4426950408889634f));
    const float tail = 0.5f * q * t * e;            // Phi(-|z|)
    const float Phi = (z >= 0.0f) ? 1.0f - tail : tail;
    h = z * Phi;
    gp = fmaf(z * 0.39894228040143268f, e, Phi);
}

// Four values of a lane from four consecutive floats at any float alignment.
__device__ __forceinline__ f32x4_t load4(const float *p) {
    f32x4_t v;
    __builtin_memcpy(&v, p, sizeof(v));
    return v;
}

// LDS image of a [64 units][16 samples] block of activations or gradients:
// the accumulator of the wave that owns row tile mt (lane l = 16 g + c: units
// 16 mt + 4 g + i of sample c) as one 16-byte slot per lane; 16 floats of
// padding per lane group spread the transposed reads (unit c of samples
// 4 ks + g) over all banks.
constexpr int kGrpStride = 80, kTileStride = 4 * kGrpStride;
__device__ __forceinline__ int slot_of(int tile, int g, int c) { return tile * kTileStride + g * kGrpStride + 4 * c; }
__device__ __forceinline__ int slot_unit(int tile, int u, int t) {
    return tile * kTileStride + (u >> 2) * kGrpStride + 4 * t + (u & 3);
}

// accumulated weight gradients of a share (see k_train)
struct TrainSums {
    f32x4_t W2[5], W1[2], W3[2];
};

// Forward, backward and weight gradients of one mini-batch.  A block of four
// waves takes 16 samples at a time (blocks stride over the 16-sample groups);
// wave w owns the hidden units 16 w .. 16 w + 15 of both hidden layers, so a
// layer is one 16 x 16 tile per wave and the four waves exchange activations
// and pre-activation gradients through LDS.  Everything is an FP32
// matrix-core product (v_mfma_f32_16x16x4f32: lane l holds A[l % 16][l / 16],
// B[l / 16][l % 16] and C[4 (l / 16) + i][l % 16], i = 0..3), hidden units as
// rows and samples as columns.  An accumulator (lane l: units 16 mt + 4 (l /
// 16) + i of sample l % 16) is the next product's B operand as it is when the
// K steps run over (mt, i), with the weight operand read at the same unit.
// The weight gradients are products over the group's samples (K = 16),
// accumulated in registers over the block's groups: dW2 = dZ2^T H1, dW1 =
// dZ1^T X, dW3 = dY^T H2 (row tile w each; dW3: column tile w), the bias
// gradients with a column of ones (feature 20 of the padded X; one more
// column tile for dW2 and dW3), the loss in the padding row 15 of dY^T.  Each
// of the nblk shares of the groups (every nblk-th) has its own partial sums.  A
// block writes those of share blockIdx.x to part[block][kMlpParams + 1]; with
// TWO it adds those of share blockIdx.x + gridDim.x, if there is one.
//
// What bounds it: a batch of 4,096 is 256 groups, one block per CU, and each
// layer waits for the one before: a chain of about 80 matrix products per wave,
// 1.1 us of the 10 us of a launch.  The rest is latency (launch and ramp,
// weights and gathered rows, four barriers, the partial rows' stores), whose
// parts have not been timed one by one.  One wave per 16 samples that walked all four row tiles
// (320 products in a chain on a quarter of the SIMDs), the activations and
// gradients sent through memory to a second kernel for the weight gradients,
// took 13.4 + 11.6 us at batch 4,096; an iteration with its partial sums and
// Adam went from 28.0 to 14.3 us.
template <bool TWO>
__global__ __launch_bounds__(256, 2) void k_train(const float *__restrict__ X, const float *__restrict__ Y,
                                                  const int32_t *__restrict__ idx, int64_t base, int nb,
                                                  const float *__restrict__ W, float *__restrict__ part_all,
                                                  int64_t n_mean, int nblk) {
    __shared__ __align__(16) float sH1[4 * kTileStride], sH2[4 * kTileStride], sZ1[4 * kTileStride],
        sZ2[4 * kTileStride], sYp[4 * 256], sdY[kTileStride], sloss[16];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    const int ngrp = (nb + 15) / 16;
    // weights of this wave's row tile, read once per block
    float a1[5], a2b[16], a3b[4];
    f32x4_t a2f[4], a3f;
#pragma unroll
    for (int ks = 0; ks < 5; ++ks) a1[ks] = W[kW1 + (16 * w + c) * kMlpIn + 4 * ks + g];
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) a2f[kt] = load4(W + kW2 + (16 * w + c) * kMlpHid + 16 * kt + 4 * g);
    a3f = load4(W + kW3 + (c < kMlpOut ? c : 0) * kMlpHid + 16 * w + 4 * g);
    if (c >= kMlpOut) a3f = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ki = 0; ki < 4; ++ki) {
        const int k = 4 * g + ki;
        a3b[ki] = W[kW3 + (k < kMlpOut ? k : 0) * kMlpHid + 16 * w + c];
        if (k >= kMlpOut) a3b[ki] = 0.0f;
    }
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int ki = 0; ki < 4; ++ki) a2b[4 * kt + ki] = W[kW2 + (16 * kt + 4 * g + ki) * kMlpHid + 16 * w + c];
    const f32x4_t b1 = load4(W + kB1 + 16 * w + 4 * g), b2 = load4(W + kB2 + 16 * w + 4 * g);
    f32x4_t b3;
#pragma unroll
    for (int i = 0; i < 4; ++i) b3[i] = (4 * g + i < kMlpOut) ? W[kB3 + 4 * g + i] : 0.0f;
    const f32x4_t zero = {0.0f, 0.0f, 0.0f, 0.0f};
    const float sc = 2.0f / ((float)n_mean * (float)kMlpOut);
    const auto work = [&](int share) {
        TrainSums G;
#pragma unroll
        for (int q = 0; q < 5; ++q) G.W2[q] = zero;
        G.W1[0] = G.W1[1] = G.W3[0] = G.W3[1] = zero;
        for (int grp = share; grp < ngrp; grp += nblk) {
            // this lane's sample as a column (t) and, for dW1, as a K step;
            // lanes past the batch compute on its first sample with zero weight
            const int t = 16 * grp + c;
            const bool ok = t < nb;
            const int64_t s = idx ? (int64_t)idx[base + (ok ? t : 0)] : base + (ok ? t : 0);
            int64_t sk[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const int tk = 16 * grp + 4 * ks + g;
                sk[ks] = idx ? (int64_t)idx[base + (tk < nb ? tk : 0)] : base + (tk < nb ? tk : 0);
            }
            float x1[5], xk[4][2], yt[4];
#pragma unroll
            for (int ks = 0; ks < 5; ++ks) x1[ks] = X[s * kMlpIn + 4 * ks + g];
#pragma unroll
            for (int i = 0; i < 4; ++i) yt[i] = Y[s * kMlpOut + (4 * g + i < kMlpOut ? 4 * g + i : 0)];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                xk[ks][0] = X[sk[ks] * kMlpIn + c];
                xk[ks][1] = X[sk[ks] * kMlpIn + (c < 4 ? 16 + c : 0)];
                if (c >= 4) xk[ks][1] = (c == 4) ? 1.0f : 0.0f;
            }
            // layer 1
            f32x4_t h1 = b1, p1, h2 = b2, p2;
#pragma unroll
            for (int ks = 0; ks < 5; ++ks) h1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[ks], x1[ks], h1, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float h, gp;
                gelu_and_prime(h1[i], h, gp);
                h1[i] = h;
                p1[i] = gp;
            }
            *reinterpret_cast<f32x4_t *>(sH1 + slot_of(w, g, c)) = h1;
            __syncthreads();
            // layer 2
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) {
                const f32x4_t b = *reinterpret_cast<const f32x4_t *>(sH1 + slot_of(kt, g, c));
#pragma unroll
                for (int ki = 0; ki < 4; ++ki) h2 = __builtin_amdgcn_mfma_f32_16x16x4f32(a2f[kt][ki], b[ki], h2, 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float h, gp;
                gelu_and_prime(h2[i], h, gp);
                h2[i] = h;
                p2[i] = gp;
            }
            *reinterpret_cast<f32x4_t *>(sH2 + slot_of(w, g, c)) = h2;
            // layer 3: each wave its own units' part of the outputs 4 g + i (row
            // 15 padding), summed over the waves in a fixed order
            f32x4_t yp = zero;
#pragma unroll
            for (int ki = 0; ki < 4; ++ki) yp = __builtin_amdgcn_mfma_f32_16x16x4f32(a3f[ki], h2[ki], yp, 0, 0, 0);
            *reinterpret_cast<f32x4_t *>(sYp + 256 * w + 4 * lane) = yp;
            __syncthreads();
            f32x4_t q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = *reinterpret_cast<const f32x4_t *>(sYp + 256 * u + 4 * lane);
            const f32x4_t y = ((q[0] + q[1]) + (q[2] + q[3])) + b3;
            f32x4_t dy;
            float l = 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float e = (ok && 4 * g + i < kMlpOut) ? y[i] - yt[i] : 0.0f;
                l += e * e;
                dy[i] = sc * e;
            }
            if (w == 0) {
                // the sample's loss: the four lane groups in a fixed order
                const float l1 = __shfl_xor(l, 16), l2 = __shfl_xor(l, 32), l3 = __shfl_xor(l, 48);
                *reinterpret_cast<f32x4_t *>(sdY + slot_of(0, g, c)) = dy;
                if (g == 0) sloss[c] = (l + l1) + (l2 + l3);
            }
            // back through layer 3 and layer 2
            f32x4_t dz2 = zero, dz1 = zero;
#pragma unroll
            for (int ki = 0; ki < 4; ++ki) dz2 = __builtin_amdgcn_mfma_f32_16x16x4f32(a3b[ki], dy[ki], dz2, 0, 0, 0);
            dz2 *= p2;
            *reinterpret_cast<f32x4_t *>(sZ2 + slot_of(w, g, c)) = dz2;
            __syncthreads();
#pragma unroll
            for (int kt = 0; kt < 4; ++kt) {
                const f32x4_t b = *reinterpret_cast<const f32x4_t *>(sZ2 + slot_of(kt, g, c));
#pragma unroll
                for (int ki = 0; ki < 4; ++ki)
                    dz1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a2b[4 * kt + ki], b[ki], dz1, 0, 0, 0);
            }
            dz1 *= p1;
            // (read back by this wave alone)
            *reinterpret_cast<f32x4_t *>(sZ1 + slot_of(w, g, c)) = dz1;
            __builtin_amdgcn_wave_barrier();
            // weight gradients over the group's samples
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const int tk = 4 * ks + g;
                const float z2 = sZ2[slot_unit(w, c, tk)], one = (c == 0) ? 1.0f : 0.0f;
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
                    G.W2[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(z2, sH1[slot_unit(nt, c, tk)], G.W2[nt], 0, 0, 0);
                G.W2[4] = __builtin_amdgcn_mfma_f32_16x16x4f32(z2, one, G.W2[4], 0, 0, 0);
                const float ys = (c < kMlpOut) ? sdY[slot_unit(0, c, tk)] : sloss[tk];
                G.W3[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(ys, sH2[slot_unit(w, c, tk)], G.W3[0], 0, 0, 0);
                if (w == 0) G.W3[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(ys, one, G.W3[1], 0, 0, 0);
                const float z1 = sZ1[slot_unit(w, c, tk)];
#pragma unroll
                for (int nt = 0; nt < 2; ++nt)
                    G.W1[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(z1, xk[ks][nt], G.W1[nt], 0, 0, 0);
            }
            __syncthreads();  // the next group rewrites the LDS images
        }
        return G;
    };
    TrainSums G = work(blockIdx.x);
    if constexpr (TWO) {
        if ((int)(blockIdx.x + gridDim.x) < nblk) {
            const TrainSums H = work(blockIdx.x + gridDim.x);
#pragma unroll
            for (int q = 0; q < 5; ++q) G.W2[q] += H.W2[q];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                G.W1[q] += H.W1[q];
                G.W3[q] += H.W3[q];
            }
        }
    }
    float *part = part_all + (int64_t)blockIdx.x * (kMlpParams + 1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int j = 16 * w + 4 * g + i;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) part[kW2 + j * kMlpHid + 16 * nt + c] = G.W2[nt][i];
        if (c == 0) part[kB2 + j] = G.W2[4][i];
        part[kW1 + j * kMlpIn + c] = G.W1[0][i];
        if (c < 4) part[kW1 + j * kMlpIn + 16 + c] = G.W1[1][i];
        if (c == 4) part[kB1 + j] = G.W1[1][i];
        const int k = 4 * g + i;
        if (k < kMlpOut) part[kW3 + k * kMlpHid + 16 * w + c] = G.W3[0][i];
        if (w == 0 && c == 0) part[k < kMlpOut ? kB3 + k : kMlpParams] = G.W3[1][i];
    }
}

// sum over the blocks' partials of 64 consecutive quantities (one per lane:
// whole cache lines) in a fixed order: partial c < nextra takes partial c +
// nchunk first; wave r of the block sums partials r, r + 8, ... in turn, the
// eight sums combined pairwise; valid in wave 0
__device__ __forceinline__ float partial_sum(int nchunk, int nextra, const float *__restrict__ part, int q,
                                             float (*red)[64]) {
    const int r = threadIdx.x >> 6, lane = threadIdx.x & 63;
    float a = 0.0f;
    float x[kTrainExtra / 8];
#pragma unroll
    for (int u = 0; u < kTrainExtra / 8; ++u) {
        const int c = r + 8 * u;
        x[u] = part[(int64_t)(c < nextra ? c + nchunk : 0) * (kMlpParams + 1) + q];
    }
    // 16 partials per wave and round, every load of a round issued first
    for (int c0 = r; c0 < nchunk; c0 += 128) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int c = c0 + 8 * u;
            v[u] = part[(int64_t)(c < nchunk ? c : c0) * (kMlpParams + 1) + q];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int c = c0 + 8 * u;
            if (u < kTrainExtra / 8 && c < nextra) v[u] += x[u < kTrainExtra / 8 ? u : 0];
            if (c < nchunk) a += v[u];
        }
    }
    red[r][lane] = a;
    __syncthreads();
    return ((red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane])) +
           ((red[4][lane] + red[5][lane]) + (red[6][lane] + red[7][lane]));
}

// one lane per quantity (parameter, or the loss for q = kMlpParams)
__global__ __launch_bounds__(512) void k_wgrad_sum(int nchunk, int nextra, const float *__restrict__ part,
                                                   int64_t n_mean, float *__restrict__ grad, float *__restrict__ loss) {
    __shared__ float red[8][64];
    const int qq = blockIdx.x * 64 + (int)(threadIdx.x & 63), q = qq <= kMlpParams ? qq : kMlpParams;
    const float s = partial_sum(nchunk, nextra, part, q, red);
    if (threadIdx.x >= 64 || qq > kMlpParams) return;
    if (q < kMlpParams) grad[q] = s;
    else loss[0] = s / ((float)n_mean * (float)kMlpOut);
}

__device__ __forceinline__ void adam_update(float *__restrict__ W, float *__restrict__ m, float *__restrict__ v,
                                            float g, const AdamArgs &a, int q) {
    const float mq = a.b1 * m[q] + (1.0f - a.b1) * g;
    const float vq = a.b2 * v[q] + (1.0f - a.b2) * g * g;
    m[q] = mq;
    v[q] = vq;
    W[q] -= a.lr * (mq * a.inv_bc1) / (sqrtf(vq * a.inv_bc2) + a.eps);
}

__global__ __launch_bounds__(512) void k_wgrad_sum_adam(int nchunk, int nextra, const float *__restrict__ part,
                                                        int64_t n_mean, float *__restrict__ W, float *__restrict__ m,
                                                        float *__restrict__ v, AdamArgs a, float *__restrict__ loss) {
    __shared__ float red[8][64];
    const int qq = blockIdx.x * 64 + (int)(threadIdx.x & 63), q = qq <= kMlpParams ? qq : kMlpParams;
    const float s = partial_sum(nchunk, nextra, part, q, red);
    if (threadIdx.x >= 64 || qq > kMlpParams) return;
    if (q < kMlpParams) adam_update(W, m, v, s, a, q);
    else loss[0] = s / ((float)n_mean * (float)kMlpOut);
}

// ---------------------------------------------------------------------------
// filter: per element L2 projection of |J| U to degree Nc - 1
// ---------------------------------------------------------------------------
__device__ __forceinline__ void cart_flux(const double q[5], double gm1, double F[15]) {
    const double r = q[0], m[3] = {q[1], q[2], q[3]}, E = q[4];
    const double ir = 1.0 / r;
    const double p = gm1 * (E - 0.5 * (m[0] * m[0] + m[1] * m[1] + m[2] * m[2]) * ir);
    for (int c = 0; c < 3; ++c) {
        F[c] = m[c];
        for (int i = 0; i < 3; ++i) F[3 * (1 + i) + c] = m[i] * m[c] * ir + (i == c ? p : 0.0);
        F[12 + c] = (E + p) * m[c] * ir;
    }
}

// Elements per block of one wave: a lane takes one xi line of an element in
// the first contraction, NF^2 lines per element.
template <int NF>
constexpr int filter_epb() { return 64 / (NF * NF); }

// Bound by its HBM bytes (6 doubles per fine point read, 20 per coarse point
// written: 180 MB from order 6 to 3 on 12,288 hexes).  The 20 products |J| Q
// and |J| F(Q) of a fine point never reach memory: the lane of a xi line forms
// them point by point and adds each into its NC projected values, so LDS
// first holds them contracted (20 NC NF^2 doubles per element, 17 KB at 6 ->
// 3, nine waves per CU; the eta and zeta contractions are written over it
// after a barrier).  With the orders as run-time values, every product in
// LDS (61 KB per element, two waves per CU) and an index division per
// multiply-add, the filter took 1,005 us; a pass of filter and features went
// from 1,038 to 99 us.
template <int NF, int NC>
__global__ __launch_bounds__(64) void k_filter(FilterArgs A) {
    constexpr int EPB = filter_epb<NF>(), L2 = NF * NF, NPF = NF * NF * NF, NPC = NC * NC * NC;
    constexpr int S1 = 20 * NC * L2, IT_ETA = 20 * NC * NF, IT_ZETA = 20 * NC * NC;
    constexpr int R_ETA = (EPB * IT_ETA + 63) / 64, R_ZETA = (EPB * IT_ZETA + 63) / 64;
    __shared__ double T[EPB][S1];
    const int64_t e0 = (int64_t)blockIdx.x * EPB;
    const double gm1 = A.gamma - 1.0;
    // xi: (a, j, k) <- sum_i P[a][i] U(i, j, k)
    {
        const int el = threadIdx.x / L2, jk = threadIdx.x % L2;
        if (el < EPB && e0 + el < A.E) {
            const int64_t e = e0 + el;
            double acc[20][NC];
#pragma unroll
            for (int f = 0; f < 20; ++f)
#pragma unroll
                for (int a = 0; a < NC; ++a) acc[f][a] = 0.0;
            // the whole line first: one wait for memory
            double ql[NF][5], iJ[NF];
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                const int p = i + NF * jk;
                for (int v = 0; v < 5; ++v) ql[i][v] = A.Qf[((int64_t)v * A.E + e) * NPF + p];
                iJ[i] = A.solgeo_f[(e * 13 + 9) * NPF + p];
            }
#pragma unroll
            for (int i = 0; i < NF; ++i) {
                const double J = 1.0 / iJ[i];
                double F[15];
                cart_flux(ql[i], gm1, F);
#pragma unroll
                for (int f = 0; f < 20; ++f) {
                    const double u = J * (f < 5 ? ql[i][f < 5 ? f : 0] : F[f < 5 ? 0 : f - 5]);
#pragma unroll
                    for (int a = 0; a < NC; ++a) acc[f][a] += A.P[a][i] * u;
                }
            }
#pragma unroll
            for (int f = 0; f < 20; ++f)
#pragma unroll
                for (int a = 0; a < NC; ++a) T[el][(f * L2 + jk) * NC + a] = acc[f][a];
        }
    }
    __syncthreads();
    // eta: (a, b, k) <- sum_j P[b][j] T(a, j, k); a thread forms the NC
    // values b of one (field, a, k)
    double r[R_ETA][NC];
#pragma unroll
    for (int q = 0; q < R_ETA; ++q) {
        const int it = threadIdx.x + 64 * q;
        const int el = it / IT_ETA, x = it % IT_ETA, f = x / (NC * NF), ak = x % (NC * NF), a = ak % NC, k = ak / NC;
#pragma unroll
        for (int b = 0; b < NC; ++b) r[q][b] = 0.0;
        if (el >= EPB || e0 + el >= A.E) continue;
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            const double t = T[el][(f * L2 + j + NF * k) * NC + a];
#pragma unroll
            for (int b = 0; b < NC; ++b) r[q][b] += A.P[b][j] * t;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < R_ETA; ++q) {
        const int it = threadIdx.x + 64 * q;
        const int el = it / IT_ETA, x = it % IT_ETA, f = x / (NC * NF), ak = x % (NC * NF), a = ak % NC, k = ak / NC;
        if (el >= EPB) continue;
#pragma unroll
        for (int b = 0; b < NC; ++b) T[el][f * (NC * NC * NF) + a + NC * (b + NC * k)] = r[q][b];
    }
    __syncthreads();
    // zeta: (a, b, c) <- sum_k P[c][k] T(a, b, k)
    double z[R_ZETA][NC];
#pragma unroll
    for (int q = 0; q < R_ZETA; ++q) {
        const int it = threadIdx.x + 64 * q;
        const int el = it / IT_ZETA, x = it % IT_ZETA, f = x / (NC * NC), ab = x % (NC * NC);
#pragma unroll
        for (int c = 0; c < NC; ++c) z[q][c] = 0.0;
        if (el >= EPB || e0 + el >= A.E) continue;
#pragma unroll
        for (int k = 0; k < NF; ++k) {
            const double t = T[el][f * (NC * NC * NF) + ab + NC * NC * k];
#pragma unroll
            for (int c = 0; c < NC; ++c) z[q][c] += A.P[c][k] * t;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < R_ZETA; ++q) {
        const int it = threadIdx.x + 64 * q;
        const int el = it / IT_ZETA, x = it % IT_ZETA, f = x / (NC * NC), ab = x % (NC * NC);
        if (el >= EPB) continue;
#pragma unroll
        for (int c = 0; c < NC; ++c) T[el][f * NPC + ab + NC * NC * c] = z[q][c];
    }
    __syncthreads();
    // divide by the coarse |J|, subgrid flux
    for (int it = threadIdx.x; it < EPB * NPC; it += 64) {
        const int el = it / NPC, p = it % NPC;
        const int64_t e = e0 + el;
        if (e >= A.E) continue;
        const double iJ = A.solgeo_c[(e * 13 + 9) * NPC + p];
        double qb[5], F[15];
        for (int v = 0; v < 5; ++v) qb[v] = T[el][v * NPC + p] * iJ;
        cart_flux(qb, gm1, F);
        for (int v = 0; v < 5; ++v) A.Qbar[((int64_t)v * A.E + e) * NPC + p] = qb[v];
        for (int k = 0; k < 15; ++k)
            A.tau[((int64_t)k * A.E + e) * NPC + p] = (k < 3) ? 0.0 : T[el][(5 + k) * NPC + p] * iJ - F[k];
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_pack(const float *W, const float *norm, unsigned char *model, hipStream_t s) {
    hipLaunchKernelGGL(k_pack, dim3(1), dim3(64), 0, s, W, norm, model);
    return hipGetLastError();
}

// The groups of a mini-batch go to T.blocks shares (one group each up to
// kTrainPartials) that are summed as T.sums partials, the first (blocks - sums)
// of which take a second share's: both numbers follow from the batch alone.
// Where the workspace holds a row for every share, each is a block of k_train
// and the sum adds the second rows; where it does not, the first blocks work
// through two shares: the same sums.
static hipError_t launch_train_partials(const float *X, const float *Y, const int32_t *idx, int64_t base, int nb,
                                        const float *W, const TrainBufs &T, int &nextra, hipStream_t s) {
    nextra = T.rows >= T.blocks ? T.blocks - T.sums : 0;
    if (T.sums + nextra == T.blocks)
        hipLaunchKernelGGL(k_train<false>, dim3(T.blocks), dim3(256), 0, s, X, Y, idx, base, nb, W, T.part, T.n_mean,
                           T.blocks);
    else
        hipLaunchKernelGGL(k_train<true>, dim3(T.sums), dim3(256), 0, s, X, Y, idx, base, nb, W, T.part, T.n_mean,
                           T.blocks);
    return hipGetLastError();
}
static constexpr int kSumBlocksMlp = (kMlpParams + 1 + 63) / 64;

hipError_t launch_train_grad(const float *X, const float *Y, const int32_t *idx, int64_t base, int nb,
                             const float *W, const TrainBufs &T, float *grad, float *loss, hipStream_t s) {
    int nextra = 0;
    hipError_t e = launch_train_partials(X, Y, idx, base, nb, W, T, nextra, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_wgrad_sum, dim3(kSumBlocksMlp), dim3(512), 0, s, T.sums, nextra, (const float *)T.part,
                       T.n_mean, grad, loss);
    return hipGetLastError();
}

hipError_t launch_train_step(const float *X, const float *Y, const int32_t *idx, int64_t base, int nb, float *W,
                             float *m, float *v, const TrainBufs &T, const AdamArgs &a, float *loss, hipStream_t s) {
    int nextra = 0;
    hipError_t e = launch_train_partials(X, Y, idx, base, nb, W, T, nextra, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_wgrad_sum_adam, dim3(kSumBlocksMlp), dim3(512), 0, s, T.sums, nextra, (const float *)T.part,
                       T.n_mean, W, m, v, a, loss);
    return hipGetLastError();
}

// flag[0] = 1 if a sample index lies outside [0, n) (flag cleared first)
__global__ __launch_bounds__(256) void k_check_idx(const int32_t *__restrict__ idx, int64_t count, int64_t n,
                                                   int *__restrict__ flag) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    const int32_t v = idx[i];
    if (v < 0 || v >= n) flag[0] = 1;
}

hipError_t launch_check_idx(const int32_t *idx, int64_t count, int64_t n, int *flag, hipStream_t s) {
    hipError_t e = launch_clear_flag(flag, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_check_idx, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, idx, count, n, flag);
    return hipGetLastError();
}

template <int NF, int NC>
static hipError_t launch_filter_t(const FilterArgs &A, hipStream_t s) {
    constexpr int EPB = filter_epb<NF>();
    hipLaunchKernelGGL((k_filter<NF, NC>), dim3((unsigned)((A.E + EPB - 1) / EPB)), dim3(64), 0, s, A);
    return hipGetLastError();
}

hipError_t launch_filter(const FilterArgs &A, hipStream_t s) {
    switch (10 * A.nf + A.nc) {
        case 32: return launch_filter_t<3, 2>(A, s);
        case 42: return launch_filter_t<4, 2>(A, s);
        case 43: return launch_filter_t<4, 3>(A, s);
        case 52: return launch_filter_t<5, 2>(A, s);
        case 53: return launch_filter_t<5, 3>(A, s);
        case 62: return launch_filter_t<6, 2>(A, s);
        case 63: return launch_filter_t<6, 3>(A, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace chorus
