// Learned spectral bounds: forward, loss + hand-written backward, Adam.
//
// The paper only requires that A is rescaled before the sign iteration so that
// it converges (Sec. III-B.2, after Eq. NS2). The 12 -> 64 -> 64 -> 2 SiLU
// perceptron predicts the normalised extreme eigenvalues of A_J from O(n^2)
// features; the scale it implies is clamped at the Gershgorin scale.
// Parameter packing: W1[64][12], b1[64], W2[64][64], b2[64], W3[2][64], b3[2].
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/nolsm.h"

#define NF 12
#define NH 64
#define NO 2
#define OFF_B1 (NH * NF)
#define OFF_W2 (OFF_B1 + NH)
#define OFF_B2 (OFF_W2 + NH * NH)
#define OFF_W3 (OFF_B2 + NH)
#define OFF_B3 (OFF_W3 + NO * NH)
#define NPAR (OFF_B3 + NO)
static_assert(NPAR == NOLSM_MLP_NPARAM, "parameter packing");

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }

// one thread per sample; parameters staged in LDS
__global__ __launch_bounds__(256) void k_mlp_forward(const float *__restrict__ prm, const float *__restrict__ norm,
                                                     const float *__restrict__ x, int B, float *__restrict__ out) {
    __shared__ float P[NPAR];
    __shared__ float nm[2 * NF];
    for (int i = threadIdx.x; i < NPAR; i += blockDim.x) P[i] = prm[i];
    for (int i = threadIdx.x; i < 2 * NF; i += blockDim.x) nm[i] = norm[i];
    __syncthreads();
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    float xs[NF];
    for (int i = 0; i < NF; ++i) xs[i] = (x[(int64_t)b * NF + i] - nm[i]) / nm[NF + i];
    float h1[NH];
    for (int j = 0; j < NH; ++j) {
        float z = P[OFF_B1 + j];
        for (int i = 0; i < NF; ++i) z += P[j * NF + i] * xs[i];
        h1[j] = silu(z);
    }
    float o0 = P[OFF_B3], o1 = P[OFF_B3 + 1];
    for (int j = 0; j < NH; ++j) {
        float z = P[OFF_B2 + j];
        for (int i = 0; i < NH; ++i) z += P[OFF_W2 + j * NH + i] * h1[i];
        const float h = silu(z);
        o0 += P[OFF_W3 + j] * h;
        o1 += P[OFF_W3 + NH + j] * h;
    }
    out[(int64_t)b * 2] = o0;
    out[(int64_t)b * 2 + 1] = o1;
}

// Loss and gradient over a batch on the FP32 matrix cores
// (v_mfma_f32_16x16x4_f32). Each wave takes 16 samples at a time through the
// whole network: A operands are samples by units, and a layer's result (lane
// l, element e of block j: sample 4 (l / 16) + e, unit 16 j + l % 16) is
// turned into the next A operand through the wave's own LDS rows, with no
// barrier. As the operands of a product over the samples (the weights'
// gradients) the results serve as they lie. Four workgroups share the work
// by hidden unit: each runs the forward pass of every sample, workgroup g
// forms the gradients that end in block g of 16 units (columns 16 g .. of
// W2, rows 16 g .. of W1 and so on). Nothing is summed across workgroups, so
// no scratch memory is needed; the waves' sums are added in wave order
// (deterministic). One workgroup with a lane per unit, its weights and
// activations read from LDS for every product, was bound by those reads: a
// step (this and Adam) of 256 samples took 94 us, now 25; of 1,024, 280 and 76.
// Eight waves of up to 256 registers: with sixteen of 128 it spilled (45 us).
#define NWAVE 8
#define LDW 68   // LDS row stride: rows 4 banks apart, 16 rows x 4 k distinct
typedef float f4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f4 mma4(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
// SiLU and its derivative from one exponential
__device__ __forceinline__ void silu2(float z, float &h, float &d) {
    const float s = 1.0f / (1.0f + expf(-z));
    h = z * s;
    d = s * (1.0f + z * (1.0f - s));
}
// Between a wave's stores to its own LDS rows and other lanes' loads of them,
// either way round: the wave's LDS accesses are executed in order, and this
// keeps the compiler to it (no instruction comes of it).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ float sum16(float v) {   // over the 16 lanes of a group
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float sum4(float v) {    // over the four groups
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}

__global__ __launch_bounds__(NWAVE * 64) void k_mlp_loss_grad(const float *__restrict__ prm, const float *__restrict__ norm,
                                                        const float *__restrict__ x, const float *__restrict__ y,
                                                        int B, float *__restrict__ grad, float *__restrict__ loss_out) {
    __shared__ float W2[NH * LDW];
    __shared__ float act[NWAVE][16 * LDW];   // a wave's 16 samples x 64 units; then its gradient sums
    __shared__ float part[NWAVE][16 * 16 + 64];
    const int t = threadIdx.x, w = t >> 6, l = t & 63, li = l & 15, lk = l >> 4, g = blockIdx.x;
    for (int i = t; i < NH * NH; i += NWAVE * 64) W2[(i / NH) * LDW + i % NH] = prm[OFF_W2 + i];
    // weights of this lane's units and of the first layer's B operand
    // (W1[16 j + li][4 s + lk])
    float w1[3][4], b1[4], b2[4], w30[4], w31[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int u = 16 * j + li;
        b1[j] = prm[OFF_B1 + u];
        b2[j] = prm[OFF_B2 + u];
        w30[j] = prm[OFF_W3 + u];
        w31[j] = prm[OFF_W3 + NH + u];
#pragma unroll
        for (int s = 0; s < 3; ++s) w1[s][j] = prm[u * NF + 4 * s + lk];
    }
    const float b30 = prm[OFF_B3], b31 = prm[OFF_B3 + 1];
    const float xm = li < NF ? norm[li] : 0.0f, xd = li < NF ? norm[NF + li] : 1.0f;
    float am[3], ad[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        am[s] = norm[4 * s + lk];
        ad[s] = norm[NF + 4 * s + lk];
    }
    __syncthreads();
    f4 gW2[4], gW1 = {0, 0, 0, 0};   // blocks (k, g) of W2's gradient; rows 16 g .. of W1's, column 12 that of b1
#pragma unroll
    for (int i = 0; i < 4; ++i) gW2[i] = (f4){0, 0, 0, 0};
    float gb2 = 0, gw30 = 0, gw31 = 0, gb30 = 0, gb31 = 0, lsum = 0;
    const float scale = 2.0f / (float)(B * NO);
    float *const A = act[w];
    for (int s0 = w * 16; s0 < B; s0 += 16 * NWAVE) {
        // layer 1: sample li as the A operand's row
        // W2's LDS rows through an offset that the compiler takes as new in
        // every pass: it would keep all of them in registers, and spill
        int o2 = 0;
        asm volatile("" : "+v"(o2));
        const float *const W = W2 + o2;
        f4 z1[4], h1[4];
        float dz1[4];   // d h1 / d z1 of block g
#pragma unroll
        for (int j = 0; j < 4; ++j) z1[j] = (f4){b1[j], b1[j], b1[j], b1[j]};
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const float a = s0 + li < B ? (x[(int64_t)(s0 + li) * NF + 4 * s + lk] - am[s]) / ad[s] : 0.0f;
#pragma unroll
            for (int j = 0; j < 4; ++j) z1[j] = mma4(a, w1[s][j], z1[j]);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float h, d;
                silu2(z1[j][e], h, d);
                h1[j][e] = h;
                if (j == g) dz1[e] = d;
                A[(4 * lk + e) * LDW + 16 * j + li] = h;
            }
        wave_sync();
        // layer 2
        f4 z2[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) z2[j] = (f4){b2[j], b2[j], b2[j], b2[j]};
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const float a = A[li * LDW + 4 * s + lk];
#pragma unroll
            for (int j = 0; j < 4; ++j) z2[j] = mma4(a, W[(16 * j + li) * LDW + 4 * s + lk], z2[j]);
        }
        // outputs, loss and their gradients, one sample per element
        f4 gz2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int b = s0 + 4 * lk + e;
            const bool valid = b < B;
            float h2[4], dz2[4], o0 = 0, o1 = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                silu2(z2[j][e], h2[j], dz2[j]);
                o0 += w30[j] * h2[j];
                o1 += w31[j] * h2[j];
            }
            o0 = sum16(o0) + b30;
            o1 = sum16(o1) + b31;
            const float d0 = valid ? o0 - y[(int64_t)b * 2] : 0.0f, d1 = valid ? o1 - y[(int64_t)b * 2 + 1] : 0.0f;
            const float q0 = d0 < 0 ? 4.0f : 1.0f, q1 = d1 < 0 ? 4.0f : 1.0f;
            const float go0 = scale * q0 * d0, go1 = scale * q1 * d1;
            lsum += q0 * d0 * d0 + q1 * d1 * d1;
            gb30 += go0;
            gb31 += go1;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                gz2[j][e] = (go0 * w30[j] + go1 * w31[j]) * dz2[j];
                if (j == g) {
                    gw30 += go0 * h2[j];
                    gw31 += go1 * h2[j];
                    gb2 += gz2[j][e];
                }
            }
        }
        // W2's gradient, columns 16 g ..: sum over samples of gz2[k] h1[i]
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j == g)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < 4; ++i) gW2[i] = mma4(gz2[i][e], h1[j][e], gW2[i]);
        // back through W2 to block g of layer 1
        wave_sync();
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) A[(4 * lk + e) * LDW + 16 * j + li] = gz2[j][e];
        wave_sync();
        f4 gh1 = {0, 0, 0, 0}, gh1b = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < 16; s += 2) {
            gh1 = mma4(A[li * LDW + 4 * s + lk], W[(4 * s + lk) * LDW + 16 * g + li], gh1);
            gh1b = mma4(A[li * LDW + 4 * s + 4 + lk], W[(4 * s + 4 + lk) * LDW + 16 * g + li], gh1b);
        }
        // W1's gradient, rows 16 g ..; column 12 of the samples is one (b1)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int b = s0 + 4 * lk + e;
            const float xs = li < NF ? (b < B ? (x[(int64_t)b * NF + li] - xm) / xd : 0.0f) : (li == NF ? 1.0f : 0.0f);
            gW1 = mma4((gh1[e] + gh1b[e]) * dz1[e], xs, gW1);
        }
        wave_sync();   // the next pass, or the sums, overwrite the rows
    }
    // the waves' sums side by side in LDS, then added in wave order
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) A[(16 * i + 4 * lk + e) * 16 + li] = gW2[i][e];
    float *const P = part[w];
#pragma unroll
    for (int e = 0; e < 4; ++e) P[(4 * lk + e) * 16 + li] = gW1[e];
    gb2 = sum4(gb2);
    gw30 = sum4(gw30);
    gw31 = sum4(gw31);
    gb30 = sum4(gb30);
    gb31 = sum4(gb31);
    lsum = sum4(lsum);
    if (l < 16) {
        P[256 + l] = gb2;
        P[272 + l] = gw30;
        P[288 + l] = gw31;
    }
    if (l == 0) {
        P[304] = gb30;
        P[305] = gb31;
        P[306] = lsum;
    }
    __syncthreads();
    for (int i = t; i < NH * 16; i += NWAVE * 64) {
        float v = 0.0f;
        for (int q = 0; q < NWAVE; ++q) v += act[q][i];
        grad[OFF_W2 + (i >> 4) * NH + 16 * g + (i & 15)] = v;
    }
    if (t < 307) {
        float v = 0.0f;
        for (int q = 0; q < NWAVE; ++q) v += part[q][t];
        const int r = t >> 4, c = t & 15;
        if (t < 256) {
            if (c < NF) grad[(16 * g + r) * NF + c] = v;
            else if (c == NF) grad[OFF_B1 + 16 * g + r] = v;
        } else if (t < 272) {
            grad[OFF_B2 + 16 * g + c] = v;
        } else if (t < 288) {
            grad[OFF_W3 + 16 * g + c] = v;
        } else if (t < 304) {
            grad[OFF_W3 + NH + 16 * g + c] = v;
        } else if (g == 0) {
            if (t < 306) grad[OFF_B3 + t - 304] = v;
            else *loss_out = v / (float)(B * NO);
        }
    }
}

// omb1 = 1 - beta1 and omb2 = 1 - beta2 are formed on the host from the
// double-precision hyper-parameters and rounded once to FP32.
__global__ void k_mlp_adam(float *p, const float *g, float *m, float *v, float lr, float b1, float b2, float omb1,
                           float omb2, float eps, float bc1, float bc2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NPAR) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + omb1 * gi;
    const float vi = b2 * v[i] + omb2 * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

extern "C" int nolsm_mlp_forward(const float *d_params, const float *d_norm, const float *d_x, int32_t B,
                                 float *d_out, void *stream) {
    if (!d_params || !d_norm || !d_x || !d_out || B < 0) return NOLSM_E_ARG;
    if (B == 0) return NOLSM_OK;
    hipLaunchKernelGGL(k_mlp_forward, dim3((B + 255) / 256), dim3(256), 0, (hipStream_t)stream, d_params, d_norm,
                       d_x, B, d_out);
    return hipGetLastError() == hipSuccess ? NOLSM_OK : NOLSM_E_HIP;
}

extern "C" int nolsm_mlp_loss_grad(const float *d_params, const float *d_norm, const float *d_x, const float *d_y,
                                   int32_t B, float *d_grad, float *d_loss, void *stream) {
    if (!d_params || !d_norm || !d_x || !d_y || !d_grad || !d_loss || B < 1) return NOLSM_E_ARG;
    hipLaunchKernelGGL(k_mlp_loss_grad, dim3(NH / 16), dim3(NWAVE * 64), 0, (hipStream_t)stream, d_params, d_norm, d_x, d_y, B,
                       d_grad, d_loss);
    return hipGetLastError() == hipSuccess ? NOLSM_OK : NOLSM_E_HIP;
}

extern "C" int nolsm_mlp_adam(float *d_params, const float *d_grad, float *d_m, float *d_v, int32_t t, double lr,
                              double beta1, double beta2, double eps, void *stream) {
    if (!d_params || !d_grad || !d_m || !d_v || t < 1) return NOLSM_E_ARG;
    const float bc1 = (float)(1.0 - pow(beta1, (double)t));
    const float bc2 = (float)(1.0 - pow(beta2, (double)t));
    const float omb1 = (float)(1.0 - beta1), omb2 = (float)(1.0 - beta2);
    hipLaunchKernelGGL(k_mlp_adam, dim3((NPAR + 255) / 256), dim3(256), 0, (hipStream_t)stream, d_params, d_grad,
                       d_m, d_v, (float)lr, (float)beta1, (float)beta2, omb1, omb2, (float)eps, bc1, bc2);
    return hipGetLastError() == hipSuccess ? NOLSM_OK : NOLSM_E_HIP;
}
