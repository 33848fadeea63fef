/*
 * Training, evaluation and target-generation kernels of the kernel surrogate
 * (4 -> 64 -> 64 -> 1 SiLU perceptron; see fspb_mlp.h).
 *
 *   k_mlp_targets  analytic K(d, u, v, a) = PDD(d) F(u, v; a, a, d) and the
 *                  features of each sample (one thread per sample)
 *   k_mlp_forward  surrogate outputs, 64 samples per wave
 *   k_mlp_grad     forward + backward of 64 samples per workgroup; BF16 matrix
 *                  cores for h1 W2^T, dz2^T h1 and dz2 W2; gradient partials
 *                  per workgroup (deterministic, no atomics)
 *   k_mlp_reduce   sum of the partials, then Adam on the FP32 masters and
 *                  fresh BF16 copies of W2 (or the plain gradient)
 */
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "fspb_mlp_device.h"

namespace fspb {

namespace {

using namespace mlp;

/* erfc(x / kScale), x = z * kScale >= 0, from a global piecewise-quadratic table. */
__device__ inline float erfc_tab(const float4 *__restrict__ tab, float x)
{
    const float xc = fminf(x, 511.999f);
    const int k = (int)xc;
    const float f = __builtin_amdgcn_fractf(xc);
    const float4 c = tab[k];
    return fmaf(fmaf(c.z, f, c.y), f, c.x);
}

__device__ inline float bracket(const float4 *__restrict__ tab, float ax, float h, float isk)
{
    const float hk = h * isk;
    const float ea = erfc_tab(tab, fabsf(fmaf(-ax, isk, hk)));
    const float eb = erfc_tab(tab, fmaf(ax, isk, hk));
    return (ax <= h ? 2.0f - ea : ea) - eb;
}

__global__ __launch_bounds__(256) void k_mlp_targets(MlpTargetDev K, const float *__restrict__ samples, int64_t n,
                                                     float *__restrict__ feats, float *__restrict__ targets)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float d = samples[4 * i], au = fabsf(samples[4 * i + 1]), av = fabsf(samples[4 * i + 2]);
    const float a = samples[4 * i + 3];
    float x[4];
    features(d, au, av, a, x);
#pragma unroll
    for (int k = 0; k < 4; ++k) feats[4 * i + k] = x[k];
    const float xp = fminf(fmaxf(d * K.pdd_inv_step, 0.0f), K.pdd_max);
    const int kp = min((int)xp, K.n_pdd - 2);
    const float fp = xp - (float)kp;
    const float pdd = fmaf(fp, K.pdd[kp + 1] - K.pdd[kp], K.pdd[kp]);
    constexpr float kIs = 0.70710678118654752f * 128.0f;
    float L = 0.0f;
    for (int t = 0; t < K.n_terms; ++t) {
        const float isk = kIs / fmaf(K.sig1[t], d, K.sig0[t]);
        const float h = 0.5f * K.c2[t] * a;
        L = fmaf(K.w4[t] * bracket(K.erfc_tab, au, h, isk), bracket(K.erfc_tab, av, h, isk), L);
    }
    targets[i] = pdd * L;
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_mlp_forward(MlpDev m, const float *__restrict__ feats, int64_t n,
                                                     float *__restrict__ out)
{
    __shared__ __align__(16) Weights W;
    stage_weights<false>(W, m.p, 0.0f, threadIdx.x, 256);
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    W2Frags wf;
    load_w2_frags(m.w2, wf);
    float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (i < n)
        for (int k = 0; k < 4; ++k) x[k] = feats[4 * i + k];
    __syncthreads();
    const float y = forward_wave<false>(W, wf, x) + m.p[kOffB3];
    if (i < n) out[i] = y;
}

/*
 * Gradient partials of 64 samples: a workgroup of four waves.  A wave makes 16 of
 * the hidden columns of layer 1, then takes 16 of the samples through layer 2,
 * the loss and the backward of both layers, and makes 16 rows of dW2.  The column
 * sums run over the samples in one order whatever the number of waves, so that a
 * network's training does not depend on the split: the waves extend them in turn
 * (s_col), each by its 16 samples.
 *
 * Bound by latency: a training step of 16384 samples is 256 workgroups, one per
 * CU.  16384 samples: 9.6 us (one wave per 64 samples: 16.4 us).
 */
constexpr int kGradBlock = 256;
constexpr int kColKinds = 3 + kMlpIn;     // b2, w3, b1, w1[0..3]
__global__ __launch_bounds__(kGradBlock) void k_mlp_grad(MlpDev m, const float *__restrict__ feats,
                                                         const float *__restrict__ targets, int64_t n_total,
                                                         int64_t base, int64_t n_step, uint64_t stride,
                                                         uint64_t offset, float inv_count,
                                                         float *__restrict__ partials)
{
    __shared__ float s_x[64][4];
    __shared__ float s_z1[64][65];
    __shared__ __align__(16) uint16_t s_h1[64 * kTStride];      // [sample][in]; from the backward on dz2 [sample][out]
    __shared__ __align__(16) uint16_t s_h1t[64 * kTStride];     // [in][sample]
    __shared__ __align__(16) uint16_t s_dz2t[64 * kTStride];    // [out][sample]
    __shared__ float s_col[4 * kColKinds][64];                  // column sums, per 16-column tile and lane
    __shared__ float s_sum[2][64];                              // gb3, loss per lane
    const int l = lane(), n = l & 15, g = l >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t mine = (int64_t)blockIdx.x * 64 + l;
    const bool valid = mine < n_step;
    const int64_t idx = valid ? (int64_t)((offset + (uint64_t)(base + mine) * stride) % (uint64_t)n_total) : 0;
    float x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    float t = 0.0f;
    if (valid) {
        for (int k = 0; k < 4; ++k) x[k] = feats[4 * idx + k];
        t = targets[idx];
    }
    const float *p = m.p;
    W2Frags wf;
    load_w2_frags(m.w2, wf);
    bf16x8 bt[4][2];                                            // W2 as the B operand of dz2 W2
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) bt[nt][ks] = frag(m.w2t + (16 * nt + n) * kMlpH + 32 * ks + 8 * g);
    float b2[4], w3[4];
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
        b2[ct] = p[kOffB2 + 16 * ct + n];
        w3[ct] = p[kOffW3 + 16 * ct + n];
    }
    // ---- layer 1: 16 hidden columns of every sample
    if (wave == 0)
        for (int k = 0; k < 4; ++k) s_x[l][k] = x[k];
#pragma unroll
    for (int j = 0; j < 16; j += 2) {
        uint32_t pair = 0;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int o = 16 * wave + j + e;
            float z = p[kOffB1 + o];
#pragma unroll
            for (int k = 0; k < kMlpIn; ++k) z = fmaf(p[kOffW1 + o * kMlpIn + k], x[k], z);
            s_z1[l][o] = z;
            const uint16_t h = bf16_bits(z * sigmoid(z));
            s_h1t[o * kTStride + l] = h;
            pair |= (uint32_t)h << (16 * e);
        }
        *reinterpret_cast<uint32_t *>(s_h1 + l * kTStride + 16 * wave + j) = pair;
    }
    __syncthreads();
    // ---- layer 2 (matrix cores) of the wave's 16 samples, layer 3, loss, backward to dz2
    float f2[4][4], q2[4][4], zs[4][4], dy[4], r2[4];           // dz2 = f2 q2
    bool vrow[4];
    {
        f32x4 acc[4];
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) acc[ct] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const bf16x8 a = frag(s_h1 + (16 * wave + n) * kTStride + 32 * ks + 8 * g);
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) acc[ct] = mfma(a, wf.b[ct][ks], acc[ct]);
        }
        float part[4] = {0, 0, 0, 0};
#pragma unroll
        for (int ct = 0; ct < 4; ++ct)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float z = acc[ct][i] + b2[ct], s = sigmoid(z);
                zs[ct][i] = z * s;
                q2[ct][i] = s * fmaf(z, 1.0f - s, 1.0f);
                part[i] = fmaf(zs[ct][i], w3[ct], part[i]);
            }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int mm = 1; mm < 16; mm <<= 1) part[i] += __shfl_xor(part[i], mm, 64);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 16 * wave + 4 * g + i;
            const float trow = __shfl(t, row, 64);
            vrow[i] = (int64_t)blockIdx.x * 64 + row < n_step;
            r2[i] = part[i] + p[kOffB3] - trow;
            dy[i] = vrow[i] ? 2.0f * r2[i] * inv_count : 0.0f;
        }
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
            const int col = 16 * ct + n;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 16 * wave + 4 * g + i;
                f2[ct][i] = dy[i] * w3[ct];
                const uint16_t q = bf16_bits(f2[ct][i] * q2[ct][i]);
                s_h1[row * kTStride + col] = q;                 // the wave's own rows: h1's are read
                s_dz2t[col * kTStride + row] = q;
            }
        }
    }
    // ---- dh1 = dz2 W2 of the wave's samples, dz1 = dh1 silu'(z1)
    f32x4 dh[4];
    float q1[4][4];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // dz2 crosses lanes of the wave
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) dh[nt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const bf16x8 a = frag(s_h1 + (16 * wave + n) * kTStride + 32 * ks + 8 * g);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) dh[nt] = mfma(a, bt[nt][ks], dh[nt]);
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float z = s_z1[16 * wave + 4 * g + i][16 * nt + n], s = sigmoid(z);
            q1[nt][i] = s * fmaf(z, 1.0f - s, 1.0f);
        }
    float xr[4][kMlpIn];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < kMlpIn; ++k) xr[i][k] = s_x[16 * wave + 4 * g + i][k];
    // ---- column sums: wave after wave
    float *out = partials + (size_t)blockIdx.x * kPartialStride;
    for (int turn = 0; turn < 4; ++turn) {
        if (wave == turn) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                float v[kColKinds];
#pragma unroll
                for (int k = 0; k < kColKinds; ++k) v[k] = turn ? s_col[kColKinds * c + k][l] : 0.0f;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[0] = fmaf(f2[c][i], q2[c][i], v[0]);
                    v[1] = fmaf(dy[i], zs[c][i], v[1]);
                    v[2] = fmaf(dh[c][i], q1[c][i], v[2]);
                    const float dz = dh[c][i] * q1[c][i];
#pragma unroll
                    for (int k = 0; k < kMlpIn; ++k) v[3 + k] = fmaf(dz, xr[i][k], v[3 + k]);
                }
#pragma unroll
                for (int k = 0; k < kColKinds; ++k) s_col[kColKinds * c + k][l] = v[k];
            }
            float gb3 = turn ? s_sum[0][l] : 0.0f, loss = turn ? s_sum[1][l] : 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (n == 0 && vrow[i]) {
                    gb3 += dy[i];
                    loss = fmaf(r2[i], r2[i], loss);
                }
            s_sum[0][l] = gb3;
            s_sum[1][l] = loss;
        }
        __syncthreads();
    }
    // ---- dW2 = dz2^T h1 (K = the 64 samples), 16 rows per wave
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        f32x4 acc = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
            acc = mfma(frag(s_dz2t + (16 * wave + n) * kTStride + 32 * ks + 8 * g),
                       frag(s_h1t + (16 * nt + n) * kTStride + 32 * ks + 8 * g), acc);
#pragma unroll
        for (int i = 0; i < 4; ++i) out[kOffW2 + (16 * wave + 4 * g + i) * kMlpH + 16 * nt + n] = acc[i];
    }
    // ---- the four lane groups' column sums
    for (int v = threadIdx.x; v < 64 * kColKinds; v += kGradBlock) {
        const int k = v >> 6, col = v & 63, c = col >> 4;
        const float *s = &s_col[kColKinds * c + k][col & 15];
        const int at = k == 0 ? kOffB2 + col : k == 1 ? kOffW3 + col : k == 2 ? kOffB1 + col
                                                                             : kOffW1 + col * kMlpIn + k - 3;
        out[at] = (s[0] + s[16]) + (s[32] + s[48]);
    }
    if (threadIdx.x < 2) {
        const float *s = s_sum[threadIdx.x];
        out[threadIdx.x ? kMlpParams : kOffB3] = (s[0] + s[16]) + (s[32] + s[48]);
    }
}

/*
 * Sum of the gradient partials and the Adam step.  A thread adds its parameter's
 * partials in order, one after another (training stays deterministic and does not
 * depend on the split), and the eight waves of a workgroup take turns at it: all
 * of them load 32 partials of the same 64 parameters, then each extends the sum.
 * Bound by the latency of the loads, so they are issued together: 256 partials
 * 4.6 us (one wave with 32 loads in flight: 8 us).
 */
constexpr int kReduceParams = 64;
constexpr int kReduceWaves = 8;
constexpr int kReduceBatch = 32;
__global__ __launch_bounds__(kReduceParams *kReduceWaves) void k_mlp_reduce(
    float *__restrict__ params, float *__restrict__ m1, float *__restrict__ m2, uint16_t *__restrict__ w2,
    uint16_t *__restrict__ w2t, const float *__restrict__ partials, int n_part, int adam, float lr, float b1, float b2,
    float eps, float bc1, float bc2, float *__restrict__ grad_out, float *__restrict__ loss_out)
{
    __shared__ float s_sum[kReduceParams];
    const int l = threadIdx.x % kReduceParams, k = blockIdx.x * kReduceParams + l;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kReduceParams);
    const bool mine = k <= kMlpParams, last = wave == kReduceWaves - 1;
    const bool update = adam && last && k < kMlpParams;
    const float o1 = update ? m1[k] : 0.0f, o2 = update ? m2[k] : 0.0f, op = update ? params[k] : 0.0f;
    float gsum = 0.0f;
    for (int w0 = 0; w0 < n_part; w0 += kReduceBatch * kReduceWaves) {
        const int w = w0 + kReduceBatch * wave, cnt = min(n_part - w, kReduceBatch);
        float v[kReduceBatch];
        if (mine) {
            const float *q = partials + (size_t)w * kPartialStride + k;
            if (cnt == kReduceBatch) {
#pragma unroll
                for (int u = 0; u < kReduceBatch; ++u) v[u] = q[(size_t)u * kPartialStride];
            } else {
#pragma unroll
                for (int u = 0; u < kReduceBatch; ++u) v[u] = u < cnt ? q[(size_t)u * kPartialStride] : 0.0f;
            }
        }
        for (int turn = 0; turn < kReduceWaves; ++turn) {
            if (wave == turn && mine) {
                gsum = w0 + turn ? s_sum[l] : 0.0f;
#pragma unroll
                for (int u = 0; u < kReduceBatch; ++u)
                    if (u < cnt) gsum += v[u];
                s_sum[l] = gsum;
            }
            __syncthreads();
        }
    }
    if (!last || !mine) return;
    if (k == kMlpParams && loss_out) __hip_atomic_store(loss_out, gsum, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    else if (grad_out) grad_out[k] = gsum;
    if (!update) return;
    const float mm = fmaf(1.0f - b1, gsum, b1 * o1);
    const float vv = fmaf(gsum, (1.0f - b2) * gsum, b2 * o2);
    m1[k] = mm;
    m2[k] = vv;
    const float pk = op - lr * (mm / bc1) / (sqrtf(vv / bc2) + eps);
    params[k] = pk;
    if (k >= kOffW2 && k < kOffB2) {
        const int o = (k - kOffW2) / kMlpH, i = (k - kOffW2) % kMlpH;
        const uint16_t q = bf16_bits(pk);
        w2[o * kMlpH + i] = q;
        w2t[i * kMlpH + o] = q;
    }
}

__global__ __launch_bounds__(256) void k_mlp_bf16_copies(const float *__restrict__ params, uint16_t *__restrict__ w2,
                                                         uint16_t *__restrict__ w2t)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= kMlpH * kMlpH) return;
    const int o = k / kMlpH, i = k % kMlpH;
    const uint16_t q = bf16_bits(params[kOffW2 + k]);
    w2[o * kMlpH + i] = q;
    w2t[i * kMlpH + o] = q;
}

}  // namespace

hipError_t launch_mlp_targets(const MlpTargetDev &k, const float *samples, int64_t n, float *features, float *targets,
                              hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_targets, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, k, samples, n, features,
                       targets);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const MlpDev &m, const float *features, int64_t n, float *out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, m, features, n, out);
    return hipGetLastError();
}

hipError_t launch_mlp_grad(const MlpDev &m, const float *features, const float *targets, int64_t n_total, int64_t base,
                           int64_t n_step, uint64_t stride, uint64_t offset, float inv_count, float *partials,
                           hipStream_t s)
{
    const unsigned groups = (unsigned)((n_step + 63) / 64);
    hipLaunchKernelGGL(k_mlp_grad, dim3(groups), dim3(kGradBlock), 0, s, m, features, targets, n_total, base, n_step, stride,
                       offset, inv_count, partials);
    return hipGetLastError();
}

hipError_t launch_mlp_reduce(float *params, float *m1, float *m2, uint16_t *w2, uint16_t *w2t, const float *partials,
                             int n_part, int adam, float lr, float b1, float b2, float eps, float bc1, float bc2,
                             float *grad_out, float *loss_out, hipStream_t s)
{
    hipLaunchKernelGGL(k_mlp_reduce, dim3((kMlpParams + 1 + kReduceParams - 1) / kReduceParams),
                       dim3(kReduceParams * kReduceWaves), 0, s, params, m1, m2, w2, w2t, partials, n_part, adam, lr, b1,
                       b2, eps, bc1, bc2, grad_out, loss_out);
    return hipGetLastError();
}

hipError_t launch_mlp_bf16_copies(const float *params, uint16_t *w2, uint16_t *w2t, hipStream_t s)
{
    hipLaunchKernelGGL(k_mlp_bf16_copies, dim3((kMlpH * kMlpH + 255) / 256), dim3(256), 0, s, params, w2, w2t);
    return hipGetLastError();
}

}  // namespace fspb
