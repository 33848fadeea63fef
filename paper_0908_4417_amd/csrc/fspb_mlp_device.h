/*
 * Wave-level building blocks of the kernel surrogate (see fspb_mlp.h):
 * BF16 rounding, SiLU, W2 fragments for v_mfma_f32_16x16x32_bf16, and the
 * forward pass of 64 samples (one per lane) used both by training and by the
 * fused fill.
 *
 * v_mfma_f32_16x16x32_bf16 operand layout (one wave): lane l supplies
 * A[m = l % 16][k = 8 (l / 16) + i] and B[k = 8 (l / 16) + i][n = l % 16],
 * i = 0..7, and receives D[m = 4 (l / 16) + i][n = l % 16], i = 0..3.
 */
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fspb_mlp.h"

namespace fspb {
namespace mlp {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kTStride = 72;     // bf16 per row of a 64x64 tile read as A/B fragments (144 B rows)

__device__ inline int lane() { return threadIdx.x & 63; }

/* float -> bfloat16 bits, round to nearest even (finite inputs). */
__device__ inline uint16_t bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ inline float sigmoid(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }

__device__ inline f32x4 mfma(const bf16x8 &a, const bf16x8 &b, const f32x4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ inline bf16x8 frag(const uint16_t *p) { return *reinterpret_cast<const bf16x8 *>(p); }

/* Fragments of W2 (A operand of W2 h1^T, and B operand of h1 W2^T): b[ct][ks] covers outputs
 * 16 ct .. 16 ct + 15 and inputs 32 ks .. 32 ks + 31. */
struct W2Frags {
    bf16x8 b[4][2];
};

__device__ inline void load_w2_frags(const uint16_t *__restrict__ w2, W2Frags &f)
{
    const int n = lane() & 15, kq = (lane() >> 4) * 8;
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) f.b[ct][ks] = frag(w2 + (16 * ct + n) * kMlpH + 32 * ks + kq);
}

/* Features of the training box, [-1, 1]^4 (square-root stretch of d, |u|, |v|). */
__device__ inline float feature_a(float a) { return (a - 0.625f) * (1.0f / 0.375f); }
__device__ inline void features(float d, float au, float av, float a, float x[4])
{
    x[0] = 2.0f * __builtin_sqrtf(fmaxf(d, 0.0f) * (1.0f / 30.0f)) - 1.0f;
    x[1] = 2.0f * __builtin_sqrtf(au * (1.0f / 3.0f)) - 1.0f;
    x[2] = 2.0f * __builtin_sqrtf(av * (1.0f / 3.0f)) - 1.0f;
    x[3] = feature_a(a);
}

/*
 * The FP32 parameters of the forward pass as it reads them (LDS), built by
 * stage_weights with every thread of the workgroup.
 */
struct Weights {
    float4 w1[kMlpH];      // W1[o][0..2] and, with FOLD, the bias with the fourth input's term added; else W1[o][3]
    float b1[kMlpH];       // not with FOLD
    alignas(16) float b2[kMlpH], w3[kMlpH];
};

template <bool FOLD>
__device__ inline void stage_weights(Weights &W, const float *__restrict__ p, float x3, int tid, int n_threads)
{
    for (int o = tid; o < kMlpH; o += n_threads) {
        const float *w = p + kOffW1 + o * kMlpIn;
        W.w1[o] = make_float4(w[0], w[1], w[2], FOLD ? fmaf(w[3], x3, p[kOffB1 + o]) : w[3]);
        W.b1[o] = p[kOffB1 + o];
        W.b2[o] = p[kOffB2 + o];
        W.w3[o] = p[kOffW3 + o];
    }
}

__device__ inline uint32_t bf16_pair(float a, float b)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 q = __builtin_convertvector((f32x2){a, b}, bf16x2);
    uint32_t u;
    __builtin_memcpy(&u, &q, sizeof u);
    return u;
}

/*
 * Forward pass of 64 samples, sample = lane, features x.  With FOLD the fourth
 * feature is the same for every sample and folded into W (x[3] is not read).
 * Returns the output for the lane's sample, without the last bias.  Every lane
 * of the wave must call it.
 *
 * Layer 2 is computed as W2 h1^T, so that h1 is its B operand: lane (g, n)
 * makes the 16 hidden values of sample n of a tile that it supplies itself
 * (inputs 32 ks + 8 g + i) and h1 needs neither LDS nor a transpose; the results
 * of a sample lie in four lanes, so the last layer's sum takes two exchanges per
 * 16 samples.  Weights are read from LDS once for all four tiles.  Bound by the
 * 256 quarter-rate instructions of the 128 SiLUs per sample: the
 * surrogate fill of a pelvis plan (9 x 576 beamlets, 4.1e8 entries) takes 15.4 ms, 24.9 with
 * h1 and the results exchanged through LDS (1125 and 1529 vector instructions per 64 entries).
 */
template <bool FOLD>
__device__ inline float forward_wave(const Weights &W, const W2Frags &wf, const float x[4])
{
    constexpr int kX = FOLD ? kMlpIn - 1 : kMlpIn;
    const int l = lane(), n = l & 15, g = l >> 4;
    float xs[4][kX];
#pragma unroll
    for (int st = 0; st < 4; ++st)
#pragma unroll
        for (int k = 0; k < kX; ++k) xs[st][k] = __shfl(x[k], 16 * st + n, 64);
    // layer 1 (FP32), h1 rounded to BF16
    uint32_t h[4][2][4];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int o = 32 * ks + 8 * g + 2 * i;
            const float4 wa = W.w1[o], wb = W.w1[o + 1];
            const float ba = FOLD ? wa.w : W.b1[o], bb = FOLD ? wb.w : W.b1[o + 1];
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                float za = fmaf(wa.z, xs[st][2], fmaf(wa.y, xs[st][1], fmaf(wa.x, xs[st][0], ba)));
                float zb = fmaf(wb.z, xs[st][2], fmaf(wb.y, xs[st][1], fmaf(wb.x, xs[st][0], bb)));
                if (!FOLD) {
                    za = fmaf(wa.w, xs[st][kX - 1], za);
                    zb = fmaf(wb.w, xs[st][kX - 1], zb);
                }
                h[st][ks][i] = bf16_pair(za * sigmoid(za), zb * sigmoid(zb));
            }
        }
    // layer 2 on the matrix cores, layer 3 as a sum over each lane's 16 outputs
    float part[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
        const f32x4 b2 = *reinterpret_cast<const f32x4 *>(&W.b2[16 * ct + 4 * g]);
        const f32x4 w3 = *reinterpret_cast<const f32x4 *>(&W.w3[16 * ct + 4 * g]);
#pragma unroll
        for (int st = 0; st < 4; ++st) {
            f32x4 z = b2;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                bf16x8 q;
                __builtin_memcpy(&q, h[st][ks], sizeof q);
                z = mfma(wf.b[ct][ks], q, z);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) part[st] = fmaf(z[i] * sigmoid(z[i]), w3[i], part[st]);
        }
    }
    float y = 0.0f;
#pragma unroll
    for (int st = 0; st < 4; ++st) {
        part[st] += __shfl_xor(part[st], 16, 64);
        part[st] += __shfl_xor(part[st], 32, 64);
        y = g == st ? part[st] : y;
    }
    return y;
}

}  // namespace mlp
}  // namespace fspb
