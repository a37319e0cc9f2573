// Pieces of the split-precision kernels: an fp32 number as two f16 or three bf16 parts, the range
// in which the f16 parts hold it, and the epilogue that chains the posterior heads and the decoder's
// hidden layer from the encoder's accumulators in bf16 parts.
#pragma once

#include <hip/hip_runtime.h>

#include "mfma_common.h"

namespace enova {

namespace {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));

// Normalised inputs are scaled by 2^4 before they are split: a |v| up to 4000 fits f16, and the parts
// hold every one to 2^-29 (to 23 bits from 2^-6 on). Windows with an input beyond 4000, and windows
// whose every input is below 2^-2, where 2^-29 would be more than the rounding of an fp32 sum, take the
// fp32 kernel (in scaled units: kSplitMax, kSplitMin).
constexpr float kSplitScale = 16.0f, kSplitUnscale = 1.0f / 16.0f;
constexpr float kSplitMax = 64000.0f, kSplitMin = 4.0f;

// 1/std of the scaled values (the scale is a power of two: (x - mean) * split_rinv(std) is exactly
// kSplitScale times (x - mean) * (1 / std)).
__device__ __forceinline__ float split_rinv(float std) { return (1.0f / std) * kSplitScale; }

// wm: the bits of a window's largest scaled |v| (an infinity's or a NaN's where one is not finite).
__device__ __forceinline__ bool split_outside(unsigned wm)
{
    return wm > __builtin_bit_cast(unsigned, kSplitMax) || (wm != 0u && wm < __builtin_bit_cast(unsigned, kSplitMin));
}

__device__ __forceinline__ void split_f16x8(const float (&v)[8], v8h &hi, v8h &lo)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const _Float16 h = static_cast<_Float16>(v[e]);
        hi[e] = h;
        lo[e] = static_cast<_Float16>(v[e] - static_cast<float>(h));
    }
}

// x as three bf16 parts (round to nearest each time: 24 bits and more between them).
__device__ __forceinline__ void split_bf16x8x3(const float (&x)[8], v8bf (&q)[3])
{
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const __bf16 a = static_cast<__bf16>(x[t]);
        const float r = x[t] - static_cast<float>(a);
        const __bf16 b = static_cast<__bf16>(r);
        q[0][t] = a;
        q[1][t] = b;
        q[2][t] = static_cast<__bf16>(r - static_cast<float>(b));
    }
}

// c += A B from three parts each: the six products down to 2^-16 of the largest, smallest first.
__device__ __forceinline__ v16f mfma6_bf16(const uint4 (&a)[3], const v8bf (&b)[3], v16f c)
{
    const v8bf a0 = __builtin_bit_cast(v8bf, a[0]), a1 = __builtin_bit_cast(v8bf, a[1]),
               a2 = __builtin_bit_cast(v8bf, a[2]);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a2, b[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b[2], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b[1], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1, b[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b[1], c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0, b[0], c, 0, 0, 0);
}

struct SplitEpiArgs {
    const uint4 *whx;            // heads [HBT][2][3 parts][64] (slot layout of the bf16 heads)
    const uint4 *wdx;            // decoder hidden layer [HBT][3 parts][64]
    const float *b1, *sc;        // bias and accumulator scale of each hidden row
    const float *bd1, *u, *bh;
    float *xchg;                 // as EpiArgs
    int lane, half, wave, wh, wn;
};

// As score_epilogue, for accumulators that hold sc[h]^-1 times the pre-activations.
template <int HB, int NBW, int WH, int NW, int ACT, typename StoreFn>
__device__ __forceinline__ void split_epilogue(v16f (&acc)[HB][NBW], const SplitEpiArgs &e, StoreFn store)
{
    // (tanhf's temporaries leave room for one window block at a time)
    constexpr int NG = ACT == ENOVA_TANH ? 1 : EpiPass<NBW>::NG;
    const int lane = e.lane, half = e.half, wave = e.wave, wh = e.wh, wn = e.wn;
    float *xz = e.xchg;
    float *xd = xz + NW * NG * 16 * 64;
#pragma unroll
    for (int g0 = 0; g0 < NBW; g0 += NG) {
        asm volatile("" ::: "memory");
        v16f z[NG];
#pragma unroll
        for (int i = 0; i < NG; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                z[i][r] = 0.0f;
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) {
            const int hbg = wh * HB + hb;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                uint4 w[3];
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    w[q] = e.whx[((hbg * 2 + m) * 3 + q) * 64 + lane];
#pragma unroll
                for (int i = 0; i < NG; ++i) {
                    float hv[8];
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const int h = hbg * 32 + crow(8 * m + t, half);
                        hv[t] = act_fn<ACT>(fmaf(acc[hb][g0 + i][8 * m + t], e.sc[h], e.b1[h]));
                    }
                    v8bf q[3];
                    split_bf16x8x3(hv, q);
                    z[i] = mfma6_bf16(w, q, z[i]);
                }
            }
        }
        if constexpr (WH > 1) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NG; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    xz[((wave * NG + i) * 16 + r) * 64 + lane] = z[i][r];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NG; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float t = 0.0f;
#pragma unroll
                    for (int w2 = 0; w2 < WH; ++w2)
                        t += xz[(((wn * WH + w2) * NG + i) * 16 + r) * 64 + lane];
                    z[i][r] = t;
                }
        }
        float kl[NG], dot[NG];
        v8bf mu[NG][3];
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            kl[i] = 0.0f;
            dot[i] = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                z[i][r] += e.bh[crow(r, half)];
                if (r < 8)
                    kl[i] += z[i][r] * z[i][r];
                else
                    kl[i] += kl_g(z[i][r]);
            }
            kl[i] += __shfl_xor(kl[i], 32);
            float mv[8];
#pragma unroll
            for (int t = 0; t < 8; ++t)
                mv[t] = z[i][t];
            split_bf16x8x3(mv, mu[i]);
        }
#pragma unroll
        for (int hb = 0; hb < HB; ++hb) {
            const int hbg = wh * HB + hb;
            uint4 w[3];
#pragma unroll
            for (int q = 0; q < 3; ++q)
                w[q] = e.wdx[(hbg * 3 + q) * 64 + lane];
            v16f d[NG];
#pragma unroll
            for (int i = 0; i < NG; ++i) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    d[i][r] = 0.0f;
                d[i] = mfma6_bf16(w, mu[i], d[i]);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int h = hbg * 32 + crow(r, half);
                const float uh = e.u[h];
                const float bh = e.bd1[h];
#pragma unroll
                for (int i = 0; i < NG; ++i)
                    dot[i] += uh * act_fn<ACT>(d[i][r] + bh);
            }
        }
        if constexpr (WH > 1) {
#pragma unroll
            for (int i = 0; i < NG; ++i)
                xd[(wave * NG + i) * 64 + lane] = dot[i];
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                float t = 0.0f;
#pragma unroll
                for (int w2 = 0; w2 < WH; ++w2)
                    t += xd[((wn * WH + w2) * NG + i) * 64 + lane];
                dot[i] = t;
            }
        }
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            dot[i] += __shfl_xor(dot[i], 32);
            store(g0 + i, 0.5f * kl[i], dot[i]);
        }
    }
}

}  // namespace

}  // namespace enova
