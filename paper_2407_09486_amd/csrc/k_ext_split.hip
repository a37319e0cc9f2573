// Fused detector-output variants (Section IV-B) of fp32 detectors on the 16-bit matrix cores: the
// KL score, md, the per-metric md vector and the reconstruction error of every window in one launch.
//
// As k_ext_fused, a tile is 256 consecutive windows of one stream whose raw super-rows are staged
// in LDS once; normalisation is per window and metric, so every lane normalises the window fragments
// that it feeds to the matrix cores. The products run as in k_score_split (see there for the error
// and the range): the normalised fragment, scaled by 2^4, is split into two f16 parts in registers,
// W1 comes as two f16 parts, and three products make one. The decoder output runs the same way: the
// hidden activations hd of a window are scaled by the power of two that puts the largest into
// [2^13, 2^14), split, and multiplied with the f16 parts of Wd2. Windows are padded to Mp = 8 or 16
// metrics a step, so that a lane's fragments always hold the same metrics, whatever the count: an odd
// count took the chunked pass before, which writes and reads every normalised window.
//
// Both contractions are bound by the matrix cores (power holds them to about 1.7 GHz); the split of
// a fragment is some 50 vector instructions for 12 matrix ops at 128 hidden units. Two window
// blocks share every weight fragment, also in the decoder: one block's parts of hd are 64
// registers, and fragments for one block alone would ask 85 bytes a clock of the L1.
// Measured on one MI355X, every output, before (k_ext_fused or the chunked pass) and now: 64 ragged
// streams of 16 metrics, W = 64, H = 128, per-window normalisation (2.1e6 windows) 9.39 -> 4.60 ms;
// 32 streams of 7 metrics, W = 60, H = 64, tanh, reference normalisation (3.6e5 windows) 1985 ->
// 300 us (most of it the chunked pass's trips through memory). The errors against 64 bits are
// smaller: scores 4.2e-7 -> 3.0e-7, md 6.1e-6 -> 4.4e-6, reconstruction error 2.3e-7 -> 5.1e-8
// on the first.
//
// Windows out of the parts' range (split.h) are marked and evaluated one by one by k_ext_list.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "split.h"
#include "variants_internal.h"

namespace enova {

namespace {

constexpr int kNb = kExtFusedNb;     // windows per tile
constexpr int kNbw = 2;              // 32-window blocks per wave

// A tile's entry in the tile map once some of its windows are left to k_ext_list.
__host__ __device__ __forceinline__ int split_mark(int s) { return -2 - s; }
__host__ __device__ __forceinline__ int split_marked(int entry) { return -2 - entry; }   // the stream, or < 0

// One metric of one window: v = (x - k) * ca, k the mean, scaled by kSplitScale, and the bits of its
// largest |v| (infinity when out of range or not finite). x(t), t < W: the metric's values. (With
// v = x * ca + cb the rounding of cb, at the scale of mean / std, doubles that of the mean.)
template <typename X>
__device__ __forceinline__ unsigned window_constants(X x, int W, int norm, float ref_mean, float ref_std, float &ca,
                                                     float &k)
{
    const float x0 = x(0);
    float mn = x0, mx = x0;
    bool finite;
    if (norm == ENOVA_NORM_WINDOW) {
        // shifted sums (shift: the window's first value): mean and population std
        const double inv_w = 1.0 / W, shift = static_cast<double>(x0);
        double s1 = 0.0, s2 = 0.0;
        for (int t = 0; t < W; ++t) {
            const float v = x(t);
            const double d = static_cast<double>(v) - shift;
            s1 += d;
            s2 = fma(d, d, s2);
            mn = fminf(mn, v);
            mx = fmaxf(mx, v);
        }
        const double mean = shift + s1 * inv_w;
        double var = (s2 - s1 * s1 * inv_w) * inv_w;
        finite = fabs(var) < INFINITY;         // NaN or infinite where a value was not
        var = var > 0.0 ? var : 0.0;
        double sd = sqrt(var);
        if (sd <= 1e-6 * fmax(1.0, fabs(mean)))
            sd = 1.0;   // constant metric inside the window
        ca = static_cast<float>(1.0 / sd) * kSplitScale;
        k = static_cast<float>(mean);
    } else {
        float odd = 0.0f;
        for (int t = 0; t < W; ++t) {
            const float v = x(t);
            odd = fmaf(v, 0.0f, odd);          // NaN where a value is not finite
            mn = fminf(mn, v);
            mx = fmaxf(mx, v);
        }
        finite = odd == 0.0f;
        ca = static_cast<float>(1.0 / static_cast<double>(ref_std)) * kSplitScale;
        k = ref_mean;
    }
    const float lo = fabsf((mn - k) * ca), hi = fabsf((mx - k) * ca);
    const bool in = lo <= kSplitMax && hi <= kSplitMax && finite;
    return in ? __float_as_uint(fmaxf(lo, hi)) : 0x7f800000u;
}

// Eight values of a window fragment, normalised, clamped to the range (only fragments of marked
// windows or under zero weights reach its ends) and split.
__device__ __forceinline__ void fragment(const float4 (&x)[2], const float (&ca)[8], const float (&k)[8], v8h &hi,
                                         v8h &lo)
{
    const float q[8] = {x[0].x, x[0].y, x[0].z, x[0].w, x[1].x, x[1].y, x[1].z, x[1].w};
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
        v[e] = __builtin_amdgcn_fmed3f((q[e] - k[e]) * ca[e], -kSplitMax, kSplitMax);
    split_f16x8(v, hi, lo);
}

// s += x with the rounding error of the sum kept in c and taken off the next term.
__device__ __forceinline__ void carry_add(float &s, float &c, float x)
{
    const float y = x - c, t = s + y;
    c = (t - s) - y;
    s = t;
}

// HB: 32-row hidden blocks; MC: 8-metric groups of a step (Mp = 8 MC).
template <int HB, int MC, int ACT>
__global__ __launch_bounds__(256, 2) void k_ext_split(ExtSplitParams p, ExtSplitShape g)
{
    constexpr int NT = 256, Mp = 8 * MC, HP = 32 * HB;
    constexpr int CP = 2 * Mp + 4;                // floats per window of the constants' table
    extern __shared__ uint4 lds[];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6, half = lane >> 5;

    const int64_t b = blockIdx.x;
    const int s = p.tile_stream[b];
    if (s < 0)
        return;
    const int64_t k0 = (b - p.tile_off[s]) * kNb;
    const int64_t ns = p.woff[s + 1] - p.woff[s];
    const int nv = static_cast<int>(ns - k0 < kNb ? ns - k0 : kNb);
    const int64_t srow = p.soff[s];
    const int64_t T = p.soff[s + 1] - srow;
    const int Q = g.Q, CPR = g.CPR, P = g.P, S = g.S, W = g.W, M = g.M;
    const int nrows = nv + Q - 1 + g.spare;

    // LDS: raw super-rows (pitch P 16-byte chunks, odd), per window its constants [ca | k] and the
    // bits of its largest |v|, bd2, and the epilogue's vectors
    uint4 *seg = lds;
    const int rows_alloc = kNb + Q - 1 + g.spare;
    float *cab = reinterpret_cast<float *>(seg + static_cast<size_t>(rows_alloc) * P);
    unsigned *wmx = reinterpret_cast<unsigned *>(cab + kNb * CP);
    float *s_bd2 = reinterpret_cast<float *>(wmx + kNb);
    float *s_b1 = s_bd2 + g.Dp;
    float *s_sc = s_b1 + HP, *s_bd1 = s_sc + HP, *s_bh = s_bd1 + HP;
    int *s_mark = reinterpret_cast<int *>(s_bh + 32);
    for (int i = tid; i < HP; i += NT) {
        s_b1[i] = p.b1[i];
        s_sc[i] = p.w1scale[i];
        s_bd1[i] = p.bd1[i];
    }
    for (int i = tid; i < g.Dp; i += NT)
        s_bd2[i] = p.bd2[i];
    if (tid < 32)
        s_bh[tid] = p.bh[tid];
    wmx[tid] = 0u;
    if (tid == 0)
        *s_mark = 0;

    // ---- stage the raw super-rows (zero past the stream's end and in the padding)
    {
        const int64_t base = (srow + k0 * S) * M, avail = (T - k0 * S) * M;
        const float *x = p.x + base;
        const bool vec = M == Mp && reinterpret_cast<uintptr_t>(x) % 16 == 0;
        const int C4 = 2 * CPR;                    // 16-byte chunks of a row
        if (vec) {
            constexpr int SU = 8;
            const int n_chunks = nrows * C4;
            for (int i0 = tid; i0 < n_chunks; i0 += NT * SU) {
                float4 v[SU];
#pragma unroll
                for (int u = 0; u < SU; ++u) {
                    const int idx = i0 + u * NT;
                    v[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                    if (idx < n_chunks && static_cast<int64_t>(idx + 1) * 4 <= avail)
                        v[u] = reinterpret_cast<const float4 *>(x)[idx];
                }
#pragma unroll
                for (int u = 0; u < SU; ++u) {
                    const int idx = i0 + u * NT;
                    if (idx < n_chunks) {
                        const int r = idx / C4;
                        reinterpret_cast<float4 *>(seg)[r * P + (idx - r * C4)] = v[u];
                    }
                }
            }
        } else {
            // element by element: step st of the tile, metric m of Mp
            constexpr int SU = 8;
            const int n_el = nrows * S * Mp;
            float *dst = reinterpret_cast<float *>(seg);
            for (int i0 = tid; i0 < n_el; i0 += NT * SU) {
                float v[SU];
#pragma unroll
                for (int u = 0; u < SU; ++u) {
                    const int idx = i0 + u * NT, st = idx / Mp, m = idx % Mp;
                    const int64_t at = static_cast<int64_t>(st) * M + m;
                    v[u] = idx < n_el && m < M && at < avail ? x[at] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < SU; ++u) {
                    const int idx = i0 + u * NT;
                    if (idx < n_el) {
                        const int r = idx / (S * Mp);
                        dst[r * P * 4 + (idx - r * S * Mp)] = v[u];
                    }
                }
            }
        }
    }
    __syncthreads();

    // ---- every window's constants, one metric per thread and pass (consecutive threads:
    // consecutive windows)
    for (int idx = tid; idx < kNb * Mp; idx += NT) {
        const int n = idx % kNb, m = idx / kNb;
        float ca = 0.0f, cb = 0.0f;
        if (n < nv && m < M) {
            const float *row = reinterpret_cast<const float *>(seg) + n * P * 4 + m;
            int q = 0, ts = 0, last = -1;
            const float rm = p.norm == ENOVA_NORM_WINDOW ? 0.0f : p.mean[static_cast<int64_t>(s) * M + m];
            const float rs = p.norm == ENOVA_NORM_WINDOW ? 1.0f : p.std[static_cast<int64_t>(s) * M + m];
            auto at = [&](int t) {   // t = 0, then 0, 1, 2, ...
                if (t == 0) {
                    q = ts = 0;
                } else if (t != last && ++ts == S) {
                    ts = 0;
                    ++q;
                }
                last = t;
                return row[q * P * 4 + ts * Mp];
            };
            const unsigned big = window_constants(at, W, p.norm, rm, rs, ca, cb);
            atomicMax(&wmx[n], big);
        }
        cab[n * CP + m] = ca;
        cab[n * CP + Mp + m] = cb;
    }
    __syncthreads();

    const int wn0 = wave * kNbw * 32;
    const bool wave_active = wn0 < nv;
    if (wave_active) {
        int rb[kNbw], wi[kNbw];
#pragma unroll
        for (int nb = 0; nb < kNbw; ++nb) {
            const int n = wn0 + nb * 32 + (lane & 31);
            wi[nb] = n < nv ? n : nv - 1;         // idle columns evaluate a valid window
            rb[nb] = wi[nb] * P;
        }

        // ---- encoder
        v16f acc[HB][kNbw];
#pragma unroll
        for (int hb = 0; hb < HB; ++hb)
#pragma unroll
            for (int nb = 0; nb < kNbw; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    acc[hb][nb][r] = 0.0f;
        {
            // the lane's fragments hold metrics 8 (half mod MC) .. + 7
            float ca[kNbw][8], cb[kNbw][8];
            const int m0 = MC == 2 ? 8 * half : 0;
#pragma unroll
            for (int nb = 0; nb < kNbw; ++nb)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    ca[nb][e] = cab[wi[nb] * CP + m0 + e];
                    cb[nb][e] = cab[wi[nb] * CP + Mp + m0 + e];
                }
            const uint4 *ap = p.w1x + lane;
            constexpr int ASTEP = HB * 2 * 64;
            int cc = half % CPR;
            int koff = (half / CPR) * P + 2 * cc;
            auto advance = [&]() {
                if (CPR == 1) {
                    koff += 2 * P;
                } else {
                    const bool wrap = cc + 2 >= CPR;
                    cc = cc + 2 - (wrap ? CPR : 0);
                    koff += 4 + (wrap ? 1 : 0);
                }
            };
            // a step's lo parts are reloaded behind its first product, the hi parts behind its
            // last: 16 matrix ops of 32 cycles or more before they are read again
            uint4 ahi[HB], alo[HB];
#pragma unroll
            for (int hb = 0; hb < HB; ++hb) {
                alo[hb] = ap[(hb * 2 + 1) * 64];
                ahi[hb] = ap[(hb * 2) * 64];
            }
            float4 raw[kNbw][2];
#pragma unroll
            for (int nb = 0; nb < kNbw; ++nb)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    raw[nb][q] = reinterpret_cast<const float4 *>(seg)[rb[nb] + koff + q];
            advance();
            const uint4 *api = ap + ASTEP;
            for (int i = 0; i < g.nsteps; ++i) {
                v8h bhi[kNbw], blo[kNbw];
#pragma unroll
                for (int nb = 0; nb < kNbw; ++nb) {
                    fragment(raw[nb], ca[nb], cb[nb], bhi[nb], blo[nb]);
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        raw[nb][q] = reinterpret_cast<const float4 *>(seg)[rb[nb] + koff + q];
                }
                advance();
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int hb = 0; hb < HB; ++hb) {
#pragma unroll
                    for (int nb = 0; nb < kNbw; ++nb)
                        acc[hb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, alo[hb]), bhi[nb],
                                                                             acc[hb][nb], 0, 0, 0);
                    alo[hb] = api[(hb * 2 + 1) * 64];
                }
#pragma unroll
                for (int hb = 0; hb < HB; ++hb)
#pragma unroll
                    for (int nb = 0; nb < kNbw; ++nb)
                        acc[hb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, ahi[hb]), blo[nb],
                                                                             acc[hb][nb], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int hb = 0; hb < HB; ++hb) {
#pragma unroll
                    for (int nb = 0; nb < kNbw; ++nb)
                        acc[hb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, ahi[hb]), bhi[nb],
                                                                             acc[hb][nb], 0, 0, 0);
                    ahi[hb] = api[(hb * 2) * 64];
                }
                api += ASTEP;
            }
        }

        // ---- posterior heads and KL score (rows 0..15 mean, 16..31 log-variance)
        v16f z[kNbw];
#pragma unroll
        for (int i = 0; i < kNbw; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                z[i][r] = 0.0f;
#pragma unroll
        for (int hb = 0; hb < HB; ++hb)
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                uint4 w[3];
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    w[q] = p.whx[((hb * 2 + m) * 3 + q) * 64 + lane];
#pragma unroll
                for (int i = 0; i < kNbw; ++i) {
                    float hv[8];
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const int h = hb * 32 + crow(8 * m + t, half);
                        hv[t] = act_fn<ACT>(fmaf(acc[hb][i][8 * m + t], s_sc[h], s_b1[h]));
                    }
                    v8bf q[3];
                    split_bf16x8x3(hv, q);
                    z[i] = mfma6_bf16(w, q, z[i]);
                }
            }
        float kl[kNbw];
        v8bf mu[kNbw][3];
#pragma unroll
        for (int i = 0; i < kNbw; ++i) {
            kl[i] = 0.0f;
            float mv[8];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                z[i][r] += s_bh[crow(r, half)];
                if (r < 8) {
                    kl[i] += z[i][r] * z[i][r];
                    mv[r] = z[i][r];
                } else {
                    kl[i] += kl_g(z[i][r]);
                }
            }
            kl[i] += __shfl_xor(kl[i], 32);
            split_bf16x8x3(mv, mu[i]);
        }

        // ---- decoder: the hidden layer's two parts, then the output blocks, each reduced against v
        // (each output block's sums join the totals with the rounding of that addition carried along:
        // plain sums of up to D / 2 terms would be the largest error of the reconstruction error)
        float sm[kNbw][MC][4], sq[kNbw], cm[kNbw][MC][4], cq[kNbw];
#pragma unroll
        for (int i = 0; i < kNbw; ++i) {
            sq[i] = cq[i] = 0.0f;
#pragma unroll
            for (int j = 0; j < MC; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    sm[i][j][e] = cm[i][j][e] = 0.0f;
        }
        if (p.decode) {
            v8h hhi[kNbw][HB][2], hlo[kNbw][HB][2];
            float down[kNbw];                     // the accumulator's scale
#pragma unroll
            for (int i = 0; i < kNbw; ++i) {
                v16f hd[HB];
                float big = 0.0f;
#pragma unroll
                for (int hb = 0; hb < HB; ++hb) {
                    uint4 w[3];
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        w[q] = p.wdx[(hb * 3 + q) * 64 + lane];
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        hd[hb][r] = 0.0f;
                    hd[hb] = mfma6_bf16(w, mu[i], hd[hb]);
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        hd[hb][r] = act_fn<ACT>(hd[hb][r] + s_bd1[hb * 32 + crow(r, half)]);
                        big = fmaxf(big, fabsf(hd[hb][r]));
                    }
                }
                big = fmaxf(big, __shfl_xor(big, 32));
                // the power of two that puts the window's largest |hd| into [2^13, 2^14)
                int e = 140 - static_cast<int>(__float_as_uint(big) >> 23);
                e = big > 0.0f ? (e < -100 ? -100 : (e > 100 ? 100 : e)) : 0;
                const float up = __uint_as_float(static_cast<unsigned>(127 + e) << 23);
                down[i] = __uint_as_float(static_cast<unsigned>(127 - e) << 23) * g.wd2_unscale;
#pragma unroll
                for (int hb = 0; hb < HB; ++hb)
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        float v[8];
#pragma unroll
                        for (int t = 0; t < 8; ++t)
                            v[t] = hd[hb][8 * m + t] * up;
                        split_f16x8(v, hhi[i][hb][m], hlo[i][hb][m]);
                    }
            }
            const int nob = g.Dp / 32;
            constexpr int NF = HB * 2;            // (hidden block, half of it) fragments, two parts each
            // a fragment's slot is refilled right after its ops with the one RF further on (of the
            // next output block where that is past the end): 12 matrix ops of 32 cycles ahead at RF = 2
            constexpr int RF = 2;
            const uint4 *wa = p.wd2x + lane;
            uint4 ahi[RF], alo[RF];
#pragma unroll
            for (int f = 0; f < RF; ++f) {
                ahi[f] = wa[(f * 2) * 64];
                alo[f] = wa[(f * 2 + 1) * 64];
            }
            for (int ob = 0; ob < nob; ++ob) {
                const uint4 *wnext = ob + 1 == nob ? p.wd2x + lane : wa + NF * 2 * 64;
                v16f o[kNbw];
#pragma unroll
                for (int i = 0; i < kNbw; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        o[i][r] = 0.0f;
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    const v8h wh = __builtin_bit_cast(v8h, ahi[f % RF]), wl = __builtin_bit_cast(v8h, alo[f % RF]);
#pragma unroll
                    for (int i = 0; i < kNbw; ++i)
                        o[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wl, hhi[i][f / 2][f % 2], o[i], 0, 0, 0);
#pragma unroll
                    for (int i = 0; i < kNbw; ++i)
                        o[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wh, hlo[i][f / 2][f % 2], o[i], 0, 0, 0);
#pragma unroll
                    for (int i = 0; i < kNbw; ++i)
                        o[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wh, hhi[i][f / 2][f % 2], o[i], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    const uint4 *src = f + RF < NF ? wa + (f + RF) * 2 * 64 : wnext + (f + RF - NF) * 2 * 64;
                    ahi[f % RF] = src[0];
                    alo[f % RF] = src[64];
                }
                wa = wnext;
                // registers 4 gq .. 4 gq + 3: elements 32 ob + 8 gq + 4 half + e of the padded window,
                // i.e. step t = (4 ob + gq) / MC, metrics 8 (gq mod MC) + 4 half + e
                float bq[kNbw];
#pragma unroll
                for (int i = 0; i < kNbw; ++i)
                    bq[i] = 0.0f;
#pragma unroll
                for (int j = 0; j < MC; ++j) {
                    float bm[kNbw][4];
#pragma unroll
                    for (int i = 0; i < kNbw; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            bm[i][e] = 0.0f;
#pragma unroll
                    for (int gq = j; gq < 4; gq += MC) {
                        const int t = (4 * ob + gq) / MC;
                        const int off = (S == 1 ? t * P : (t / S) * P + (t % S) * (Mp / 4)) + 2 * j + half;
                        const bool in = t < W;    // the last block's padding
                        const float4 bd = reinterpret_cast<const float4 *>(s_bd2)[ob * 8 + 2 * gq + half];
                        const float bdv[4] = {bd.x, bd.y, bd.z, bd.w};
#pragma unroll
                        for (int i = 0; i < kNbw; ++i) {
                            const float4 x4 = reinterpret_cast<const float4 *>(seg)[in ? rb[i] + off : rb[i]];
                            const float4 *cw = reinterpret_cast<const float4 *>(cab + wi[i] * CP) + 2 * j + half;
                            const float4 a4 = cw[0], b4 = cw[Mp / 4];
                            const float v[4] = {(x4.x - b4.x) * a4.x, (x4.y - b4.y) * a4.y, (x4.z - b4.z) * a4.z,
                                                (x4.w - b4.w) * a4.w};
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float mo = fmaf(o[i][4 * gq + e], down[i], bdv[e]);
                                const float d = in ? fmaf(v[e], kSplitUnscale, -mo) : 0.0f;
                                bm[i][e] += d;
                                bq[i] = fmaf(d, d, bq[i]);
                            }
                        }
                    }
#pragma unroll
                    for (int i = 0; i < kNbw; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            carry_add(sm[i][j][e], cm[i][j][e], bm[i][e]);
                }
#pragma unroll
                for (int i = 0; i < kNbw; ++i)
                    carry_add(sq[i], cq[i], bq[i]);
            }
        }

        // ---- results: each lane half holds four metrics of every group, over all steps
#pragma unroll
        for (int i = 0; i < kNbw; ++i) {
            const int n = wn0 + i * 32 + (lane & 31);
            float tot = 0.0f;
#pragma unroll
            for (int j = 0; j < MC; ++j)
                tot += (sm[i][j][0] + sm[i][j][1]) + (sm[i][j][2] + sm[i][j][3]);
            tot += __shfl_xor(tot, 32);
            const float sqt = sq[i] + __shfl_xor(sq[i], 32);
            if (n >= nv)
                continue;
            if (split_outside(wmx[n])) {
                *s_mark = 1;
                continue;
            }
            const int64_t w = p.woff[s] + k0 + n;
            if (half == 0) {
                if (p.scores)
                    p.scores[w] = 0.5f * kl[i];
                if (p.md)
                    p.md[w] = tot * g.inv_d;
                if (p.rec)
                    p.rec[w] = sqt * g.inv_d;
            }
            if (p.mdm)
#pragma unroll
                for (int j = 0; j < MC; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int m = 8 * j + 4 * half + e;
                        if (m < M)
                            p.mdm[w * M + m] = sm[i][j][e] * g.inv_w;
                    }
        }
    }
    __syncthreads();
    if (tid == 0 && *s_mark)
        p.tile_stream[b] = split_mark(s);
}

// The marked tiles' windows outside the split's range, one block a window, in plain fp32 sums. A
// thread finds out for each window of the tile whether it is one (the statistics from global
// memory), then the block evaluates those. Rare by construction, so built for size, not speed.
__global__ __launch_bounds__(256) void k_ext_list(ExtSplitParams p, ExtSplitShape g)
{
    extern __shared__ float sm[];
    __shared__ int s_pick[kNb];
    __shared__ float red[256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int D = g.D, H = g.H, L = g.L, M = g.M, W = g.W;
    float *v = sm, *h = v + D, *ml = h + H, *hd = ml + 2 * L, *ca = hd + H, *cb = ca + M;   // cb: k
    const int64_t step = gridDim.x;
    for (int64_t first = blockIdx.x; first < g.list_grid; first += 256 * step) {
        uint64_t mask[4];   // the same in every wave
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = first + (q * 64 + lane) * step;
            mask[q] = __ballot(i < g.list_grid && split_marked(p.tile_stream[i]) >= 0);
        }
#pragma unroll 1
        for (int q = 0; q < 4; ++q)
            for (uint64_t mk = mask[q]; mk; mk &= mk - 1) {
                const int64_t b = first + (q * 64 + __builtin_ctzll(mk)) * step;
                const int s = split_marked(p.tile_stream[b]);
                const int64_t k0 = (b - p.tile_off[s]) * kNb;
                const int64_t ns = p.woff[s + 1] - p.woff[s];
                const int nv = static_cast<int>(ns - k0 < kNb ? ns - k0 : kNb);
                const float *mean = p.mean + static_cast<int64_t>(s) * M, *std = p.std + static_cast<int64_t>(s) * M;
                auto constants = [&](int n, int m, float &a, float &c) {
                    const float *x = p.x + (p.soff[s] + (k0 + n) * g.S) * M + m;
                    const bool own = p.norm == ENOVA_NORM_WINDOW;
                    return window_constants([&](int t) { return x[static_cast<int64_t>(t) * M]; }, W, p.norm,
                                            own ? 0.0f : mean[m], own ? 1.0f : std[m], a, c);
                };
                __syncthreads();   // the previous tile's picks are no longer read
                s_pick[tid] = 0;
                if (tid < nv) {
                    unsigned big = 0u;
                    for (int m = 0; m < M; ++m) {
                        float a, c;
                        big = max(big, constants(tid, m, a, c));
                    }
                    s_pick[tid] = split_outside(big) ? 1 : 0;
                }
                __syncthreads();
                for (int n = 0; n < nv; ++n) {
                    if (!s_pick[n])
                        continue;
                    const float *x = p.x + (p.soff[s] + (k0 + n) * g.S) * M;
                    const int64_t w = p.woff[s] + k0 + n;
                    for (int m = tid; m < M; m += 256) {
                        float a, c;
                        constants(n, m, a, c);
                        ca[m] = a * kSplitUnscale;
                        cb[m] = c;
                    }
                    __syncthreads();
                    for (int j = tid; j < D; j += 256)
                        v[j] = (x[j] - cb[j % M]) * ca[j % M];
                    __syncthreads();
                    auto dot = [&](const float *a, const float *c, int k) {
                        float t = 0.0f;
                        for (int j = lane; j < k; j += 64)
                            t = fmaf(a[j], c[j], t);
#pragma unroll
                        for (int off = 32; off >= 1; off >>= 1)
                            t += __shfl_xor(t, off);
                        return t;
                    };
                    auto act = [&](float a) { return g.act == ENOVA_TANH ? tanhf(a) : (a < 0.0f ? 0.0f : a); };
                    for (int i = wave; i < H; i += 4) {
                        const float t = dot(p.w1 + static_cast<int64_t>(i) * D, v, D);
                        if (lane == 0)
                            h[i] = act(t + p.b1[i]);
                    }
                    __syncthreads();
                    for (int i = wave; i < 2 * L; i += 4) {
                        const float t = dot(p.wml + static_cast<int64_t>(i) * H, h, H);
                        if (lane == 0)
                            ml[i] = t + p.bml[i];
                    }
                    __syncthreads();
                    for (int i = tid; i < H; i += 256) {
                        float t = 0.0f;
                        for (int l = 0; l < L; ++l)
                            t = fmaf(p.wd1[static_cast<int64_t>(i) * L + l], ml[l], t);
                        hd[i] = act(t + p.bd1[i]);
                    }
                    if (tid == 0 && p.scores) {
                        float kl = 0.0f;
                        for (int l = 0; l < L; ++l)
                            kl += ml[l] * ml[l] + kl_g(ml[L + l]);
                        p.scores[w] = 0.5f * kl;
                    }
                    __syncthreads();
                    if (p.decode) {
                        float sq = 0.0f;
                        for (int j = tid; j < D; j += 256) {
                            const float *row = p.wd2 + static_cast<int64_t>(j) * H;
                            float t = 0.0f;
                            for (int i = 0; i < H; ++i)
                                t = fmaf(row[i], hd[i], t);
                            v[j] = (v[j] - p.bd2d[j]) - t;
                            sq = fmaf(v[j], v[j], sq);
                        }
                        red[tid] = sq;
                        __syncthreads();
                        for (int m = tid; m < M; m += 256) {
                            float t = 0.0f;
                            for (int k = 0; k < W; ++k)
                                t += v[k * M + m];
                            ca[m] = t;
                            if (p.mdm)
                                p.mdm[w * M + m] = t * g.inv_w;
                        }
                        __syncthreads();
                        if (tid == 0) {
                            float t = 0.0f, e = 0.0f;
                            for (int m = 0; m < M; ++m)
                                t += ca[m];
                            for (int k = 0; k < 256; ++k)
                                e += red[k];
                            if (p.md)
                                p.md[w] = t * g.inv_d;
                            if (p.rec)
                                p.rec[w] = e * g.inv_d;
                        }
                    }
                    __syncthreads();
                }
            }
    }
}

using SplitKernel = void (*)(ExtSplitParams, ExtSplitShape);

template <int MC, int ACT>
SplitKernel pick_hb(int hb)
{
    switch (hb) {
    case 1: return k_ext_split<1, MC, ACT>;
    case 2: return k_ext_split<2, MC, ACT>;
    case 4: return k_ext_split<4, MC, ACT>;
    default: return nullptr;
    }
}

SplitKernel pick(const Geometry &g, const SplitGeometry &sg)
{
    const bool relu = g.act == ENOVA_RELU;
    if (sg.Mp == 8)
        return relu ? pick_hb<1, ENOVA_RELU>(g.HB) : pick_hb<1, ENOVA_TANH>(g.HB);
    return relu ? pick_hb<2, ENOVA_RELU>(g.HB) : pick_hb<2, ENOVA_TANH>(g.HB);
}

int padded_d(const Geometry &g, const SplitGeometry &sg) { return (g.W * sg.Mp + 31) / 32 * 32; }

// The output blocks' last rows read super-rows past the window's Q only under the t < W test; the
// encoder's prefetch is one step, as in k_score_split.
size_t lds_bytes(const Geometry &g, const SplitGeometry &sg)
{
    const size_t rows = static_cast<size_t>(kNb + sg.Q - 1 + sg.spare);
    return rows * sg.P * 16 +
           sizeof(float) * (static_cast<size_t>(kNb) * (2 * sg.Mp + 4) + kNb + padded_d(g, sg) + 3 * static_cast<size_t>(g.Hp) + 32 + 4);
}

size_t list_lds_bytes(const Geometry &g)
{
    return sizeof(float) * (static_cast<size_t>(g.D) + 2 * static_cast<size_t>(g.H) + 2 * g.L + 2 * static_cast<size_t>(g.M));
}

}  // namespace

bool ext_split_supported(const Geometry &g, const SplitGeometry &sg)
{
    return sg.ok && (sg.Mp == 8 || sg.Mp == 16) && g.HB <= 4 && lds_bytes(g, sg) <= kLdsLimit / 2 &&
           list_lds_bytes(g) <= 120 * 1024;
}

int ext_split_rows(const Geometry &g, const SplitGeometry &sg) { return padded_d(g, sg); }

// A tile's chain of steps takes about 0.18 us per padded element of a window however few tiles there
// are (73 to 93 us at Dp = 480, 205 us at 1024), and that is the pass until the tiles fill the chip; the
// chunked evaluation spreads few windows over its products' tiles, 50 us and 1.1e-5 us per window and
// element (7 metrics, W = 60, H = 64: 48 us for 1000 windows, 73 for 4000, 142 for 16000). They meet at
// n D = (0.18 Dp - 50) / 1.1e-5.
bool ext_split_pays(const Geometry &g, const SplitGeometry &sg, int64_t n_windows)
{
    return n_windows * g.D + 4500000 >= 16400LL * padded_d(g, sg);
}

hipError_t prepare_ext_split(const Geometry &g, const SplitGeometry &sg)
{
    SplitKernel k = pick(g, sg);
    if (!k)
        return hipErrorInvalidValue;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                             static_cast<int>(lds_bytes(g, sg)));
    if (e != hipSuccess)
        return e;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(k_ext_list), hipFuncAttributeMaxDynamicSharedMemorySize,
                               120 * 1024);
}

hipError_t launch_ext_split(const Geometry &g, const SplitGeometry &sg, const ExtSplitParams &p, float wd2_unscale,
                            int64_t grid, hipStream_t st)
{
    if (grid <= 0)
        return hipSuccess;
    SplitKernel k = pick(g, sg);
    if (!k)
        return hipErrorInvalidValue;
    ExtSplitShape sh{};
    sh.M = g.M;
    sh.S = g.S;
    sh.W = g.W;
    sh.D = g.D;
    sh.H = g.H;
    sh.L = g.L;
    sh.act = g.act;
    sh.Q = sg.Q;
    sh.CPR = sg.CPR;
    sh.P = sg.P;
    sh.nsteps = sg.nsteps;
    sh.spare = sg.spare;
    sh.Dp = padded_d(g, sg);
    sh.wd2_unscale = wd2_unscale;
    sh.inv_w = 1.0f / static_cast<float>(g.W);
    sh.inv_d = 1.0f / static_cast<float>(g.D);
    sh.list_grid = grid;
    hipLaunchKernelGGL(k, dim3(static_cast<unsigned>(grid)), dim3(256), lds_bytes(g, sg), st, p, sh);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_ext_list, dim3(static_cast<unsigned>(grid < 512 ? grid : 512)), dim3(256), list_lds_bytes(g),
                       st, p, sh);
    return hipGetLastError();
}

}  // namespace enova
