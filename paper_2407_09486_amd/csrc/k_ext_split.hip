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
// 247 us (most of it the chunked pass's trips through memory). The errors against 64 bits are
// smaller: scores 4.2e-7 -> 3.0e-7, md 6.1e-6 -> 4.4e-6, reconstruction error 2.3e-7 -> 5.1e-8
// on the first.
//
// Windows out of the parts' range (split.h) are marked and evaluated in fp32, by k_ext_fused_list or, of shapes
// that it does not take, by k_ext_list; detectors whose output weights stand too far apart for one scale take
// the fp32 passes.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "split.h"
#include "variants_internal.h"

namespace enova {

namespace {

constexpr int kNb = kExtFusedNb;     // windows per tile
constexpr int kNbw = 2;              // 32-window blocks per wave

// Normalisation: v = (x - k) * ca, k the mean, scaled by kSplitScale. (With v = x * ca + cb the rounding of
// cb, at the scale of mean / std, doubles that of the mean.)
__device__ __forceinline__ float scaled_rstd(double std) { return static_cast<float>(1.0 / std) * kSplitScale; }

// The bits of a value's |v|, more than infinity's where x is not a number.
__device__ __forceinline__ unsigned size_of(float x, float ca, float k)
{
    return __float_as_uint((x - k) * ca) & 0x7fffffffu;
}

// One metric of one window against itself: its constants, and the bits of its largest |v| (infinity when
// out of range or not finite). x(t), t < W: the metric's values.
template <typename X>
__device__ __forceinline__ unsigned window_constants(X x, int W, float &ca, float &k)
{
    // shifted sums (shift: the window's first value): mean and population std
    const float x0 = x(0);
    float mn = x0, mx = x0;
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
    const bool finite = fabs(var) < INFINITY;   // NaN or infinite where a value was not
    var = var > 0.0 ? var : 0.0;
    double sd = sqrt(var);
    if (sd <= 1e-6 * fmax(1.0, fabs(mean)))
        sd = 1.0;   // constant metric inside the window
    ca = scaled_rstd(sd);
    k = static_cast<float>(mean);
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

    // ---- every window's constants and largest |v|
    if (p.norm == ENOVA_NORM_WINDOW) {
        // one metric per thread and pass (consecutive threads: consecutive windows)
        for (int idx = tid; idx < kNb * Mp; idx += NT) {
            const int n = idx % kNb, m = idx / kNb;
            float ca = 0.0f, cb = 0.0f;
            if (n < nv && m < M) {
                const float *row = reinterpret_cast<const float *>(seg) + n * P * 4 + m;
                int q = 0, ts = 0, last = -1;
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
                const unsigned big = window_constants(at, W, ca, cb);
                atomicMax(&wmx[n], big);
            }
            cab[n * CP + m] = ca;
            cab[n * CP + Mp + m] = cb;
        }
    } else {
        // the same constants for all: the largest |v| of each super-row, and of its steps that a window ends
        // with, then of the windows. (By window and metric this was a fifth of the pass on few windows.) The
        // rows' maxima take the table's place until it is filled: 5120 floats at the least, at most 2 x 1706 + 32.
        unsigned *rowm = reinterpret_cast<unsigned *>(cab), *tailm = rowm + rows_alloc;
        float *rc = reinterpret_cast<float *>(tailm + rows_alloc);
        const int rows = nv + Q - 1, tail = W - (Q - 1) * S;
        const float *mean = p.mean + static_cast<int64_t>(s) * M, *std = p.std + static_cast<int64_t>(s) * M;
        if (tid < M) {
            rc[tid] = scaled_rstd(std[tid]);
            rc[Mp + tid] = mean[tid];
        }
        __syncthreads();
        for (int r = tid; r < rows; r += NT) {
            const float *row = reinterpret_cast<const float *>(seg) + r * P * 4;
            unsigned full = 0u, part = 0u;
            for (int ts = 0; ts < S; ++ts) {
                unsigned big = 0u;
#pragma unroll 4
                for (int m = 0; m < M; ++m)
                    big = max(big, size_of(row[ts * Mp + m], rc[m], rc[Mp + m]));
                full = max(full, big);
                part = ts < tail ? max(part, big) : part;
            }
            rowm[r] = full;
            tailm[r] = part;
        }
        __syncthreads();
        unsigned big = 0u;
        if (tid < nv) {
            big = tailm[tid + Q - 1];
#pragma unroll 8
            for (int q = 0; q < Q - 1; ++q)
                big = max(big, rowm[tid + q]);
        }
        __syncthreads();
        wmx[tid] = big;
        float ca[Mp], cb[Mp];
#pragma unroll
        for (int m = 0; m < Mp; ++m) {
            ca[m] = m < M ? scaled_rstd(std[m]) : 0.0f;
            cb[m] = m < M ? mean[m] : 0.0f;
        }
#pragma unroll
        for (int m = 0; m < Mp; ++m) {
            cab[tid * CP + m] = ca[m];
            cab[tid * CP + Mp + m] = cb[m];
        }
    }
    __syncthreads();

    // windows outside the range (a wave holds 64) are left to the list; waves without any other are done
    static_assert(kNb == NT && kNbw == 2, "a thread per window, a mask's word per wave");
    const bool out = tid < nv && split_outside(wmx[tid]);
    const uint64_t outside = __ballot(out);
    if (__syncthreads_or(out)) {
        if (lane == 0)
            p.masks[b * 4 + wave] = outside;
        if (tid == 0)
            p.marks[1 + atomicAdd(p.marks, 1u)] = static_cast<unsigned>(b);
    }
    const int wn0 = wave * kNbw * 32;
    if (__any(tid < nv && !out)) {
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
            if (n >= nv || ((outside >> (n - wn0)) & 1u))
                continue;
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
}

// a[t] = w[k + t], zero from index K on.
template <int N>
__device__ __forceinline__ void load_row(const float *w, int k, int K, float (&a)[N])
{
    typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));   // of any alignment
    static_assert(N % 4 == 0, "16-byte loads");
    if (k + N <= K) {
#pragma unroll
        for (int q = 0; q < N / 4; ++q) {
            const f4 v = *reinterpret_cast<const f4 *>(w + k + 4 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                a[4 * q + e] = v[e];
        }
    } else {
#pragma unroll
        for (int t = 0; t < N; ++t)
            a[t] = k + t < K ? w[k + t] : 0.0f;
    }
}

// The windows that k_ext_split left, in fp32 (of shapes that k_ext_fused_list does not take): up to 64 of a marked tile (a mask's word) at a time, the
// parts dealt out evenly over the blocks. The windows are the columns of fp32 matrix ops whose other
// operand is a dense weight matrix read in place; in a run of 2 N reduction indices op t takes index t of
// the lower lanes' and index N + t of the upper lanes' half, so that a lane reads whole cache lines. The
// encoder's inputs are normalised into LDS once for the four waves, 64 indices of every window at a
// time, while the previous ones are multiplied; its waves are 32-row blocks by shares of each run (added
// in order). The output's blocks go to the waves in turn, and a lane adds its rows' v - m' per metric in
// a place of its own in LDS.
// This is for data that leaves the range for long (a metric constant over the reference prefix that
// moves later, gaps held as NaN). One window per block and serial dot products, as it was first, took 26.6 ms
// for 32 streams x 8192 steps x 7 metrics, W = 60, H = 64, tanh, half of the windows out; now 0.55 (0.18 in range;
// chunked evaluation 1.97).
constexpr int kExtListWin = 64, kExtListPitch = 65;   // windows, and floats of a row of them in LDS
constexpr int kExtListRun = 64;                       // reduction indices of a run
constexpr int kExtListPart = 2 * kExtListRun * kExtListPitch;   // two runs; partial sums later
static_assert(kExtListPart >= 8 * 16 * kExtListWin && kExtListPart >= 4 * 2 * 16 * 64, "partial sums");

template <int HB>
__global__ __launch_bounds__(256, 2) void k_ext_list(ExtSplitParams p, ExtSplitShape g)
{
    constexpr int C = kExtListWin, PITCH = kExtListPitch, RUN = kExtListRun, Hp = 32 * HB;
    constexpr int SL = 4 / HB, NT = RUN / 2 / SL;   // shares of a run, and the ops of one
    extern __shared__ float lsm[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5, col = lane & 31;
    const int D = g.D, H = g.H, L = g.L, M = g.M, W = g.W;
    // LDS: constants [M][C] (factor, mean), activations [Hp][PITCH], two runs of inputs or partial sums,
    // squares [8][C], the windows
    float2 *cak = reinterpret_cast<float2 *>(lsm);
    float *act = lsm + 2 * M * C, *part = act + Hp * PITCH, *sqs = part + kExtListPart;
    int *s_col = reinterpret_cast<int *>(sqs + 8 * C);
    float *ml = part + 4 * 16 * 64;   // [32][C], behind the heads' partial sums
    const int64_t count = p.marks[0];
    auto activation = [&](float a) { return g.act == ENOVA_TANH ? tanhf(a) : (a < 0.0f ? 0.0f : a); };
    // c[nb] += w[row] act over the groups [g0, g1) of 32 hidden units, of column blocks first, first + 1
    // (rows past the end give rows that are not used)
    auto product = [&](const float *w, int row, int rows, int g0, int g1, int first, int nbs, v16f (&c)[2]) {
        const float *wr = w + static_cast<int64_t>(row < rows ? row : rows - 1) * H;
        float a[2][16];
        if (g0 < g1)
            load_row<16>(wr, 32 * g0 + 16 * half, H, a[0]);
#pragma unroll
        for (int i = 0; i < HB; ++i) {
            if (i < g0 || i >= g1)
                continue;
            const int u = i & 1;
            if (i == g0 && u == 1)
#pragma unroll
                for (int t = 0; t < 16; ++t)
                    a[1][t] = a[0][t];
            if (i + 1 < g1)
                load_row<16>(wr, 32 * (i + 1) + 16 * half, H, a[u ^ 1]);
            const float *b = act + (32 * i + 16 * half) * PITCH + 32 * first + col;
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                c[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][t], b[t * PITCH], c[0], 0, 0, 0);
                if (nbs > 1)
                    c[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][t], b[t * PITCH + 32], c[1], 0, 0, 0);
            }
        }
    };
    for (int64_t it = blockIdx.x; it < 4 * count; it += gridDim.x) {
        const int quarter = static_cast<int>(it / count);
        const int64_t b = p.marks[1 + it - quarter * count];
        const uint64_t mask = p.masks[b * 4 + quarter];
        if (mask == 0)
            continue;
        const int s = p.tile_stream[b], cnt = __popcll(mask), nbs = cnt > 32 ? 2 : 1;
        const int64_t k0 = (b - p.tile_off[s]) * kNb + quarter * C;
        const float *xs = p.x + (p.soff[s] + k0 * g.S) * M;   // window n of the word starts at n S M
        const int64_t w0 = p.woff[s] + k0;
        if (tid < C && ((mask >> tid) & 1u))
            s_col[__popcll(mask & ((1ull << tid) - 1ull))] = tid;
        __syncthreads();
        // column c's window (past the last: that one again)
        auto window = [&](int c) { return xs + static_cast<int64_t>(s_col[min(c, cnt - 1)]) * g.S * M; };
        for (int i = tid; i < M * C; i += 256) {
            const int m = i / C;
            const float *x = window(i - m * C) + m;
            float mean, f;
            if (p.norm == ENOVA_NORM_WINDOW) {
                const double shift = x[0], inv_w = 1.0 / W;
                double s1 = 0.0, s2 = 0.0;
#pragma unroll 8
                for (int t = 0; t < W; ++t) {
                    const double d = static_cast<double>(x[static_cast<int64_t>(t) * M]) - shift;
                    s1 += d;
                    s2 = fma(d, d, s2);
                }
                const double mu = shift + s1 * inv_w, var = (s2 - s1 * s1 * inv_w) * inv_w;
                double sd = sqrt(var > 0.0 ? var : 0.0);
                if (sd <= 1e-6 * fmax(1.0, fabs(mu)))
                    sd = 1.0;   // constant metric inside the window
                f = static_cast<float>(1.0 / sd);
                mean = static_cast<float>(mu);
            } else {
                f = static_cast<float>(1.0 / static_cast<double>(p.std[static_cast<int64_t>(s) * M + m]));
                mean = p.mean[static_cast<int64_t>(s) * M + m];
            }
            cak[i] = make_float2(f, mean);
        }
        __syncthreads();

        // ---- encoder: wave = hidden block + HB share
        v16f c[2];
        auto clear = [&]() {
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    c[nb][r] = 0.0f;
        };
        clear();
        {
            const int row = 32 * (wave % HB) + col;
            const float *wr = p.w1 + static_cast<int64_t>(row < H ? row : H - 1) * D;
            const int at = 32 * half + NT * (wave / HB);   // of the run: this lane's first index
            // staging: thread = column and quarter of the run
            const int sc = tid >> 2, sk = 16 * (tid & 3);
            const float *xw = window(sc);
            float a[2][NT], v[16];
            auto put = [&](int run) {
                float *dst = part + (run & 1) * RUN * PITCH + sk * PITCH + sc;
                const int k = run * RUN + sk;
                int m = k % M;
#pragma unroll
                for (int t = 0; t < 16; ++t) {
                    const float2 q = cak[m * C + sc];
                    // past the end zero, not the metric's normalised zero: that may be infinite
                    dst[t * PITCH] = k + t < D ? (v[t] - q.y) * q.x : 0.0f;
                    m = m + 1 == M ? 0 : m + 1;
                }
            };
            load_row<16>(xw, sk, D, v);
            load_row<NT>(wr, at, D, a[0]);
            put(0);
            const int runs = (D + RUN - 1) / RUN;
            for (int r0 = 0; r0 < runs; r0 += 2) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int run = r0 + u;
                    if (run >= runs)
                        break;
                    const int next = run + 1 < runs ? run + 1 : run;
                    load_row<16>(xw, next * RUN + sk, D, v);
                    load_row<NT>(wr, next * RUN + at, D, a[u ^ 1]);
                    __syncthreads();   // the run is staged, and the one before no longer read
                    const float *bq = part + (run & 1) * RUN * PITCH + at * PITCH + col;
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        c[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][t], bq[t * PITCH], c[0], 0, 0, 0);
                        if (nbs > 1)
                            c[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[u][t], bq[t * PITCH + 32], c[1], 0, 0, 0);
                    }
                    if (next > run)
                        put(next);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                part[((wave * 2 + nb) * 16 + r) * 64 + lane] = c[nb][r];
        __syncthreads();
        for (int i = tid; i < HB * 2 * 16 * 64; i += 256) {
            const int ln = i & 63, r = (i >> 6) & 15, nb = (i >> 10) & 1, hb = i >> 11;
            float t = 0.0f;
#pragma unroll
            for (int sl = 0; sl < SL; ++sl)
                t += part[(((sl * HB + hb) * 2 + nb) * 16 + r) * 64 + ln];
            const int h = 32 * hb + crow(r, ln >> 5);
            act[h * PITCH + nb * 32 + (ln & 31)] = h < H ? activation(t + p.b1[h]) : 0.0f;
        }
        __syncthreads();

        // ---- heads [mu; logvar]: wave = column block + 2 share of the hidden units
        clear();
        const int nbw = wave & 1, sh = wave >> 1;
        if (nbw < nbs)
            product(p.wml, col, 2 * L, HB * sh / 2, HB * (sh + 1) / 2, nbw, 1, c);
#pragma unroll
        for (int r = 0; r < 16; ++r)
            part[(wave * 16 + r) * 64 + lane] = c[0][r];
        __syncthreads();
        for (int i = tid; i < 2 * 16 * 64; i += 256) {
            const int ln = i & 63, r = (i >> 6) & 15, nb = i >> 10, row = crow(r, ln >> 5);
            const float t = part[(nb * 16 + r) * 64 + ln] + part[((2 + nb) * 16 + r) * 64 + ln];
            ml[row * C + nb * 32 + (ln & 31)] = t + (row < 2 * L ? p.bml[row] : 0.0f);
        }
        __syncthreads();
        if (tid < cnt && p.scores) {
            float kl = 0.0f;
            for (int l = 0; l < L; ++l)
                kl += ml[l * C + tid] * ml[l * C + tid] + kl_g(ml[(L + l) * C + tid]);
            p.scores[w0 + s_col[tid]] = 0.5f * kl;
        }
        if (!p.decode) {
            __syncthreads();
            continue;
        }

        // ---- decoder: hidden layer, then the output blocks against v
        if (wave < HB) {
            const int row = 32 * wave + col;
            float a[8];
            load_row<8>(p.wd1 + static_cast<int64_t>(row < H ? row : H - 1) * L, 8 * half, L, a);
            clear();
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float *b = ml + (8 * half + t) * C + col;   // (the rows from L on are log-variances)
                const float b0 = 8 * half + t < L ? b[0] : 0.0f, b1 = 8 * half + t < L ? b[32] : 0.0f;
                c[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t], b0, c[0], 0, 0, 0);
                if (nbs > 1)
                    c[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t], b1, c[1], 0, 0, 0);
            }
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int h = 32 * wave + crow(r, half);
                    act[h * PITCH + nb * 32 + col] = h < H ? activation(c[nb][r] + p.bd1[h]) : 0.0f;
                }
        }
        __syncthreads();
        for (int i = tid; i < 8 * M * C; i += 256)
            part[i] = 0.0f;
        __syncthreads();
        // with M a divisor of 32 a lane's rows 8 q + e of every block belong to one metric, and its sums
        // stay in registers
        const bool fixed = 32 % M == 0;
        float sq[2] = {0.0f, 0.0f}, own[2][2][4];
#pragma unroll
        for (int i = 0; i < 16; ++i)
            own[i >> 3][(i >> 2) & 1][i & 3] = 0.0f;
        float *sums = part + (wave * 2 + half) * M * C;   // this lane's: [M][C], column nb * 32 + col
        const float *xc[2] = {window(col), window(32 + col)};
        for (int ob = wave; ob * 32 < D; ob += 4) {
            float xv[4][2][4], bd[4][4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j0 = 32 * ob + 8 * q + 4 * half;
                load_row<4>(p.bd2d, j0, D, bd[q]);
                load_row<4>(xc[0], j0, D, xv[q][0]);
                if (nbs > 1)
                    load_row<4>(xc[1], j0, D, xv[q][1]);
            }
            clear();
            product(p.wd2, 32 * ob + col, D, 0, HB, 0, nbs, c);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j0 = 32 * ob + 8 * q + 4 * half;
                int m = j0 % M;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb)
                        if (nb < nbs) {
                            const float2 k = cak[m * C + nb * 32 + col];
                            const float v = (xv[q][nb][e] - k.y) * k.x - bd[q][e];
                            const float d = j0 + e < D ? v - c[nb][4 * q + e] : 0.0f;
                            if (fixed)
                                own[nb][q & 1][e] += d;
                            else
                                sums[m * C + nb * 32 + col] += d;
                            sq[nb] = fmaf(d, d, sq[nb]);
                        }
                    m = m + 1 == M ? 0 : m + 1;
                }
            }
        }
        if (fixed)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int nb = i >> 3, q = (i >> 2) & 1, e = i & 3;
                sums[(8 * q + 4 * half + e) % M * C + nb * 32 + col] += own[nb][q][e];
            }
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
            sqs[(wave * 2 + half) * C + nb * 32 + col] = sq[nb];
        __syncthreads();
        for (int i = tid; i < M * C; i += 256) {
            const int m = i / C, cc = i - m * C;
            float t = 0.0f;
            for (int k = 0; k < 8; ++k)
                t += part[(k * M + m) * C + cc];
            act[i] = t;
            if (p.mdm && cc < cnt)
                p.mdm[(w0 + s_col[cc]) * M + m] = t * g.inv_w;
        }
        __syncthreads();
        if (tid < cnt) {
            float t = 0.0f, e = 0.0f;
            for (int m = 0; m < M; ++m)
                t += act[m * C + tid];
            for (int k = 0; k < 8; ++k)
                e += sqs[k * C + tid];
            if (p.md)
                p.md[w0 + s_col[tid]] = t * g.inv_d;
            if (p.rec)
                p.rec[w0 + s_col[tid]] = e * g.inv_d;
        }
        __syncthreads();   // the LDS is written again
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
           sizeof(float) * (static_cast<size_t>(kNb) * (2 * sg.Mp + 4) + kNb + padded_d(g, sg) + 3 * static_cast<size_t>(g.Hp) + 32);
}

// (at most 75.3 KiB: 16 metrics and 128 hidden units)
size_t list_lds_bytes(const Geometry &g)
{
    return sizeof(float) * (kExtListWin * (2 * static_cast<size_t>(g.M) + 8 + 1) + kExtListPitch * static_cast<size_t>(g.Hp) +
                            kExtListPart);
}

SplitKernel pick_list(int hb) { return hb == 1 ? k_ext_list<1> : hb == 2 ? k_ext_list<2> : k_ext_list<4>; }

}  // namespace

bool ext_split_supported(const Geometry &g, const SplitGeometry &sg)
{
    return sg.ok && (sg.Mp == 8 || sg.Mp == 16) && g.HB <= 4 && lds_bytes(g, sg) <= kLdsLimit / 2;
}

int ext_split_rows(const Geometry &g, const SplitGeometry &sg) { return padded_d(g, sg); }

// On few windows the pass takes as long as one tile's chain of steps: some 25 us, 0.06 us + 0.45 ns per
// (padded) hidden unit for every padded element of a window, tanh's epilogue, and against the window itself
// 0.038 us for every element's share in its statistics. The chunked evaluation spreads few windows over its
// products' tiles: 50 us and, a window, 2 to 4 ns and more with its elements and their products. Measured, in us,
// under reference and window normalisation, this pass (the same from 500 windows to 16000, within 5) and the
// chunked one at 500, 4000, 8000, 16000 windows:
//   7 metrics, W = 60, H = 64, tanh (Dp = 480)     76  91    61  74  89 123    52  72  92 138
//   7 metrics, W = 128, S = 5, H = 5, tanh (1024)  109 141   59  75  93 130    52  71  96 148
//   7 metrics, W = 120, H = 32      (Dp = 960)     90 122    58  71  89 128    51  67  93 145
//   5 metrics, W = 64, H = 128      (Dp = 512)     86  96    60  73  86 121    55  71  91 137
//   12 metrics, W = 64, H = 64      (Dp = 1024)   111 140    61  82 110 158    52  75 110 171
//   12 metrics, W = 128, H = 32     (Dp = 2048)   174 235    61  80 112 160    55  77 116 177
//   13 metrics, W = 32, H = 128, tanh (Dp = 512)  133 152    62  78  90 125    54  73  89 133
//   6 metrics, W = 16, S = 3, H = 100, tanh (128)  81  81    61  66  75 102    52  63  78 115
//   1 metric, W = 60, H = 64        (Dp = 480)     60  60    55  55  56  67    54  76 103 155
//   1 metric, W = 200, H = 128      (Dp = 1600)   202 210    62  68  78 102    64  90 121 188
//   3 metrics, W = 30, H = 24       (Dp = 240)     43  41    56  60  69  92    47  61  80 119
bool ext_split_pays(const Geometry &g, const SplitGeometry &sg, int64_t n_windows, int norm)
{
    const bool own = norm == ENOVA_NORM_WINDOW;
    const double D = g.D, H = g.H;
    double chain = 25.0 + padded_d(g, sg) * (0.06 + 0.00045 * g.Hp);
    if (g.act == ENOVA_TANH)
        chain += g.Hp > 64 ? 42.0 : 11.0;
    if (own)
        chain += 0.038 * D;
    const double each = own ? 4e-3 + 2.3e-6 * D + 1.5e-8 * D * H : 1.9e-3 + 2.4e-6 * D + 2.2e-8 * D * H;
    return (own ? 50.0 : 56.0) + each * static_cast<double>(n_windows) >= chain;
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
    if (ext_fused_list_supported(g))
        return prepare_ext_fused_list(g);
    return hipFuncSetAttribute(reinterpret_cast<const void *>(pick_list(g.HB)), hipFuncAttributeMaxDynamicSharedMemorySize,
                               static_cast<int>(kLdsLimit / 2));
}

static ExtSplitShape shape_of(const Geometry &g, const SplitGeometry &sg)
{
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
    sh.inv_w = 1.0f / static_cast<float>(g.W);
    sh.inv_d = 1.0f / static_cast<float>(g.D);
    return sh;
}

hipError_t launch_ext_split(const Geometry &g, const SplitGeometry &sg, const ExtSplitParams &p, float wd2_unscale,
                            int64_t grid, hipStream_t st)
{
    if (grid <= 0)
        return hipSuccess;
    SplitKernel k = pick(g, sg);
    if (!k)
        return hipErrorInvalidValue;
    ExtSplitShape sh = shape_of(g, sg);
    sh.wd2_unscale = wd2_unscale;
    hipLaunchKernelGGL(k, dim3(static_cast<unsigned>(grid)), dim3(256), lds_bytes(g, sg), st, p, sh);
    return hipGetLastError();
}

hipError_t launch_ext_list(const Geometry &g, const SplitGeometry &sg, const ExtSplitParams &p, int64_t grid,
                           hipStream_t st)
{
    if (grid <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(pick_list(g.HB), dim3(static_cast<unsigned>(std::min<int64_t>(4 * grid, 512))), dim3(256),
                       list_lds_bytes(g), st, p, shape_of(g, sg));
    return hipGetLastError();
}

}  // namespace enova
