// Scoring of fp32 detectors on the 16-bit matrix cores (gfx950).
//
// The encoder's first layer is 2*H*D flops per window, and the fp32 matrix ops that k_score_mfma
// uses run at 1/16 of the f16 rate. Here every normalised input and every first-layer weight is
// held as a sum of two f16 numbers (hi = round(x), lo = round(x - hi): 22 to 23 significant bits
// in the 32 bits that one fp32 number takes), and
//
//     C[h][n] = sum_k Whi Vhi + Whi Vlo + Wlo Vhi        (fp32 accumulation)
//
// runs as three v_mfma_f32_32x32x16_f16 per 16 reduction steps. The dropped Wlo Vlo and the
// remainders are below 2^-22 of a product; an fp32 chain of D products accumulates more rounding
// than that (D/2 roundings of the partial sum against 3 D / 16 here). Measured against 64 bits,
// the scores' relative error (2-norm) went from 4.3e-7 to 3.2e-7 at D = 512 and from 5.2e-7 to
// 3.6e-7 at D = 1024. One MI355X, whole scoring calls before and after: 64 services of 16384 steps x
// 8 metrics, W = 64, H = 64: 602 -> 240 us; 512 ragged streams x 16 metrics, W = 64, H = 128 (1.6e7
// windows): 31.3 -> 10.7 ms (410 fp32-equivalent TFLOP/s); 96 streams x 7 metrics, W = 60, H = 64,
// tanh: 1006 -> 349 us.
//
// Range. f16 ends at 65504 and its numbers are 2^-24 apart below 2^-14, so V is scaled by 2^4
// and each row of W1 by a power of two that puts its largest weight into [2^13, 2^14); both come
// off exactly with the bias (one fused multiply-add). Detectors whose inputs' weights stand so far
// apart that the parts' fixed 2^-29 of a small input would show take the fp32 kernel (decided at
// set-up). So do the windows whose largest |v| exceeds kSplitMax (or is not finite), or is not zero but
// below kSplitMin: they are left to k_score_mfma's list mode, which goes through the marked tiles. Waves
// without a window of their own kind skip the products on both sides. The choice depends on the
// window's own steps alone (a super-row's maximum is kept for all its steps and for those that a
// window ends with), so scores stay independent of what else a stream or a batch holds.
//
// The posterior heads and the decoder's hidden layer chain from the accumulators as in the other
// kernels, on 32x32x16 bf16 ops: activations, mu and weights as three bf16 parts each (24 bits,
// the full exponent range), six products.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.h"
#include "mfma_common.h"
#include "split.h"

namespace enova {

namespace {

struct SplitShape {
    int M, S, Mp, Q, CPR, P, nsteps, spare, tail_rows;
    float inv_d;
};

template <int HB, int NBW, int WH, int ACT>
__global__ __launch_bounds__(256, 2) void k_score_split(ScoreParams p, SplitShape g)
{
    constexpr int NW = 4, NT = 256;
    constexpr int WN = NW / WH;                   // window groups
    constexpr int HBT = HB * WH;                  // hidden blocks of the tile
    constexpr int NB = WN * NBW * 32;             // windows per tile
    constexpr int HP = 32 * HBT;
    extern __shared__ uint4 lds[];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6, half = lane >> 5;
    const int wh = wave % WH, wn = wave / WH;

    // ---- tile -> (stream, first window)
    const int64_t b = blockIdx.x;
    const int s = p.tile_stream[b];
    if (s < 0)
        return;
    const int64_t k0 = (b - p.tile_off[s]) * NB;
    const int64_t ns = p.woff[s + 1] - p.woff[s];
    const int nv = static_cast<int>(ns - k0 < NB ? ns - k0 : NB);
    const int64_t srow = p.soff[s];
    const int64_t T = p.soff[s + 1] - srow;

    const int Q = g.Q, CPR = g.CPR, P = g.P, M = g.M, Mp = g.Mp, S = g.S;
    const int nrows = nv + Q - 1 + g.spare;
    // LDS: the segment [rows][P] chunks (chunk c of a row: hi at 2c, lo at 2c + 1; P is odd so that
    // consecutive rows start in different banks), then per column of a super-row its mean, scaled
    // 1/std and offset, per row the sums and the largest |v| (both for the whole row and for the steps
    // that a window's last row has; one maximum where these are all), and b1, its row scale, bd1, u, biases
    uint4 *seg = lds;
    const int rows_alloc = NB + Q - 1 + g.spare;
    const size_t seg_chunks = static_cast<size_t>(rows_alloc) * P;
    constexpr size_t XCHG = WH > 1 ? epi_xchg_floats(NW, NBW) / 4 : 0;
    const int SMp = CPR * 8;
    float *cmean = reinterpret_cast<float *>(seg + (seg_chunks > XCHG ? seg_chunks : XCHG));
    float *crinv = cmean + SMp;
    int *coff = reinterpret_cast<int *>(crinv + SMp);
    float *rs = reinterpret_cast<float *>(coff + SMp);
    float *ps = rs + rows_alloc;
    unsigned *rm = reinterpret_cast<unsigned *>(ps + rows_alloc);
    const bool whole = g.tail_rows == S;
    unsigned *rt = whole ? rm : rm + rows_alloc;
    float *s_b1 = reinterpret_cast<float *>(rt + rows_alloc);
    float *s_sc = s_b1 + HP, *s_bd1 = s_sc + HP, *s_u = s_bd1 + HP, *s_bh = s_u + HP;
    int *s_mark = reinterpret_cast<int *>(s_bh + 32), *s_look = s_mark + 1;

    for (int i = tid; i < HP; i += NT) {
        s_b1[i] = p.b1[i];
        s_sc[i] = p.w1scale[i];
        s_bd1[i] = p.bd1[i];
        s_u[i] = p.u[i];
    }
    if (tid < 32)
        s_bh[tid] = p.bh[tid];
    if (tid == 0)
        *s_mark = *s_look = 0;
    for (int j = tid; j < SMp; j += NT) {
        const int tt = j / Mp;
        const int m = j - tt * Mp;
        if (m < M) {
            cmean[j] = p.mean[static_cast<int64_t>(s) * M + m];
            crinv[j] = split_rinv(p.std[static_cast<int64_t>(s) * M + m]);
            coff[j] = tt * M + m;
        } else {
            cmean[j] = 0.0f;
            crinv[j] = 0.0f;
            coff[j] = -1;
        }
    }
    for (int r = tid; r < nrows; r += NT)
        rm[r] = rt[r] = 0u;
    __syncthreads();

    // ---- stage: super-row r of the tile covers stream steps (k0 + r)*S .. +S-1
    const int64_t eavail = (T - k0 * S) * M;       // stream elements from super-row 0 on
    const int64_t ebase = (srow + k0 * S) * M;     // element index of super-row 0
    const bool linear = Mp == M && ebase % 4 == 0 && reinterpret_cast<uintptr_t>(p.x) % 16 == 0;
    const int tail_elems = g.tail_rows * Mp;
    const float *x = static_cast<const float *>(p.x);
    constexpr int SU = 4;                          // chunks (32 bytes) in flight per thread
    const int n_chunks = nrows * CPR;
    for (int base = tid; base < n_chunks; base += NT * SU) {
        float4 raw[SU][2];
        bool vec[SU];
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int idx = base + u * NT;
            vec[u] = idx < n_chunks && linear && static_cast<int64_t>(idx + 1) * 8 <= eavail;
            if (vec[u]) {
                const float4 *src = reinterpret_cast<const float4 *>(x + ebase + static_cast<int64_t>(idx) * 8);
                raw[u][0] = src[0];
                raw[u][1] = src[1];
            }
        }
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int idx = base + u * NT;
            if (idx >= n_chunks)
                break;
            const int r = idx / CPR, c = idx - r * CPR;
            float v[8];
            if (vec[u]) {
                v[0] = raw[u][0].x;
                v[1] = raw[u][0].y;
                v[2] = raw[u][0].z;
                v[3] = raw[u][0].w;
                v[4] = raw[u][1].x;
                v[5] = raw[u][1].y;
                v[6] = raw[u][1].z;
                v[7] = raw[u][1].w;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    v[e] = (v[e] - cmean[c * 8 + e]) * crinv[c * 8 + e];
            } else {
                // padding, the stream's end, or a row start that is not 16-byte aligned
                const int64_t rel = static_cast<int64_t>(r) * S * M;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int off = coff[c * 8 + e];
                    v[e] = 0.0f;
                    if (off >= 0 && rel + off < eavail)
                        v[e] = (x[ebase + rel + off] - cmean[c * 8 + e]) * crinv[c * 8 + e];
                }
            }
            unsigned big = 0u, bits[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                bits[e] = __float_as_uint(v[e]) & 0x7fffffffu;
                big = max(big, bits[e]);
                v[e] = bits[e] > __float_as_uint(kSplitMax) ? 0.0f : v[e];
            }
            v8h hi, lo;
            split_f16x8(v, hi, lo);
            seg[r * P + 2 * c] = __builtin_bit_cast(uint4, hi);
            seg[r * P + 2 * c + 1] = __builtin_bit_cast(uint4, lo);
            atomicMax(&rm[r], big);
            if (!whole && c * 8 < tail_elems) {
                unsigned tail = 0u;
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    tail = c * 8 + e < tail_elems ? max(tail, bits[e]) : tail;
                atomicMax(&rt[r], tail);
            }
        }
    }
    __syncthreads();

    // ---- per-super-row sums of the staged values (full row, and the window's tail part)
    for (int r = tid; r < nrows; r += NT) {
        float full = 0.0f, part = 0.0f;
        for (int c = 0; c < CPR; ++c) {
            const v8h hi = __builtin_bit_cast(v8h, seg[r * P + 2 * c]);
            const v8h lo = __builtin_bit_cast(v8h, seg[r * P + 2 * c + 1]);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float v = static_cast<float>(hi[e]) + static_cast<float>(lo[e]);
                full += v;
                if (c * 8 + e < tail_elems)
                    part += v;
            }
        }
        rs[r] = full;
        ps[r] = part;
        if (split_outside(rm[r]) || split_outside(rt[r]))
            *s_look = 1;   // else every window's largest |v| is in range, or zero
    }

    // ---- main contraction
    int rb[NBW];
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
        const int n = wn * NBW * 32 + nb * 32 + (lane & 31);
        rb[nb] = (n < nv ? n : nv - 1) * P;   // idle columns re-read a valid window
    }
    v16f acc[HB][NBW];
#pragma unroll
    for (int hb = 0; hb < HB; ++hb)
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[hb][nb][r] = 0.0f;
    bool wave_active = wn * NBW * 32 < nv;
    // A fragments of step i, block hb, part q: w1x[((i * HBT + hb) * 2 + q) * 64 + lane]
    const uint4 *ap = p.w1x + (wh * HB * 2) * 64 + lane;
    constexpr int ASTEP = HBT * 2 * 64;
    const int dpitch = P - 2 * CPR;
    int cc = half % CPR;
    int koff = (half / CPR) * P + 2 * cc;
    auto advance = [&]() {
        // two chunks on; with one chunk per row that is two rows
        if (CPR == 1) {
            koff += 2 * P;
        } else {
            const bool wrap = cc + 2 >= CPR;
            cc = cc + 2 - (wrap ? CPR : 0);
            koff += 4 + (wrap ? dpitch : 0);
        }
    };
    __syncthreads();
    // windows outside the range (by lane, of each window block), and whether the wave, or the block, has
    // any other
    uint64_t outside[NBW];
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb)
        outside[nb] = 0u;
    if (*s_look) {
        bool inside = false;
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb) {
            const int n = wn * NBW * 32 + nb * 32 + (lane & 31);
            unsigned wm = 0u;
            const int row0 = rb[nb] / P;
#pragma unroll 8
            for (int qq = half; qq < Q - 1; qq += 2)
                wm = max(wm, rm[row0 + qq]);
            wm = max(wm, rt[row0 + Q - 1]);
            wm = max(wm, static_cast<unsigned>(__shfl_xor(static_cast<int>(wm), 32)));
            const bool out = split_outside(wm);
            outside[nb] = __ballot(out);
            inside |= n < nv && !out;
            if (n < nv && out)
                atomicOr(s_mark, 1 << (n / kListNb));
        }
        wave_active = __any(inside);
        const bool any = __syncthreads_or(wave_active);
        if (tid == 0 && *s_mark)
            p.marks[1 + atomicAdd(p.marks, 1u)] = static_cast<unsigned>(b) << 4 | static_cast<unsigned>(*s_mark);
        if (!any)
            return;
    }
    if (wave_active) {
        // W1 fragments run two steps ahead in a register ring (a step is 3*HB*NBW matrix ops of 32
        // cycles), window fragments one step; a packed zero step and the spare rows make every
        // prefetch past the last step valid
        uint4 a[2][HB][2], bq[2][NBW][2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int hb = 0; hb < HB; ++hb)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    a[j][hb][q] = ap[j * ASTEP + (hb * 2 + q) * 64];
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
            for (int q = 0; q < 2; ++q)
                bq[0][nb][q] = seg[rb[nb] + koff + q];
        advance();
        const uint4 *api = ap + 2 * ASTEP;
        for (int i = 0; i < g.nsteps; i += 2) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
#pragma unroll
                for (int nb = 0; nb < NBW; ++nb)
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        bq[j ^ 1][nb][q] = seg[rb[nb] + koff + q];
                advance();
                __builtin_amdgcn_sched_barrier(0);
                // the three products of one accumulator are HB*NBW ops apart
#pragma unroll
                for (int t = 0; t < 3; ++t) {
#pragma unroll
                    for (int hb = 0; hb < HB; ++hb) {
                        const v8h av = __builtin_bit_cast(v8h, a[j][hb][t == 0 ? 1 : 0]);
#pragma unroll
                        for (int nb = 0; nb < NBW; ++nb)
                            acc[hb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                                av, __builtin_bit_cast(v8h, bq[j][nb][t == 1 ? 1 : 0]), acc[hb][nb], 0, 0, 0);
                    }
                    if (t == 0) {
                        // the lo parts are no longer read: reload them behind the first product
#pragma unroll
                        for (int hb = 0; hb < HB; ++hb)
                            a[j][hb][1] = api[j * ASTEP + (hb * 2 + 1) * 64];
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int hb = 0; hb < HB; ++hb)
                    a[j][hb][0] = api[j * ASTEP + (hb * 2) * 64];
            }
            api += 2 * ASTEP;
        }
    }

    // ---- epilogue
    const bool storer = wh == 0 && wave_active;
    if (WH > 1 || wave_active) {
        const SplitEpiArgs ea{p.whx, p.wdx, s_b1, s_sc, s_bd1, s_u, s_bh, reinterpret_cast<float *>(seg),
                              lane, half, wave, wh, wn};
        split_epilogue<HB, NBW, WH, NW, ACT>(acc, ea, [&](int nb, float sc, float dot) __attribute__((always_inline)) {
            // window mean of the staged inputs: super-rows rb .. rb+Q-1, the last one partially
            const int n = wn * NBW * 32 + nb * 32 + (lane & 31);
            float vsum = 0.0f;
            const int row0 = rb[nb] / P;
            for (int qq = half; qq < Q - 1; qq += 2)
                vsum += rs[row0 + qq];
            if (((Q - 1) & 1) == half)
                vsum += ps[row0 + Q - 1];
            vsum += __shfl_xor(vsum, 32);
            if (storer && half == 0 && n < nv && !((outside[nb] >> lane) & 1u)) {
                const int64_t w = p.woff[s] + k0 + n;
                p.scores[w] = sc;
                if (p.md)
                    p.md[w] = vsum * kSplitUnscale * g.inv_d - (dot + p.sum_bd2) * g.inv_d;
                if (p.write_flags)
                    p.flags[w] = sc > p.threshold ? 1 : 0;
            }
        });
    }
}

using SplitKernel = void (*)(ScoreParams, SplitShape);

template <int ACT>
SplitKernel pick_act(int hbt, bool small)
{
    switch (hbt) {
    case 1: return small ? k_score_split<1, 1, 1, ACT> : k_score_split<1, 4, 1, ACT>;
    case 2: return small ? k_score_split<2, 1, 1, ACT> : k_score_split<2, 4, 1, ACT>;
    case 4: return small ? k_score_split<4, 1, 1, ACT> : k_score_split<4, 2, 1, ACT>;
    case 8: return small ? k_score_split<4, 1, 2, ACT> : k_score_split<4, 2, 2, ACT>;
    default: return nullptr;
    }
}

SplitKernel pick(const Geometry &g, bool small)
{
    return g.act == ENOVA_RELU ? pick_act<ENOVA_RELU>(g.HB, small) : pick_act<ENOVA_TANH>(g.HB, small);
}

int split_nb(int hbt, bool small)
{
    switch (hbt) {
    case 1:
    case 2: return small ? 128 : 512;
    case 4: return small ? 128 : 256;
    default: return small ? 64 : 128;
    }
}

size_t split_lds(const Geometry &g, const SplitGeometry &sg, int nb)
{
    const int hbt = g.HB;
    const size_t rows = static_cast<size_t>(nb + sg.Q - 1 + sg.spare);
    const size_t per_row = g.W % g.S == 0 ? 3 : 4;   // floats: two sums, one or two maxima
    const size_t xchg = hbt == 8 ? epi_xchg_floats(4, nb / 64) * sizeof(float) : 0;
    const size_t hp = 32 * static_cast<size_t>(hbt);
    return std::max(rows * sg.P * 16, xchg) + 3 * sizeof(float) * 8 * sg.CPR + per_row * sizeof(float) * rows +
           sizeof(float) * (4 * hp + 32 + 4);
}

}  // namespace

SplitGeometry plan_split(const Geometry &g)
{
    SplitGeometry s;
    if (!g.mfma_ok || g.dtype != ENOVA_F32 || g.H > 256 || g.L > 16)
        return s;
    int mp = g.M;
    while ((static_cast<int64_t>(g.S) * mp) % 8)
        ++mp;
    const int64_t cpr = static_cast<int64_t>(g.S) * mp / 8;
    const int64_t kc = (static_cast<int64_t>(g.Q) * cpr + 3) / 4 * 4;
    if (cpr >= (1 << 16) || kc >= (1 << 22))
        return s;
    s.Mp = mp;
    s.Q = g.Q;
    s.CPR = static_cast<int>(cpr);
    s.P = 2 * s.CPR + 1;
    s.nsteps = static_cast<int>(kc / 2);
    // the furthest chunk that a prefetch of window fragments reads: one step past the last
    s.spare = static_cast<int>((kc + 1) / cpr - s.Q + 2);
    s.nb_small = split_nb(g.HB, true);
    s.nb_large = split_nb(g.HB, false);
    s.lds_small = split_lds(g, s, s.nb_small);
    s.lds_large = split_lds(g, s, s.nb_large);
    // the large tile where two blocks fit a compute unit's LDS, else the small one alone
    if (s.lds_large > kLdsLimit / 2) {
        s.nb_large = s.nb_small;
        s.lds_large = s.lds_small;
    }
    s.ok = s.lds_small <= kLdsLimit / 2;
    return s;
}

hipError_t prepare_score_split(const Geometry &g, const SplitGeometry &sg)
{
    for (const bool small : {true, false}) {
        SplitKernel k = pick(g, small);
        if (!k)
            return hipErrorInvalidValue;
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 static_cast<int>(small ? sg.lds_small : sg.lds_large));
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

hipError_t launch_score_split(const Geometry &g, const SplitGeometry &sg, const ScoreParams &p, int nb, int64_t grid,
                              hipStream_t st)
{
    if (grid <= 0)
        return hipSuccess;
    const bool small = nb == sg.nb_small;
    SplitKernel k = pick(g, small);
    if (!k || (!small && nb != sg.nb_large))
        return hipErrorInvalidValue;
    SplitShape sh;
    sh.M = g.M;
    sh.S = g.S;
    sh.Mp = sg.Mp;
    sh.Q = sg.Q;
    sh.CPR = sg.CPR;
    sh.P = sg.P;
    sh.nsteps = sg.nsteps;
    sh.spare = sg.spare;
    sh.tail_rows = g.W - (g.Q - 1) * g.S;
    sh.inv_d = 1.0f / static_cast<float>(g.D);
    hipLaunchKernelGGL(k, dim3(static_cast<unsigned>(grid)), dim3(256), small ? sg.lds_small : sg.lds_large, st, p,
                       sh);
    return hipGetLastError();
}

}  // namespace enova
