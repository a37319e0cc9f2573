// Configuration scans (Section IV-A, Eqs. (4)-(6)): per-window OLS fits with the slope's t-test,
// and per-stream KDE quantiles of the last window. All statistics in fp64, every reduction in a
// fixed order.
#include <hip/hip_runtime.h>

#include <cmath>

#include "config_internal.h"

namespace enova {

namespace {

constexpr int kCfgThreads = 256;
constexpr int kCfgMaxW = 4096;   // the per-stream kernel holds one window of four columns in LDS (80 KiB at most)
constexpr size_t kCfgScanLds = 48 * 1024;

template <int DT>
__device__ __forceinline__ float load_value(const void *x, int64_t idx)
{
    if constexpr (DT == ENOVA_BF16)
        return __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t *>(x)[idx]) << 16);
    else
        return static_cast<const float *>(x)[idx];
}

// The window's line, t-test and memory line from its means and centred sums.
__device__ __forceinline__ void cfg_window_out(const CfgParams &c, const CfgScanOut &o, int64_t out, double rm, double fm,
                                               double mm, double sxx, double sxy, double syy, double sxz)
{
    const int W = c.W;
    double a, b, t, g0, g1;
    if (sxx == 0.0) {
        a = fm;
        b = 0.0;
        t = 0.0;
        g0 = mm;
        g1 = 0.0;
    } else {
        b = sxy / sxx;
        a = fm - b * rm;
        const double rss = fmax(syy - b * sxy, 0.0);
        t = b == 0.0 ? 0.0 : (rss == 0.0 ? copysign(HUGE_VAL, b) : b * sqrt((W - 2) * sxx / rss));
        g1 = sxz / sxx;
        g0 = mm - g1 * rm;
    }
    if (o.a)
        o.a[out] = static_cast<float>(a);
    if (o.b)
        o.b[out] = static_cast<float>(b);
    if (o.t)
        o.t[out] = static_cast<float>(t);
    if (o.sig)
        o.sig[out] = fabs(t) > c.t_crit ? 1 : 0;
    if (o.g0)
        o.g0[out] = static_cast<float>(g0);
    if (o.g1)
        o.g1[out] = static_cast<float>(g1);
}

// Means and centred sums of a window by two passes over its samples.
struct CfgSums {
    double rm, fm, mm, sxx, sxy, syy, sxz;
};
__device__ __forceinline__ CfgSums cfg_two_pass(const float *r, const float *f, const float *m, int W)
{
    double sr = 0.0, sf = 0.0, smu = 0.0;
    for (int j = 0; j < W; ++j) {
        sr += r[j];
        sf += f[j];
        smu += m[j];
    }
    CfgSums q{sr / W, sf / W, smu / W, 0.0, 0.0, 0.0, 0.0};
    for (int j = 0; j < W; ++j) {
        const double dx = r[j] - q.rm, dy = f[j] - q.fm, dz = m[j] - q.mm;
        q.sxx = fma(dx, dx, q.sxx);
        q.sxy = fma(dx, dy, q.sxy);
        q.syy = fma(dy, dy, q.syy);
        q.sxz = fma(dx, dz, q.sxz);
    }
    return q;
}

// Windows that share few steps (or are too long for the prefix form below): one thread per window,
// two passes over its samples in LDS (means, then centred sums).
template <int DT>
__global__ __launch_bounds__(kCfgThreads) void k_cfg_scan(CfgParams c, int nb, const void *__restrict__ x,
                                                          const int64_t *__restrict__ soff,
                                                          const int64_t *__restrict__ woff,
                                                          const int64_t *__restrict__ tile_off,
                                                          const int *__restrict__ tile_stream, CfgScanOut o)
{
    extern __shared__ float sm[];
    const int s = tile_stream[blockIdx.x];
    if (s < 0)
        return;
    const int64_t k0 = (static_cast<int64_t>(blockIdx.x) - tile_off[s]) * nb;
    const int64_t nwin = woff[s + 1] - woff[s];
    const int nw = static_cast<int>(nwin - k0 < nb ? nwin - k0 : nb);
    const int W = c.W, S = c.S, M = c.M;
    const int seg = (nw - 1) * S + W;
    const int pitch = (nb - 1) * S + W;
    float *xr = sm, *xf = sm + pitch, *xm = sm + 2 * pitch;
    const int64_t row0 = soff[s] + k0 * S;
    for (int i = threadIdx.x; i < seg; i += kCfgThreads) {
        const int64_t base = (row0 + i) * M;
        xr[i] = load_value<DT>(x, base + c.col_r);
        xf[i] = load_value<DT>(x, base + c.col_f);
        xm[i] = load_value<DT>(x, base + c.col_m);
    }
    __syncthreads();
    const int w = threadIdx.x;
    if (w >= nw)
        return;
    const float *r = xr + w * S, *f = xf + w * S, *m = xm + w * S;
    const CfgSums q = cfg_two_pass(r, f, m, W);
    cfg_window_out(c, o, woff[s] + k0 + w, q.rm, q.fm, q.mm, q.sxx, q.sxy, q.syy, q.sxz);
}

// Overlapping windows. The two passes cost 16 issue slots of fp64 per sample of every window, 14 W
// flops, although neighbouring windows share all but S samples. Here a block of nb windows forms the
// prefix sums of its (nb - 1) S + W samples once -- of dx, dy, dz (the three columns less the
// block's first values, exact or rounded in fp64), dx^2, dx dy, dy^2, dx dz and dz^2 -- and each
// window's sums are differences of two of them: some 25 fp64 operations a sample and 60 a window.
// Precision. A difference carries the rounding of the block's whole sum, about 2^-52 P, and a
// centred sum Sxx = sum dx^2 - (sum dx)^2 / W is what is left of it. Where Sxx, Syy - b Sxy and Szz
// are each above 1e-4 of their block sum the outputs are within 1e-9 (they are stored as fp32); a
// window below that (a column constant over the window but not over the block, a perfect line)
// takes the two passes, so that exact zeros stay exact. A column constant over the whole block
// has all its sums exactly zero.
// Measured (1024 services x 16384 steps, W = 64, S = 1): 676 -> 288 us for the scan kernel, with blocks of 448
// windows (a shuffle scan of all eight quantities in every thread: 388 us, and with blocks of 512 421).
constexpr int kCfgSumsN = 8;
constexpr double kCfgKeep = 1e-4;

template <int DT>
__global__ __launch_bounds__(kCfgThreads) void k_cfg_scan_prefix(CfgParams c, int nb, const void *__restrict__ x,
                                                                 const int64_t *__restrict__ soff,
                                                                 const int64_t *__restrict__ woff,
                                                                 const int64_t *__restrict__ tile_off,
                                                                 const int *__restrict__ tile_stream, CfgScanOut o)
{
    extern __shared__ double cfg_pre[];   // prefix sums [8][pp], then the columns [3][pitch] floats
    __shared__ double wtot[kCfgThreads / 64][kCfgSumsN];
    const int s = tile_stream[blockIdx.x];
    if (s < 0)
        return;
    const int64_t k0 = (static_cast<int64_t>(blockIdx.x) - tile_off[s]) * nb;
    const int64_t nwin = woff[s + 1] - woff[s];
    const int nw = static_cast<int>(nwin - k0 < nb ? nwin - k0 : nb);
    const int W = c.W, S = c.S, M = c.M;
    const int seg = (nw - 1) * S + W;
    const int pitch = (nb - 1) * S + W;
    const int pp = (pitch + 1) | 1;       // odd: the eight quantities of a sample in different banks
    float *xr = reinterpret_cast<float *>(cfg_pre + kCfgSumsN * pp), *xf = xr + pitch, *xm = xf + pitch;
    const int64_t row0 = soff[s] + k0 * S;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < seg; i += kCfgThreads) {
        const int64_t base = (row0 + i) * M;
        xr[i] = load_value<DT>(x, base + c.col_r);
        xf[i] = load_value<DT>(x, base + c.col_f);
        xm[i] = load_value<DT>(x, base + c.col_m);
    }
    __syncthreads();
    // thread tid owns the samples tid * per .. + per - 1
    const int per = (seg + kCfgThreads - 1) / kCfgThreads;
    const int i0 = tid * per < seg ? tid * per : seg, i1 = i0 + per < seg ? i0 + per : seg;
    const double pr = xr[0], pf = xf[0], pm = xm[0];
    double v[kCfgSumsN];
#pragma unroll
    for (int k = 0; k < kCfgSumsN; ++k)
        v[k] = 0.0;
    auto add = [&](double (&t)[kCfgSumsN], int i) {
        const double dx = xr[i] - pr, dy = xf[i] - pf, dz = xm[i] - pm;
        t[0] += dx;
        t[1] += dy;
        t[2] += dz;
        t[3] = fma(dx, dx, t[3]);
        t[4] = fma(dx, dy, t[4]);
        t[5] = fma(dy, dy, t[5]);
        t[6] = fma(dx, dz, t[6]);
        t[7] = fma(dz, dz, t[7]);
    };
    for (int i = i0; i < i1; ++i)
        add(v, i);
    // exclusive prefix of the threads' sums (in the space of the samples' prefixes): thread (k, grp)
    // takes eight threads' sums of quantity k, so one scan a thread; eight shuffle scans in every
    // thread took a quarter of the kernel
    const int used = (seg + per - 1) / per;       // threads that own samples, at most min(256, seg)
    if (tid < used)
#pragma unroll
        for (int k = 0; k < kCfgSumsN; ++k)
            cfg_pre[k * pp + tid] = v[k];
    __syncthreads();
    {
        const int k = tid & 7, grp = tid >> 3;
        double own[8], sum = 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            own[u] = grp * 8 + u < used ? cfg_pre[k * pp + grp * 8 + u] : 0.0;
            sum += own[u];
        }
        double inc = sum;
#pragma unroll
        for (int off = 8; off < 64; off <<= 1) {
            const double u = __shfl_up(inc, off);
            inc += lane >= off ? u : 0.0;
        }
        if (lane >= 56)
            wtot[wave][k] = inc;
        __syncthreads();
        const double before = __shfl_up(inc, 8);
        double run = lane >= 8 ? before : 0.0;
        for (int w = 0; w < wave; ++w)
            run += wtot[w][k];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (grp * 8 + u < used)
                cfg_pre[k * pp + grp * 8 + u] = run;
            run += own[u];
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kCfgSumsN; ++k)
        v[k] = tid < used ? cfg_pre[k * pp + tid] : 0.0;
    __syncthreads();
    for (int i = i0; i < i1; ++i) {
#pragma unroll
        for (int k = 0; k < kCfgSumsN; ++k)
            cfg_pre[k * pp + i] = v[k];
        add(v, i);
    }
    if (i1 == seg && i0 < i1)   // the owner of the last sample
#pragma unroll
        for (int k = 0; k < kCfgSumsN; ++k)
            cfg_pre[k * pp + seg] = v[k];
    __syncthreads();
    const double inv_w = 1.0 / W;
    const double pxx = cfg_pre[3 * pp + seg], pyy = cfg_pre[5 * pp + seg], pzz = cfg_pre[7 * pp + seg];
    for (int w = tid; w < nw; w += kCfgThreads) {
        const int at = w * S;
        double d[kCfgSumsN];
#pragma unroll
        for (int k = 0; k < kCfgSumsN; ++k) {
            const double *p = cfg_pre + k * pp + at;
            d[k] = p[W] - p[0];
        }
        CfgSums q;
        const double mx = d[0] * inv_w, my = d[1] * inv_w, mz = d[2] * inv_w;
        q.rm = pr + mx;
        q.fm = pf + my;
        q.mm = pm + mz;
        q.sxx = fma(-d[0], mx, d[3]);
        q.sxy = fma(-d[0], my, d[4]);
        q.syy = fma(-d[1], my, d[5]);
        q.sxz = fma(-d[0], mz, d[6]);
        const double szz = fma(-d[2], mz, d[7]);
        const bool xc = pxx == 0.0, yc = pyy == 0.0, zc = pzz == 0.0;
        // false where a sum is not a number: those windows, too, take the two passes
        const bool good = (xc || q.sxx > kCfgKeep * pxx) && (zc || szz > kCfgKeep * pzz) &&
                          (yc || (xc && q.syy > kCfgKeep * pyy) ||
                           (q.syy - q.sxy * (q.sxy / q.sxx)) > kCfgKeep * pyy);
        if (good) {
            // exactly zero where a column is constant over the block
            if (xc)
                q.sxx = q.sxy = q.sxz = 0.0;
            if (yc)
                q.sxy = q.syy = 0.0;
            if (zc)
                q.sxz = 0.0;
        } else {
            q = cfg_two_pass(xr + at, xf + at, xm + at, W);
        }
        cfg_window_out(c, o, woff[s] + k0 + w, q.rm, q.fm, q.mm, q.sxx, q.sxy, q.syy, q.sxz);
    }
}

// Fixed-order block sum: a butterfly in each wave, then the four wave sums as (w0 + w1) +
// (w2 + w3); every thread gets the total. Two barriers (a tree over the threads took one per
// level).
static_assert(kCfgThreads == 256, "four waves");
__device__ __forceinline__ double wave_sum_cfg(double v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
        v += __shfl_xor(v, m);
    return v;
}

__device__ double block_sum(double v, double *red)
{
    v = wave_sum_cfg(v);
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = v;
    __syncthreads();
    const double r = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    return r;
}

// Two fixed-order block sums at once.
__device__ void block_sum2(double a, double b, double *red, double &ra, double &rb)
{
    a = wave_sum_cfg(a);
    b = wave_sum_cfg(b);
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = a;
        red[4 + (threadIdx.x >> 6)] = b;
    }
    __syncthreads();
    ra = (red[0] + red[1]) + (red[2] + red[3]);
    rb = (red[4] + red[5]) + (red[6] + red[7]);
    __syncthreads();
}

// Linearly interpolated sample quantile of sorted v[0..n).
__device__ double sorted_quantile(const float *v, int n, double p)
{
    const double h = (n - 1) * p;
    const int lo = static_cast<int>(floor(h));
    const int hi = lo + 1 < n ? lo + 1 : n - 1;
    return static_cast<double>(v[lo]) + (h - lo) * (static_cast<double>(v[hi]) - static_cast<double>(v[lo]));
}

// Quantile at level q of the Gaussian KDE of v[0..n) (Silverman's bandwidth): the root of its
// distribution function minus q. `sorted` is scratch of np2 floats (np2: a power of two >= n).
__device__ double kde_quantile(const float *v, int n, int np2, double q, float *sorted, double *red)
{
    for (int i = threadIdx.x; i < np2; i += kCfgThreads)
        sorted[i] = i < n ? v[i] : INFINITY;
    __syncthreads();
    // bitonic sort, ascending
    for (int k = 2; k <= np2; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < np2; i += kCfgThreads) {
                const int l = i ^ j;
                if (l > i) {
                    const bool up = (i & k) == 0;
                    const float x = sorted[i], y = sorted[l];
                    if ((x > y) == up) {
                        sorted[i] = y;
                        sorted[l] = x;
                    }
                }
            }
            __syncthreads();
        }
    }
    double part = 0.0;
    for (int i = threadIdx.x; i < n; i += kCfgThreads)
        part += v[i];
    const double mean = block_sum(part, red) / n;
    part = 0.0;
    for (int i = threadIdx.x; i < n; i += kCfgThreads) {
        const double d = v[i] - mean;
        part = fma(d, d, part);
    }
    const double ss = block_sum(part, red);
    const double sd = n > 1 ? sqrt(ss / (n - 1)) : 0.0;
    const double iqr = sorted_quantile(sorted, n, 0.75) - sorted_quantile(sorted, n, 0.25);
    const double spread = iqr > 0.0 ? fmin(sd, iqr / 1.34) : sd;
    const double h = 0.9 * spread * pow(static_cast<double>(n), -0.2);
    if (h == 0.0)
        return v[0];
    // Safeguarded Newton on F(x) - q (F' is the KDE density): every evaluation also tightens the
    // bracket [lo, hi], and a step that would leave it becomes a bisection step; stops when the
    // bracket can no longer shrink, the step vanishes, or a Newton step falls below 2^-26 of the
    // bracket's magnitude (taken: quadratic convergence then puts it within rounding of the root,
    // where the sums' rounding noise would otherwise keep the iterates moving).
    double lo = sorted[0] - 10.0 * h, hi = sorted[n - 1] + 10.0 * h;
    const double scale = 1.0 / (h * 1.4142135623730951);
    const double dens = 1.0 / (h * 2.5066282746310002 * n);   // 1 / (h sqrt(2 pi) n)
    double x = 0.5 * (lo + hi);
    for (int it = 0; it < 200; ++it) {
        double pf = 0.0, pd = 0.0;
        for (int i = threadIdx.x; i < n; i += kCfgThreads) {
            const double u = (x - v[i]) * scale;
            pf += 0.5 * erfc(-u);
            pd += exp(-u * u);
        }
        double F, f1;
        block_sum2(pf, pd, red, F, f1);
        F /= n;
        f1 *= dens;
        if (F < q)
            lo = x;
        else
            hi = x;
        double nx = f1 > 0.0 ? x - (F - q) / f1 : 0.5 * (lo + hi);
        const bool newton = nx > lo && nx < hi;
        if (!newton)
            nx = 0.5 * (lo + hi);
        if (nx == x || !(0.5 * (lo + hi) > lo && 0.5 * (lo + hi) < hi))
            break;
        if (newton && fabs(nx - x) <= 0x1p-26 * fmax(fabs(lo), fabs(hi))) {
            x = nx;
            break;
        }
        x = nx;
    }
    return x;
}

// One block per stream: the last window's fits, the regime and the KDE limits.
template <int DT>
__global__ __launch_bounds__(kCfgThreads) void k_cfg_stream(CfgParams c, const void *__restrict__ x,
                                                            const int64_t *__restrict__ soff, CfgStreamOut o)
{
    extern __shared__ float cfg_dyn[];   // four columns of the window [W] each, sort scratch [np2]
    __shared__ double red[2 * kCfgThreads];
    const int s = blockIdx.x;
    const int W = c.W, S = c.S, M = c.M;
    float *vr = cfg_dyn, *vf = vr + W, *vt = vf + W, *vm = vt + W, *sorted = vm + W;
    const int64_t T = soff[s + 1] - soff[s];
    const int64_t nw = T >= W ? (T - W) / S + 1 : 0;
    if (nw == 0) {
        if (threadIdx.x == 0) {
            if (o.sig)
                o.sig[s] = 0;
            if (o.n_limit)
                o.n_limit[s] = NAN;
            if (o.t_limit)
                o.t_limit[s] = NAN;
            if (o.max_num_seqs)
                o.max_num_seqs[s] = NAN;
            if (o.gpu_memory)
                o.gpu_memory[s] = NAN;
        }
        return;
    }
    const int64_t row0 = soff[s] + (nw - 1) * S;
    for (int i = threadIdx.x; i < W; i += kCfgThreads) {
        const int64_t base = (row0 + i) * M;
        vr[i] = load_value<DT>(x, base + c.col_r);
        vf[i] = load_value<DT>(x, base + c.col_f);
        vt[i] = load_value<DT>(x, base + c.col_t);
        vm[i] = load_value<DT>(x, base + c.col_m);
    }
    __syncthreads();
    double p0 = 0.0, p1 = 0.0, p2 = 0.0;
    for (int i = threadIdx.x; i < W; i += kCfgThreads) {
        p0 += vr[i];
        p1 += vf[i];
        p2 += vm[i];
    }
    const double rm = block_sum(p0, red) / W, fm = block_sum(p1, red) / W, mm = block_sum(p2, red) / W;
    double q0 = 0.0, q1 = 0.0, q2 = 0.0, q3 = 0.0;
    for (int i = threadIdx.x; i < W; i += kCfgThreads) {
        const double dx = vr[i] - rm, dy = vf[i] - fm, dz = vm[i] - mm;
        q0 = fma(dx, dx, q0);
        q1 = fma(dx, dy, q1);
        q2 = fma(dy, dy, q2);
        q3 = fma(dx, dz, q3);
    }
    const double sxx = block_sum(q0, red), sxy = block_sum(q1, red), syy = block_sum(q2, red),
                 sxz = block_sum(q3, red);
    double t = 0.0, g0 = mm, g1 = 0.0;
    if (sxx != 0.0) {
        const double b = sxy / sxx;
        const double rss = fmax(syy - b * sxy, 0.0);
        t = b == 0.0 ? 0.0 : (rss == 0.0 ? copysign(HUGE_VAL, b) : b * sqrt((W - 2) * sxx / rss));
        g1 = sxz / sxx;
        g0 = mm - g1 * rm;
    }
    const bool sig = fabs(t) > c.t_crit;
    const double q = sig ? c.q_extreme : 0.5;
    int np2 = 1;
    while (np2 < W)
        np2 <<= 1;
    const double nl = kde_quantile(vf, W, np2, q, sorted, red);
    const double tl = kde_quantile(vt, W, np2, q, sorted, red);
    if (threadIdx.x == 0) {
        const double mns = nl * tl;
        if (o.sig)
            o.sig[s] = sig ? 1 : 0;
        if (o.n_limit)
            o.n_limit[s] = nl;
        if (o.t_limit)
            o.t_limit[s] = tl;
        if (o.max_num_seqs)
            o.max_num_seqs[s] = mns;
        if (o.gpu_memory)
            o.gpu_memory[s] = g0 + g1 * mns;
    }
}

}  // namespace

// The prefix form where windows share at least three quarters of their steps and a block of 64
// windows or more fits its LDS (four blocks a compute unit). A block takes as many windows as leave
// every thread at most two samples and the 512 prefixes whole, 511 samples: rounds of 2^k windows, as it
// was for all but W + 447 S < 512, left threads without one (1024 services x 8192 steps, in us: W = 128,
// S = 1: 199 -> 171, W = 64, S = 2: 185 -> 138, S = 4: 175 -> 123, W = 270, S = 1: 347 -> 211). A few windows
// over one a thread would cost a second round of them: 257 of W = 256 take 220 us against 205, 281 of 232 211
// against 205, 297 of 216 200 against 203.
constexpr size_t kCfgPrefixLds = 39 * 1024;

static size_t prefix_lds_bytes(const CfgParams &c, int nb)
{
    const size_t pitch = static_cast<size_t>(nb - 1) * c.S + c.W;
    return sizeof(double) * kCfgSumsN * ((pitch + 1) | 1) + sizeof(float) * 3 * pitch;
}

static int prefix_windows_per_block(const CfgParams &c)
{
    if (4LL * c.S > c.W)
        return 0;
    constexpr int kSamples = 2 * kCfgThreads - 1, kFewOver = 36;
    int nb = c.W <= kSamples ? (kSamples - c.W) / c.S + 1 : 0;
    if (nb > kCfgThreads && nb < kCfgThreads + kFewOver)
        nb = kCfgThreads;
    return nb >= 64 ? nb : (prefix_lds_bytes(c, 64) <= kCfgPrefixLds ? 64 : 0);
}

int cfg_scan_windows_per_block(const CfgParams &c)
{
    if (const int nb = prefix_windows_per_block(c))
        return nb;
    for (int nb = kCfgThreads; nb >= 1; nb >>= 1)
        if (cfg_scan_lds_bytes(c, nb) <= kCfgScanLds)
            return nb;
    return 0;
}

size_t cfg_scan_lds_bytes(const CfgParams &c, int nb)
{
    return 3 * sizeof(float) * (static_cast<size_t>(nb - 1) * c.S + c.W);
}

hipError_t launch_cfg_scan(const CfgParams &c, int nb, const void *x, const int64_t *soff, const int64_t *woff,
                           const int64_t *tile_off, const int *tile_stream, int64_t grid, const CfgScanOut &o,
                           hipStream_t st)
{
    if (grid <= 0)
        return hipSuccess;
    using Kernel = void (*)(CfgParams, int, const void *, const int64_t *, const int64_t *, const int64_t *, const int *,
                            CfgScanOut);
    const bool prefix = prefix_windows_per_block(c) == nb && nb > 0;
    const bool bf = c.dtype == ENOVA_BF16;
    const Kernel k = prefix ? (bf ? static_cast<Kernel>(k_cfg_scan_prefix<ENOVA_BF16>) : k_cfg_scan_prefix<ENOVA_F32>)
                            : (bf ? static_cast<Kernel>(k_cfg_scan<ENOVA_BF16>) : k_cfg_scan<ENOVA_F32>);
    const size_t lds = prefix ? prefix_lds_bytes(c, nb) : cfg_scan_lds_bytes(c, nb);
    hipLaunchKernelGGL(k, dim3(static_cast<unsigned>(grid)), dim3(kCfgThreads), lds, st, c, nb, x, soff, woff, tile_off,
                       tile_stream, o);
    return hipGetLastError();
}

hipError_t launch_cfg_stream(const CfgParams &c, const void *x, const int64_t *soff, int n, const CfgStreamOut &o,
                             hipStream_t st)
{
    if (n <= 0)
        return hipSuccess;
    if (c.W > kCfgMaxW)
        return hipErrorInvalidValue;
    int np2 = 1;
    while (np2 < c.W)
        np2 <<= 1;
    const size_t lds = sizeof(float) * (4 * static_cast<size_t>(c.W) + np2);
    const void *fn = c.dtype == ENOVA_BF16 ? reinterpret_cast<const void *>(k_cfg_stream<ENOVA_BF16>)
                                           : reinterpret_cast<const void *>(k_cfg_stream<ENOVA_F32>);
    if (lds > 64 * 1024) {   // windows beyond 3276 steps need more than the default dynamic LDS
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        if (e != hipSuccess)
            return e;
    }
    if (c.dtype == ENOVA_BF16)
        hipLaunchKernelGGL(k_cfg_stream<ENOVA_BF16>, dim3(static_cast<unsigned>(n)), dim3(kCfgThreads), lds, st, c, x,
                           soff, o);
    else
        hipLaunchKernelGGL(k_cfg_stream<ENOVA_F32>, dim3(static_cast<unsigned>(n)), dim3(kCfgThreads), lds, st, c, x,
                           soff, o);
    return hipGetLastError();
}

}  // namespace enova
