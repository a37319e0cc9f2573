// Peaks-over-threshold calibration (Section IV-B cites Siffer et al. 2017), entirely on the device:
// one wait for the caller, at the end.
//
// The level quantile t is the exact order statistic of the calibration scores (a radix select over
// their float keys); the excesses Y over t follow a generalised Pareto distribution GPD(gamma,
// sigma), fitted by Grimshaw's reduction of the likelihood: with x = gamma/sigma the score
// equations collapse to u(x) v(x) = 1, u = mean 1/(1+xY), v = 1 + mean log(1+xY), evaluated without
// cancellation as
//     w(x) = b - a - a b = 0,   a = mean xY/(1+xY) = 1 - u,   b = mean log1p(xY) = v - 1.
// Roots are bracketed on geometric grids of both admissible intervals: (0, B], B =
// 2 (mean - min) / min^2, which spans many decades once there are many peaks, and (-1/Y_max, 0),
// resolved geometrically towards both ends; each bracket is refined by Newton's method kept inside
// it (w' from two more sums): the first point is the secant of the grid's w at the bracket's ends, a
// step that lands strictly inside is taken, else false position through the ends (Illinois), else
// the midpoint, and a bracket ends once |w| is within the rounding of the sums it is formed from,
// once the step falls below 2^-26 of the point (quadratic convergence then puts the new point
// within rounding of the root; a tighter test only meets the rounding noise of the sums), or when
// it can no longer be split. The exponential tail (gamma = 0, sigma = mean Y) is always a
// candidate, and the candidate of largest log-likelihood wins (ties: smaller |gamma|). Below ten
// peaks the method of moments takes the place of the likelihood.
//
// The call is latency-bound until there are millions of scores: with the decisions between its
// kernels taken on the host it was some 30 launches and six round trips (376 us for 64 services of
// 16321 windows, 340 us of a single service's detection). Here every decision is left in device
// memory (PotState) for the next launch: 185 us, and 141 us for that detection. The fit's evaluations run as pairs of a
// k_pot_eval over the whole chip and a k_pot_step of one block, which moves from the grid to Newton
// steps, to the candidates, to the end; launches past the end leave at once, and a fit that needs
// more of them than were queued gets them from the host.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "block_scan.h"
#include "gpd_math.h"
#include "pot_internal.h"

namespace enova {

namespace {

// Order-preserving map of a float to an unsigned key, and back.
__device__ __forceinline__ uint32_t fkey(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_float(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// The calibration set's offsets (cal[s] = calibration scores before stream s: the windows wholly
// inside each stream's reference prefix), the radix select's start and the cleared bins. One block.
__global__ __launch_bounds__(1024) void k_pot_begin(const int64_t *__restrict__ soff, const int64_t *__restrict__ woff,
                                                    int n, int W, int S, float ref_frac, double level,
                                                    int64_t *__restrict__ cal, PotState *__restrict__ st)
{
    __shared__ int64_t wsum[16];
    const int tid = threadIdx.x;
    const int64_t chunk = (static_cast<int64_t>(n) + 1023) / 1024;
    const int64_t a = tid * chunk, b = a + chunk < n ? a + chunk : n;
    auto count = [&](int64_t s) -> int64_t {
        const int64_t c = woff[s + 1] - woff[s];
        const int64_t R = ref_len_dev(ref_frac, soff[s + 1] - soff[s]);
        const int64_t k = R >= W ? (R - W) / S + 1 : 0;
        return k < c ? k : c;
    };
    for (int i = tid; i < kPotPasses * 256; i += 1024)
        (&st->hist[0][0])[i] = 0u;
    int64_t local = 0;
    for (int64_t s = a; s < b; ++s)
        local += count(s);
    int64_t total;
    int64_t run = block_scan_excl<1024>(local, wsum, total);
    for (int64_t s = a; s < b; ++s) {
        cal[s] = run;
        run += count(s);
    }
    if (tid == 0) {
        cal[n] = total;
        int64_t rank = static_cast<int64_t>(ceil(level * static_cast<double>(total))) - 1;
        rank = rank < 0 ? 0 : (rank > total - 1 ? total - 1 : rank);
        st->n_cal = total;
        st->sel[0] = PotSelect{0u, 0, rank, 0};
        st->err = total <= 0 ? kPotNoWindows : 0;
        st->phase = kPotGrid;
        st->n_peaks = 0;
    }
}

// The radix select after `pass` passes: sel[pass - 1] and the bins of that pass give the digit that
// holds the rank (256 threads, thread d on bin d). Every block forms it for itself; block 0 leaves
// it in sel[pass] for the next launch.
__device__ __forceinline__ PotSelect pot_pick(PotState *st, int pass, int64_t *wsum, PotSelect *out)
{
    if (pass == 0)
        return st->sel[0];
    const PotSelect prev = st->sel[pass - 1];
    const int d = threadIdx.x;
    const int64_t c = st->hist[pass - 1][d];
    int64_t total;
    const int64_t before = block_scan_excl<256>(c, wsum, total);
    if (d == 0)
        *out = PotSelect{0u, 1, 0, 0};   // the rank was lost unless a thread below finds it
    __syncthreads();
    if (c > 0 && prev.rank >= before && prev.rank < before + c)
        *out = PotSelect{(prev.prefix << 8) | static_cast<uint32_t>(d), prev.lost, prev.rank - before,
                         prev.n_greater + total - before - c};
    __syncthreads();
    const PotSelect r = *out;
    if (blockIdx.x == 0 && d == 0)
        st->sel[pass] = r;
    return r;
}

// The calibration scores ITEMS * 256 * blockIdx.x + 256 j + tid, j < ITEMS: their places in `scores`
// (calibration scores of a stream are its first windows) through the offsets, kept in LDS when
// there are at most kPotLds of them.
constexpr int kPotLds = 2048;

struct PotWalk {
    const int64_t *off;
    int64_t n_cal, start;
    int s;
    __device__ __forceinline__ PotWalk(const int64_t *cal, int n, int64_t n_cal_, int64_t start_, int64_t *lds)
        : off(cal), n_cal(n_cal_), start(start_), s(0)
    {
        if (n < kPotLds) {
            for (int i = threadIdx.x; i <= n; i += 256)
                lds[i] = cal[i];
            __syncthreads();
            off = lds;
        }
        int lo = 0, hi = n - 1;
        while (lo < hi) {   // the stream of the block's first score
            const int mid = (lo + hi + 1) >> 1;
            if (off[mid] <= start)
                lo = mid;
            else
                hi = mid - 1;
        }
        s = lo;
    }
    __device__ __forceinline__ bool at(int j, const int64_t *woff, int64_t &i)
    {
        const int64_t ci = start + j * 256 + static_cast<int>(threadIdx.x);
        if (ci >= n_cal)
            return false;
        while (off[s + 1] <= ci)
            ++s;
        i = woff[s] + (ci - off[s]);
        return true;
    }
};

// Pass `pass` of the select: the histogram of the next 8-bit digit among the keys with the prefix, over
// `rounds` runs of 256 ITEMS scores a block. A block's start (the select's state, the bins before, the
// offsets, the search) is a chain of loads that large calls pay once for several runs: 1.3e8 scores of
// 4096 streams, of which half are calibration scores, 4.55 -> 3.95 ms for the threshold call.
template <int ITEMS>
__global__ __launch_bounds__(256) void k_pot_hist(const float *__restrict__ scores, const int64_t *__restrict__ woff,
                                                  const int64_t *__restrict__ cal, int n, int pass, int rounds,
                                                  PotState *st)
{
    __shared__ int64_t lds[kPotLds];
    __shared__ unsigned h[256];
    __shared__ int64_t wsum[4];
    __shared__ PotSelect pick;
    const int64_t n_cal = st->n_cal, start = static_cast<int64_t>(blockIdx.x) * 256 * ITEMS * rounds;
    if (start >= n_cal && blockIdx.x > 0)
        return;
    const PotSelect sel = pot_pick(st, pass, wsum, &pick);
    h[threadIdx.x] = 0u;
    __syncthreads();
    if (n_cal > 0) {
        PotWalk w(cal, n, n_cal, start, lds);
        const int shift = 24 - 8 * pass;
        for (int r = 0; r < rounds; ++r, w.start += 256 * ITEMS) {
            float v[ITEMS];
            bool on[ITEMS];
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                int64_t i;
                on[j] = w.at(j, woff, i);
                v[j] = on[j] ? scores[i] : 0.0f;
            }
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const uint32_t key = fkey(v[j]);
                if (on[j] && (pass == 0 || (key >> (shift + 8)) == sel.prefix))
                    atomicAdd(&h[(key >> shift) & 255u], 1u);
            }
        }
    }
    __syncthreads();
    if (h[threadIdx.x])
        atomicAdd(&st->hist[pass][threadIdx.x], h[threadIdx.x]);
}

// Peaks, pass 1: how many keys above the level quantile's each block holds.
template <int ITEMS>
__global__ __launch_bounds__(256) void k_pot_count(const float *__restrict__ scores, const int64_t *__restrict__ woff,
                                                   const int64_t *__restrict__ cal, int n, PotState *st,
                                                   int64_t *__restrict__ counts)
{
    __shared__ int64_t lds[kPotLds];
    __shared__ int64_t wsum[4];
    __shared__ PotSelect pick;
    const int tid = threadIdx.x;
    const int64_t n_cal = st->n_cal, start = static_cast<int64_t>(blockIdx.x) * 256 * ITEMS;
    if (start >= n_cal && blockIdx.x > 0) {
        if (tid == 0)
            counts[blockIdx.x] = 0;
        return;
    }
    const PotSelect sel = pot_pick(st, kPotPasses, wsum, &pick);
    int cnt = 0;
    if (n_cal > 0) {
        PotWalk w(cal, n, n_cal, start, lds);
        float v[ITEMS];
        bool on[ITEMS];
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            int64_t i;
            on[j] = w.at(j, woff, i);
            v[j] = on[j] ? scores[i] : 0.0f;
        }
#pragma unroll
        for (int j = 0; j < ITEMS; ++j)
            cnt += on[j] && fkey(v[j]) > sel.prefix ? 1 : 0;
    }
    int64_t total;
    block_scan_excl<256>(cnt, wsum, total);
    if (tid == 0)
        counts[blockIdx.x] = total;
}

// Exclusive scan of the block counts by one block, and the checks that end the select.
__global__ __launch_bounds__(1024) void k_pot_offsets(const int64_t *__restrict__ counts, int64_t nblk,
                                                      int64_t *__restrict__ off, PotState *__restrict__ st,
                                                      int64_t cap)
{
    __shared__ int64_t wsum[16];
    const int tid = threadIdx.x;
    const int64_t chunk = (nblk + 1023) / 1024;
    const int64_t a = tid * chunk, b = a + chunk < nblk ? a + chunk : nblk;
    int64_t local = 0;
    for (int64_t i = a; i < b; ++i)
        local += counts[i];
    int64_t total;
    int64_t r = block_scan_excl<1024>(local, wsum, total);
    for (int64_t i = a; i < b; ++i) {
        off[i] = r;
        r += counts[i];
    }
    if (tid == 0) {
        const PotSelect sel = st->sel[kPotPasses];
        const float t = key_float(sel.prefix);
        st->t = static_cast<double>(t);
        st->n_peaks = total;
        if (st->err == 0) {
            if (sel.lost)
                st->err = kPotLost;
            else if (!isfinite(t))
                st->err = kPotLevelNotFinite;
            else if (total != sel.n_greater || total > cap)
                st->err = kPotCount;
        }
    }
}

// Pass 2: the excesses y = score - t of the peaks, in calibration order (stable).
template <int ITEMS>
__global__ __launch_bounds__(256) void k_pot_compact(const float *__restrict__ scores,
                                                     const int64_t *__restrict__ woff, const int64_t *__restrict__ cal,
                                                     int n, const PotState *__restrict__ st,
                                                     const int64_t *__restrict__ off, double *__restrict__ y,
                                                     int64_t cap)
{
    __shared__ int64_t lds[kPotLds];
    __shared__ int wcnt[4][ITEMS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t n_cal = st->n_cal, start = static_cast<int64_t>(blockIdx.x) * 256 * ITEMS;
    if (start >= n_cal || st->err)
        return;
    const uint32_t key_t = st->sel[kPotPasses].prefix;
    const double t = st->t;
    PotWalk w(cal, n, n_cal, start, lds);
    float v[ITEMS];
    uint64_t mask[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        int64_t i;
        const bool on = w.at(j, woff, i);
        v[j] = on ? scores[i] : 0.0f;
        mask[j] = on ? 1u : 0u;
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        mask[j] = __ballot(mask[j] && fkey(v[j]) > key_t);
        if (lane == 0)
            wcnt[wave][j] = __popcll(mask[j]);
    }
    __syncthreads();
    int64_t pos = off[blockIdx.x];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        int64_t at = pos;
        for (int q = 0; q < 4; ++q) {
            at += q < wave ? wcnt[q][j] : 0;
            pos += wcnt[q][j];
        }
        if ((mask[j] >> lane) & 1u) {
            at += __popcll(mask[j] & ((1ull << lane) - 1ull));
            if (at < cap)
                y[at] = static_cast<double>(v[j]) - t;
        }
    }
}

// Wave-wide sum in a fixed butterfly order (every lane ends with the same value).
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
        v += __shfl_xor(v, m);
    return v;
}

// Sum, minimum and maximum of chunk blockIdx.x of kPotStatBlocks of the excesses, in a fixed order.
__global__ __launch_bounds__(256) void k_pot_stats(const double *__restrict__ y, PotState *__restrict__ st)
{
    __shared__ double red[3][4];
    if (st->err)
        return;
    const int64_t n = st->n_peaks;
    const int64_t chunk = (n + kPotStatBlocks - 1) / kPotStatBlocks;
    const int64_t lo = blockIdx.x * chunk, hi = lo + chunk < n ? lo + chunk : n;
    double sum = 0.0, mn = INFINITY, mx = -INFINITY;
    for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
        const double v = y[i];
        sum += v;
        mn = fmin(mn, v);
        mx = fmax(mx, v);
    }
    sum = wave_sum(sum);
    for (int m = 32; m >= 1; m >>= 1) {
        mn = fmin(mn, __shfl_xor(mn, m));
        mx = fmax(mx, __shfl_xor(mx, m));
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = sum;
        red[1][threadIdx.x >> 6] = mn;
        red[2][threadIdx.x >> 6] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        st->part[0][blockIdx.x] = ((red[0][0] + red[0][1]) + red[0][2]) + red[0][3];
        st->part[1][blockIdx.x] = fmin(fmin(red[1][0], red[1][1]), fmin(red[1][2], red[1][3]));
        st->part[2][blockIdx.x] = fmax(fmax(red[2][0], red[2][1]), fmax(red[2][2], red[2][3]));
    }
}

__device__ double pot_quantile(double t, double gamma, double sigma, double ratio)
{
    if (fabs(gamma) < 1e-9)
        return t - sigma * log(ratio);
    return t + sigma / gamma * (pow(ratio, -gamma) - 1.0);
}

__device__ void pot_finish(PotState *st, double gamma, double sigma, int method, double q)
{
    const double ratio = q * static_cast<double>(st->n_cal) / static_cast<double>(st->n_peaks);
    st->gamma = gamma;
    st->sigma = sigma;
    st->method = method;
    st->z = method == 0 ? st->t : pot_quantile(st->t, gamma, sigma, ratio);
    st->phase = kPotDone;
}

// One block: the excesses' statistics; below ten peaks the whole fit (method of moments on the
// sorted excesses), else the grids of both admissible intervals.
__global__ __launch_bounds__(1024) void k_pot_fit_begin(const double *__restrict__ y, double q,
                                                        PotState *__restrict__ st)
{
    __shared__ double s_mean, s_min, s_max;
    const int tid = threadIdx.x;
    if (st->err)
        return;
    const int64_t n = st->n_peaks;
    if (n < 10) {
        if (tid == 0) {
            double ex[10];
            int k = 0;
            bool finite = true;
            for (; k < n; ++k) {   // insertion sort
                const double v = y[k];
                finite &= isfinite(v);
                int i = k;
                for (; i > 0 && ex[i - 1] > v; --i)
                    ex[i] = ex[i - 1];
                ex[i] = v;
            }
            double m = 0.0, s2 = 0.0;
            for (int i = 0; i < k; ++i)
                m += ex[i];
            m /= static_cast<double>(n);
            for (int i = 0; i < k; ++i)
                s2 += (ex[i] - m) * (ex[i] - m);
            s2 /= static_cast<double>(n - 1);       // unbiased sample variance
            if (!finite)
                st->err = kPotNotFinite;
            else if (n < 2 || !(s2 > 0.0))
                pot_finish(st, NAN, NAN, 0, q);
            else
                pot_finish(st, 0.5 * (1.0 - m * m / s2), 0.5 * m * (1.0 + m * m / s2), 1, q);
        }
        return;
    }
    if (tid < 64) {
        // lane l holds the partials l, l + 64, ... in order, a butterfly the lanes
        double sum = 0.0, mn = INFINITY, mx = -INFINITY;
        for (int i = tid; i < kPotStatBlocks; i += 64) {
            sum += st->part[0][i];
            mn = fmin(mn, st->part[1][i]);
            mx = fmax(mx, st->part[2][i]);
        }
        sum = wave_sum(sum);
        for (int m = 32; m >= 1; m >>= 1) {
            mn = fmin(mn, __shfl_xor(mn, m));
            mx = fmax(mx, __shfl_xor(mx, m));
        }
        if (tid == 0) {
            st->ysum = sum;
            if (!isfinite(sum) || !isfinite(mx))
                st->err = kPotNotFinite;
            s_mean = sum / static_cast<double>(n);
            s_min = mn;
            s_max = mx;
        }
    }
    __syncthreads();
    const double ymean = s_mean, ymin = s_min, ymax = s_max;
    const double eps = 1e-8 / ymean;
    const double f0 = eps * ymax, right = 2.0 * (ymean - ymin) / (ymin * ymin);
    const bool has_left = f0 < 0.5, has_right = right > 2.0 * eps;
    const int i = tid % kPotGridPoints;
    const double at = static_cast<double>(i) / static_cast<double>(kPotGridPoints - 1);
    if (tid < kPotGridPoints) {
        if (has_left) {
            const double zlo = log(f0 / (1.0 - f0)), zhi = 30.0;
            const double z = zlo + (zhi - zlo) * at;
            st->xs[i] = -(1.0 / (1.0 + exp(-z))) / ymax;
        }
    } else if (has_right) {
        st->xs[(has_left ? kPotGridPoints : 0) + i] = eps * pow(right / eps, at);
    }
    if (tid == 0)
        st->npts = ((has_left ? 1 : 0) + (has_right ? 1 : 0)) * kPotGridPoints;
}

// Chunks of the excesses for npts evaluation points: about 2048 blocks in all (eight per compute
// unit: the fp64 reciprocal and logarithm chains need several waves per SIMD), and at least 1024
// excesses per chunk.
__device__ __forceinline__ int pot_split(int64_t n, int groups)
{
    int64_t s = (2048 + groups - 1) / groups;
    const int64_t cap = n / 1024;
    s = s > cap ? cap : s;
    return static_cast<int>(s < 1 ? 1 : s);
}

// Likelihood sums at the state's points: item (group of kPotX points, chunk of the excesses), each
// excess loaded once for the group's points. part[v][chunk][point], v = sum xy/(1+xy), sum
// log1p(xy) and, in Newton steps, their derivatives sum y/(1+xy)^2 and sum y/(1+xy).
template <bool DER>
__device__ __forceinline__ void pot_eval_item(const double *__restrict__ y, const PotState *__restrict__ st, int grp,
                                              int j, int nsplit, int64_t n, int npts, double (*red)[4 * kPotX],
                                              double *__restrict__ part)
{
    constexpr int NV = DER ? 4 : 2;
    double x[kPotX];
#pragma unroll
    for (int k = 0; k < kPotX; ++k) {
        const int i = grp * kPotX + k;
        x[k] = i < npts ? st->xs[i] : 0.0;
    }
    const int64_t chunk = (n + nsplit - 1) / nsplit;
    const int64_t lo = j * chunk, hi = lo + chunk < n ? lo + chunk : n;
    double acc[NV][kPotX];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int k = 0; k < kPotX; ++k)
            acc[v][k] = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
        const double yi = y[i];
#pragma unroll
        for (int k = 0; k < kPotX; ++k) {
            double ta, tb, r;
            gpd_terms(x[k] * yi, ta, tb, r);
            acc[0][k] += ta;
            acc[1][k] += tb;
            if constexpr (DER) {
                const double yr = yi * r;
                acc[2][k] += yr * r;
                acc[3][k] += yr;
            }
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int k = 0; k < kPotX; ++k)
            acc[v][k] = wave_sum(acc[v][k]);
    __syncthreads();   // the previous item's sums are no longer read
    if (lane == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int k = 0; k < kPotX; ++k)
                red[wave][v * kPotX + k] = acc[v][k];
    }
    __syncthreads();
    if (threadIdx.x < NV * kPotX) {
        const int v = threadIdx.x / kPotX, k = threadIdx.x - v * kPotX, c = threadIdx.x;
        const int i = grp * kPotX + k;
        if (i < npts)
            part[(static_cast<int64_t>(v) * nsplit + j) * npts + i] =
                ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
    }
}

__global__ __launch_bounds__(256) void k_pot_eval(const double *__restrict__ y, const PotState *__restrict__ st,
                                                  double *__restrict__ part)
{
    __shared__ double red[4][4 * kPotX];
    if (st->err || st->phase == kPotDone)
        return;
    const int npts = st->npts;
    const int64_t n = st->n_peaks;
    const int groups = (npts + kPotX - 1) / kPotX;
    if (groups == 0)
        return;
    const int nsplit = pot_split(n, groups);
    for (int it = blockIdx.x; it < groups * nsplit; it += gridDim.x) {
        const int grp = it / nsplit, j = it - grp * nsplit;
        if (st->phase == kPotNewton)
            pot_eval_item<true>(y, st, grp, j, nsplit, n, npts, red, part);
        else
            pot_eval_item<false>(y, st, grp, j, nsplit, n, npts, red, part);
    }
}

__device__ __forceinline__ double pot_w(double sa, double sb, double n)
{
    const double a = sa / n, b = sb / n;
    return b - a - a * b;
}

// One block: adds the chunk sums of every point (fixed order) and moves the fit on.
__global__ __launch_bounds__(1024) void k_pot_step(const double *__restrict__ part, double q, PotState *__restrict__ st)
{
    __shared__ int s_roots, s_br, wr[16], wb[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (st->err || st->phase == kPotDone)
        return;
    const int phase = st->phase, npts = st->npts;
    const int64_t n = st->n_peaks;
    const double N = static_cast<double>(n);
    const int groups = (npts + kPotX - 1) / kPotX;
    const int nsplit = groups ? pot_split(n, groups) : 1;
    const int nv = phase == kPotNewton ? 4 : 2;
    if (npts > 64) {
        // thread per point: the chunks in order, eight loads in flight
        for (int v = 0; v < nv; ++v)
            for (int i = tid; i < npts; i += 1024) {
                const double *p = part + static_cast<int64_t>(v) * nsplit * npts + i;
                double s = 0.0;
                for (int j0 = 0; j0 < nsplit; j0 += 8) {
                    double t[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        t[u] = j0 + u < nsplit ? p[static_cast<int64_t>(j0 + u) * npts] : 0.0;
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        s += t[u];
                }
                st->sum[v][i] = s;
            }
    } else {
        // wave per (sum, point): lane l the chunks l, l + 64, ..., then a butterfly
        for (int k = wave; k < nv * npts; k += 16) {
            const int v = k / npts, i = k - v * npts;
            const double *p = part + static_cast<int64_t>(v) * nsplit * npts + i;
            double s = 0.0;
            for (int j = lane; j < nsplit; j += 64)
                s += p[static_cast<int64_t>(j) * npts];
            s = wave_sum(s);
            if (lane == 0)
                st->sum[v][i] = s;
        }
    }
    __threadfence_block();
    __syncthreads();
    if (phase == kPotGrid) {
        // exact roots and sign changes to the next point of the same grid, both in grid order
        const int i = tid, gi = i % kPotGridPoints;
        double wi = 0.0, wn = 0.0;
        bool root = false, br = false;
        if (i < npts) {
            wi = pot_w(st->sum[0][i], st->sum[1][i], N);
            root = wi == 0.0;
            if (!root && gi + 1 < kPotGridPoints) {
                wn = pot_w(st->sum[0][i + 1], st->sum[1][i + 1], N);
                br = wi * wn < 0.0;
            }
        }
        const uint64_t mr = __ballot(root), mb = __ballot(br), below = (1ull << lane) - 1ull;
        if (lane == 0) {
            wr[wave] = __popcll(mr);
            wb[wave] = __popcll(mb);
        }
        if (tid == 0)
            s_roots = s_br = 0;
        __syncthreads();
        int ra = __popcll(mr & below), ba = __popcll(mb & below);
        for (int k = 0; k < 16; ++k) {
            if (k < wave) {
                ra += wr[k];
                ba += wb[k];
            }
            if (tid == 0) {
                s_roots += wr[k];
                s_br += wb[k];
            }
        }
        if (root)
            st->roots[ra] = st->xs[i];
        if (br) {
            const double x0 = st->xs[i], x1 = st->xs[i + 1];
            const double lo = x0 < x1 ? x0 : x1, hi = x0 < x1 ? x1 : x0;
            const double xsec = x0 - wi * (x1 - x0) / (wn - wi);
            PotBracket k;
            k.lo = lo;
            k.hi = hi;
            k.wlo = x0 < x1 ? wi : wn;
            k.whi = x0 < x1 ? wn : wi;
            k.lo_neg = k.wlo < 0.0;
            k.x = xsec > lo && xsec < hi ? xsec : 0.5 * (lo + hi);
            k.root = 0.0;
            k.done = 0;
            k.side = 0;
            k.evals = 0;
            st->br[ba] = k;
        }
        __threadfence_block();
        __syncthreads();
        if (tid == 0) {
            st->n_roots = s_roots;
            st->n_br = s_br;
        }
    } else if (phase == kPotNewton) {
        // thread per open bracket (point i belongs to bracket owner[i])
        for (int i = tid; i < npts; i += 1024) {
            PotBracket k = st->br[st->owner[i]];
            const double x = k.x;
            const double a = st->sum[0][i] / N, b = st->sum[1][i] / N, da = st->sum[2][i] / N,
                         db = st->sum[3][i] / N;
            const double wv = b - a - a * b;
            const double wd = db - da - da * b - a * db;
            if (wv == 0.0) {
                k.done = 1;
                k.root = x;
            } else {
                const int side = (wv < 0.0) == (k.lo_neg != 0) ? -1 : 1;
                if (side < 0) {
                    k.lo = x;
                    k.wlo = wv;
                    if (k.side < 0)
                        k.whi *= 0.5;
                } else {
                    k.hi = x;
                    k.whi = wv;
                    if (k.side > 0)
                        k.wlo *= 0.5;
                }
                k.side = side;
                const double xn = x - wv / wd;
                const bool inside = xn > k.lo && xn < k.hi;     // false for NaN
                // when the Newton step leaves the bracket: false position through the ends, else
                // the midpoint
                const double xf = k.lo - k.wlo * (k.hi - k.lo) / (k.whi - k.wlo);
                const double mid = xf > k.lo && xf < k.hi ? xf : 0.5 * (k.lo + k.hi);
                const double tol = 0x1p-26 * fmax(fabs(k.lo), fabs(k.hi));
                ++k.evals;
                // |w| within the rounding of the sums it is formed from: x is a root to fp64 resolution
                if (fabs(wv) <= 0x1p-46 * (fabs(b) + fabs(a) + fabs(a * b))) {
                    k.done = 1;
                    k.root = x;
                } else if (inside && fabs(xn - x) <= tol) {
                    k.done = 1;
                    k.root = xn;
                } else if (!inside && !(mid > k.lo && mid < k.hi)) {
                    k.done = 1;
                    k.root = mid;
                } else {
                    k.x = inside ? xn : mid;
                    if (k.evals >= kPotRounds) {
                        k.done = 1;
                        k.root = k.x;
                    }
                }
            }
            st->br[st->owner[i]] = k;
        }
    } else if (tid == 0) {
        // candidates: the exponential tail and every root
        const double ymean = st->ysum / N;
        double bg = 0.0, bs = ymean;
        double bl = -N * log(ymean) - st->ysum / ymean;
        for (int i = 0; i < npts; ++i) {
            const double g = st->sum[1][i] / N;
            if (g == 0.0 || !isfinite(g))
                continue;
            const double s = g / st->xs[i];
            if (!(s > 0.0))
                continue;
            const double ll = -N * log(s) - (1.0 + 1.0 / g) * st->sum[1][i];   // sum log1p(g y / s)
            if (ll > bl || (ll == bl && fabs(g) < fabs(bg))) {
                bg = g;
                bs = s;
                bl = ll;
            }
        }
        pot_finish(st, bg, bs, 2, q);
    }
    if (phase == kPotLast)
        return;
    __threadfence_block();
    __syncthreads();
    if (tid == 0) {
        // the open brackets' points, or once none is left every root's
        int k = 0;
        for (int b = 0; b < st->n_br; ++b)
            if (!st->br[b].done) {
                st->owner[k] = b;
                st->xs[k++] = st->br[b].x;
            }
        if (k > 0) {
            st->phase = kPotNewton;
        } else {
            for (; k < st->n_roots; ++k)
                st->xs[k] = st->roots[k];
            for (int b = 0; b < st->n_br; ++b)
                st->xs[k++] = st->br[b].root;
            st->phase = kPotLast;
        }
        st->npts = k;
    }
}

// The result for the host, and the flags of every score once the fit has ended.
__global__ __launch_bounds__(256) void k_pot_flag(const float *__restrict__ scores, int64_t n,
                                                  const PotState *__restrict__ st, PotOut *__restrict__ out,
                                                  uint8_t *__restrict__ flags)
{
    if (blockIdx.x == 0 && threadIdx.x == 0)
        *out = PotOut{st->err, st->phase, st->method, 0, st->n_cal, st->n_peaks, st->t, st->z, st->gamma, st->sigma};
    if (!flags || st->err || st->phase != kPotDone)
        return;
    const float thr = static_cast<float>(st->z);
    const int64_t step = static_cast<int64_t>(gridDim.x) * 256;
    for (int64_t i = blockIdx.x * 256LL + threadIdx.x; i < n; i += step)
        flags[i] = scores[i] > thr ? 1 : 0;
}

}  // namespace

// Scores per thread: few where there are few scores, so that they still fill the chip.
static int pot_items(int64_t n_windows) { return n_windows > (4 << 20) ? 16 : 4; }

int64_t pot_blocks(int64_t n_windows)
{
    const int64_t per = 256LL * pot_items(n_windows);
    return (n_windows + per - 1) / per;
}

hipError_t launch_pot_select(const Geometry &g, const float *scores, const int64_t *soff, const int64_t *woff, int n,
                             int64_t n_windows, double level, const PotWork &w, hipStream_t st)
{
    hipLaunchKernelGGL(k_pot_begin, dim3(1), dim3(1024), 0, st, soff, woff, n, g.W, g.S, g.ref_frac, level, w.cal,
                       w.state);
    const dim3 grid(static_cast<unsigned>(pot_blocks(n_windows)));
    const bool wide = pot_items(n_windows) == 16;
    // about 8192 blocks, four to a place on the chip, where there are more runs than that
    const int rounds = static_cast<int>((pot_blocks(n_windows) + 8191) / 8192);
    const dim3 hgrid(static_cast<unsigned>((pot_blocks(n_windows) + rounds - 1) / rounds));
    for (int pass = 0; pass < kPotPasses; ++pass)
        if (wide)
            hipLaunchKernelGGL(k_pot_hist<16>, hgrid, dim3(256), 0, st, scores, woff, w.cal, n, pass, rounds, w.state);
        else
            hipLaunchKernelGGL(k_pot_hist<4>, hgrid, dim3(256), 0, st, scores, woff, w.cal, n, pass, rounds, w.state);
    if (wide)
        hipLaunchKernelGGL(k_pot_count<16>, grid, dim3(256), 0, st, scores, woff, w.cal, n, w.state, w.counts);
    else
        hipLaunchKernelGGL(k_pot_count<4>, grid, dim3(256), 0, st, scores, woff, w.cal, n, w.state, w.counts);
    return hipGetLastError();
}

hipError_t launch_pot_peaks(const float *scores, const int64_t *woff, int n, int64_t n_windows, double q,
                            const PotWork &w, hipStream_t st)
{
    const int64_t nblk = pot_blocks(n_windows);
    hipLaunchKernelGGL(k_pot_offsets, dim3(1), dim3(1024), 0, st, w.counts, nblk, w.offsets, w.state, w.cap);
    const dim3 grid(static_cast<unsigned>(nblk));
    if (pot_items(n_windows) == 16)
        hipLaunchKernelGGL(k_pot_compact<16>, grid, dim3(256), 0, st, scores, woff, w.cal, n, w.state, w.offsets,
                           w.y, w.cap);
    else
        hipLaunchKernelGGL(k_pot_compact<4>, grid, dim3(256), 0, st, scores, woff, w.cal, n, w.state, w.offsets, w.y,
                           w.cap);
    hipLaunchKernelGGL(k_pot_stats, dim3(kPotStatBlocks), dim3(256), 0, st, w.y, w.state);
    hipLaunchKernelGGL(k_pot_fit_begin, dim3(1), dim3(1024), 0, st, w.y, q, w.state);
    return hipGetLastError();
}

hipError_t launch_pot_rounds(int rounds, double q, const PotWork &w, hipStream_t st)
{
    // blocks for the most items an evaluation of w.cap excesses can have
    const int64_t chunks = std::max<int64_t>(1, w.cap / 1024);
    const unsigned grid = static_cast<unsigned>(std::min<int64_t>(2048, 2 * kPotGridPoints / kPotX * chunks));
    for (int r = 0; r < rounds; ++r) {
        hipLaunchKernelGGL(k_pot_eval, dim3(grid), dim3(256), 0, st, w.y, w.state, w.part);
        hipLaunchKernelGGL(k_pot_step, dim3(1), dim3(1024), 0, st, w.part, q, w.state);
    }
    return hipGetLastError();
}

hipError_t launch_pot_flag(const float *scores, int64_t n_windows, const PotWork &w, PotOut *out, uint8_t *flags,
                           hipStream_t st)
{
    int64_t blocks = flags ? (n_windows + 1023) / 1024 : 1;
    if (blocks > 8192)
        blocks = 8192;
    hipLaunchKernelGGL(k_pot_flag, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, scores, n_windows, w.state,
                       out, flags);
    return hipGetLastError();
}

}  // namespace enova
