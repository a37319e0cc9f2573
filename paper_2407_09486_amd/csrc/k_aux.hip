// Bandwidth-bound helper kernels: reference statistics, per-stream scans, flags and the
// radix-select passes of the peaks-over-threshold calibration.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "gpd_math.h"
#include "internal.h"

namespace enova {

namespace {

template <int DT>
__device__ __forceinline__ float load_x(const void *x, int64_t idx)
{
    if constexpr (DT == ENOVA_F32) {
        return static_cast<const float *>(x)[idx];
    } else {
        uint32_t b = static_cast<const uint16_t *>(x)[idx];
        return __uint_as_float(b << 16);
    }
}

__device__ __forceinline__ int64_t ref_len_dev(float ref_frac, int64_t T)
{
    return static_cast<int64_t>(floor(static_cast<double>(ref_frac) * static_cast<double>(T)));
}

__device__ __forceinline__ void finish_stats(double x0, double s1, double s2, int64_t R, float *mean,
                                             float *std)
{
    if (R <= 0) {
        *mean = 0.0f;
        *std = 1.0f;
        return;
    }
    const double inv = 1.0 / static_cast<double>(R);
    const double m1 = s1 * inv;
    const double mu = x0 + m1;
    double var = s2 * inv - m1 * m1;
    var = var > 0.0 ? var : 0.0;
    double sd = sqrt(var);
    if (sd <= 1e-6 * fmax(1.0, fabs(mu)))
        sd = 1.0;   // the metric is constant over the reference prefix
    *mean = static_cast<float>(mu);
    *std = static_cast<float>(sd);
}

// Reference statistics. A stream's reference prefix of R steps is cut into K = stat_chunks(R, M)
// chunks of equal length (the last one shorter): each chunk's sums (fp64, of the values less the
// stream's first value of the metric, and of their squares) are formed in a fixed order, and the K
// chunk sums are added in order, so a stream's statistics depend on that stream alone and not on
// how the chunks are spread over blocks.
constexpr int kStatThreads = 256;
constexpr int kStatMaxChunks = 32;
constexpr int kStatChunk = 16384;   // elements of a chunk at the least (64 per thread)

__device__ __forceinline__ int stat_chunks(int64_t R, int M)
{
    const int64_t k = (R * M + kStatChunk - 1) / kStatChunk;
    return static_cast<int>(k < 1 ? 1 : (k > kStatMaxChunks ? kStatMaxChunks : k));
}

// VEC consecutive elements from idx (a multiple of VEC) of a 16-byte aligned x, in one load.
template <int DT, int VEC>
__device__ __forceinline__ void load_vec(const void *x, int64_t idx, float (&v)[VEC])
{
    if constexpr (VEC == 1) {
        v[0] = load_x<DT>(x, idx);
    } else if constexpr (DT == ENOVA_F32) {
        static_assert(VEC == 4, "16-byte loads");
        const float4 q = *reinterpret_cast<const float4 *>(static_cast<const float *>(x) + idx);
        v[0] = q.x;
        v[1] = q.y;
        v[2] = q.z;
        v[3] = q.w;
    } else {
        static_assert(VEC == 4, "8-byte loads");
        const uint2 q = *reinterpret_cast<const uint2 *>(static_cast<const uint16_t *>(x) + idx);
        v[0] = __uint_as_float(q.x << 16);
        v[1] = __uint_as_float(q.x & 0xffff0000u);
        v[2] = __uint_as_float(q.y << 16);
        v[3] = __uint_as_float(q.y & 0xffff0000u);
    }
}

// Sums of the metrics m0 .. m0 + mc - 1 (mc <= 256) over the steps t0 .. t1 - 1 of one stream,
// whose first value of metric m0 + c is x[at + c]: with nc = mc / VEC, thread tid < per * nc takes
// the VEC metrics from m0 + (tid % nc) * VEC and every per-th step from tid / nc on (neighbouring
// lanes read neighbouring elements also where nc does not divide 256, whose last 256 % nc threads
// idle), several loads in flight; then thread c < mc adds the partial sums of its metric in step
// order. a, b: that metric's sums.
template <int DT, int VEC>
__device__ __forceinline__ void stat_chunk(const void *__restrict__ x, int64_t at, int M, int mc, int64_t t0,
                                           int64_t t1, double (*red)[VEC][kStatThreads], double &a, double &b)
{
    constexpr int U = 8;
    const int tid = threadIdx.x;
    const int nc = mc / VEC;
    const int per = kStatThreads / nc;
    const int r = tid / nc, c = (tid - r * nc) * VEC;
    double s1[VEC], s2[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e)
        s1[e] = s2[e] = 0.0;
    if (r < per && t0 < t1) {
        double x0[VEC];
        float v[U][VEC];
        load_vec<DT, VEC>(x, at + c, v[0]);
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            x0[e] = static_cast<double>(v[0][e]);
        auto add = [&](const float (&q)[VEC]) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const double d = static_cast<double>(q[e]) - x0[e];
                s1[e] += d;
                s2[e] = fma(d, d, s2[e]);
            }
        };
        const int64_t step = static_cast<int64_t>(per) * M;
        int64_t i = at + (t0 + r) * M + c;
        const int64_t end = at + t1 * M;   // step t's element at + t M + c lies below it iff t < t1
        for (; i + (U - 1) * step < end; i += U * step) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                load_vec<DT, VEC>(x, i + u * step, v[u]);
#pragma unroll
            for (int u = 0; u < U; ++u)
                add(v[u]);
        }
        for (; i < end; i += step) {
            load_vec<DT, VEC>(x, i, v[0]);
            add(v[0]);
        }
    }
    // lanes of a wave with the same metrics add up by a butterfly where nc divides a wave, which
    // leaves one partial sum per wave; otherwise every thread keeps its own
    const bool fold = nc <= 64 && 64 % nc == 0;
    if (fold)
        for (int off = 32; off >= nc; off >>= 1)
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                s1[e] += __shfl_xor(s1[e], off);
                s2[e] += __shfl_xor(s2[e], off);
            }
    __syncthreads();   // the previous chunk's sums are no longer read
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        red[0][e][tid] = s1[e];
        red[1][e][tid] = s2[e];
    }
    __syncthreads();
    a = b = 0.0;
    if (tid < mc) {
        const int e = tid % VEC, k = tid / VEC;
        const int n = fold ? kStatThreads / 64 : per, d = fold ? 64 : nc;
        for (int j = 0; j < n; ++j) {
            a += red[0][e][k + j * d];
            b += red[1][e][k + j * d];
        }
    }
}

// Block (s, j) of n x G: the chunks j, j + G, ... of stream s. With G = 1 the block holds every
// chunk and writes the statistics; otherwise it writes its chunks' sums to part[s][chunk][M][2]
// and stat_finish adds them. The work is HBM-bound (half the input once): one block per stream
// left the chip idle on few streams and waited for the longest of ragged ones, and metric counts
// that do not divide 256 took one thread per metric (96 streams x 7 metrics x 10k steps: 1.05 ms,
// now 0.01).
template <int DT, int VEC>
__device__ __forceinline__ void ref_stats_block(const void *__restrict__ x, const int64_t *__restrict__ soff, int M,
                                                float ref_frac, int s, int j, int G, double *__restrict__ part,
                                                float *__restrict__ mean, float *__restrict__ std)
{
    __shared__ double red[2][VEC][kStatThreads];
    const int tid = threadIdx.x;
    const int64_t base = soff[s];
    const int64_t R = ref_len_dev(ref_frac, soff[s + 1] - base);
    const int K = stat_chunks(R, M);
    if (j >= K)
        return;
    const int64_t len = (R + K - 1) / K;
    for (int m0 = 0; m0 < M; m0 += kStatThreads) {
        const int mc = M - m0 < kStatThreads ? M - m0 : kStatThreads;
        const int64_t at = base * M + m0;
        double sa = 0.0, sb = 0.0;
        for (int k = j; k < K; k += G) {
            const int64_t t0 = k * len, t1 = t0 + len < R ? t0 + len : R;
            double a, b;
            stat_chunk<DT, VEC>(x, at, M, mc, t0, t1, red, a, b);
            if (tid < mc && G > 1) {
                double *p = part + ((static_cast<int64_t>(s) * kStatMaxChunks + k) * M + m0 + tid) * 2;
                p[0] = a;
                p[1] = b;
            }
            sa += a;
            sb += b;
        }
        if (tid < mc && G == 1) {
            const double x0 = R > 0 ? static_cast<double>(load_x<DT>(x, at + tid)) : 0.0;
            const int64_t o = static_cast<int64_t>(s) * M + m0 + tid;
            finish_stats(x0, sa, sb, R, mean + o, std + o);
        }
    }
}

// Statistics i = s * M + m of the streams whose chunk sums are in part (added in chunk order,
// eight loads in flight).
template <int DT>
__device__ __forceinline__ void stat_finish(const void *__restrict__ x, const int64_t *__restrict__ soff, int M,
                                            float ref_frac, int64_t i, const double *__restrict__ part,
                                            float *__restrict__ mean, float *__restrict__ std)
{
    const int64_t s = i / M, m = i - s * M;
    const int64_t base = soff[s];
    const int64_t R = ref_len_dev(ref_frac, soff[s + 1] - base);
    const int K = stat_chunks(R, M);
    const double2 *p = reinterpret_cast<const double2 *>(part) + s * kStatMaxChunks * M + m;
    const double x0 = R > 0 ? static_cast<double>(load_x<DT>(x, base * M + m)) : 0.0;
    double sa = 0.0, sb = 0.0;
    for (int k0 = 0; k0 < K; k0 += 8) {
        double2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v[u] = k0 + u < K ? p[static_cast<int64_t>(k0 + u) * M] : make_double2(0.0, 0.0);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            sa += v[u].x;
            sb += v[u].y;
        }
    }
    finish_stats(x0, sa, sb, R, mean + i, std + i);
}

template <int DT, int VEC>
__global__ __launch_bounds__(kStatThreads) void k_ref_stats(const void *__restrict__ x,
                                                            const int64_t *__restrict__ soff, int M, float ref_frac,
                                                            int G, double *__restrict__ part,
                                                            float *__restrict__ mean, float *__restrict__ std)
{
    const int s = blockIdx.x / G;
    ref_stats_block<DT, VEC>(x, soff, M, ref_frac, s, blockIdx.x - s * G, G, part, mean, std);
}

template <int DT>
__global__ __launch_bounds__(256) void k_stat_finish(const void *__restrict__ x, const int64_t *__restrict__ soff,
                                                     int64_t total, int M, float ref_frac,
                                                     const double *__restrict__ part, float *__restrict__ mean,
                                                     float *__restrict__ std)
{
    const int64_t i = blockIdx.x * 256LL + threadIdx.x;
    if (i < total)
        stat_finish<DT>(x, soff, M, ref_frac, i, part, mean, std);
}

// Exclusive prefix of each thread's value over the block's NT threads, and the block's total: a
// shuffle scan in each wave, then the wave totals in wave order (integer sums: any order gives
// the same). Two barriers; one thread walking the 1024 sums in LDS took 10 of the kernel's 13 us.
template <int NT>
__device__ __forceinline__ int64_t block_scan_excl(int64_t v, int64_t *wsum, int64_t &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int64_t o = __shfl_up(inc, off);
        if (lane >= off)
            inc += o;
    }
    if (lane == 63)
        wsum[wave] = inc;
    __syncthreads();
    int64_t base = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
        const int64_t t = wsum[w];
        base += w < wave ? t : 0;
        sum += t;
    }
    total = sum;
    return base + inc - v;
}

// Single-block exclusive scan of a per-stream count (see launch_stream_scan).
struct ScanArgs {
    const int64_t *soff, *woff;
    int n, mode, div, W, S;
    float ref_frac;
    int64_t *out;
};

template <int NT>
__device__ __forceinline__ void stream_scan_block(const ScanArgs &g, int64_t *wsum)
{
    const int tid = threadIdx.x;
    const int64_t chunk = (static_cast<int64_t>(g.n) + NT - 1) / NT;
    const int64_t a = tid * chunk;
    const int64_t b = a + chunk < g.n ? a + chunk : g.n;
    auto count = [&](int64_t s) -> int64_t {
        int64_t c = g.woff[s + 1] - g.woff[s];
        if (g.mode == 1) {
            const int64_t R = ref_len_dev(g.ref_frac, g.soff[s + 1] - g.soff[s]);
            const int64_t cal = R >= g.W ? (R - g.W) / g.S + 1 : 0;
            c = cal < c ? cal : c;
        }
        return g.div > 1 ? (c + g.div - 1) / g.div : c;
    };
    int64_t local = 0;
    for (int64_t s = a; s < b; ++s)
        local += count(s);
    int64_t total;
    int64_t run = block_scan_excl<NT>(local, wsum, total);
    if (tid == 0)
        g.out[g.n] = total;
    for (int64_t s = a; s < b; ++s) {
        g.out[s] = run;
        run += count(s);
    }
}

__global__ __launch_bounds__(1024) void k_stream_scan(ScanArgs g)
{
    __shared__ int64_t wsum[16];
    stream_scan_block<1024>(g, wsum);
}

// First launch of a scoring pass: block 0 scans the tile counts while the others form the
// reference statistics (chunk sums when G > 1), which the scan does not need; the second launch,
// k_tile_map, then maps the tiles and finishes the statistics. Two launches instead of four, and
// the scan (3 us) hidden behind the statistics.
template <int DT, int VEC>
__global__ __launch_bounds__(kStatThreads) void k_prep(ScanArgs g, const void *__restrict__ x, int M, int G,
                                                       double *__restrict__ part, float *__restrict__ mean,
                                                       float *__restrict__ std)
{
    if (blockIdx.x == 0) {
        __shared__ int64_t wsum[kStatThreads / 64];
        stream_scan_block<kStatThreads>(g, wsum);
        return;
    }
    const int b = blockIdx.x - 1;
    const int s = b / G;
    ref_stats_block<DT, VEC>(x, g.soff, M, g.ref_frac, s, b - s * G, G, part, mean, std);
}

// Stream of every tile of the matrix-core kernel (one binary search per tile, done once here
// with full occupancy instead of as a chain of dependent loads at the start of each tile), and
// with f.part the statistics whose chunk sums k_prep left there.
struct StatFinish {
    const double *part;
    const void *x;
    const int64_t *soff;
    int dtype, M;
    float ref_frac;
    float *mean, *std;
};

__global__ __launch_bounds__(256) void k_tile_map(const int64_t *__restrict__ tile_off, int n, int64_t grid,
                                                  int *__restrict__ map, StatFinish f)
{
    const int64_t first = blockIdx.x * 256LL + threadIdx.x, step = static_cast<int64_t>(gridDim.x) * 256;
    if (f.part)
        for (int64_t i = first; i < static_cast<int64_t>(n) * f.M; i += step) {
            if (f.dtype == ENOVA_F32)
                stat_finish<ENOVA_F32>(f.x, f.soff, f.M, f.ref_frac, i, f.part, f.mean, f.std);
            else
                stat_finish<ENOVA_BF16>(f.x, f.soff, f.M, f.ref_frac, i, f.part, f.mean, f.std);
        }
    const int64_t total = tile_off[n];
    for (int64_t b = first; b < grid; b += step) {
        int s = -1;
        if (b < total) {
            int lo = 0, hi = n - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (tile_off[mid] <= b)
                    lo = mid;
                else
                    hi = mid - 1;
            }
            s = lo;
        }
        map[b] = s;
    }
}

__global__ void k_flag(const float *__restrict__ scores, int64_t n, float thr,
                       uint8_t *__restrict__ flags)
{
    const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += stride)
        flags[i] = scores[i] > thr ? 1 : 0;
}

// Order-preserving map of a float to an unsigned key.
__device__ __forceinline__ uint32_t fkey(float f)
{
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

constexpr int kCalItems = 16;   // calibration scores per thread per block

// Upper-bound search: the stream s with cal_off[s] <= ci < cal_off[s+1].
__device__ __forceinline__ int find_stream(const int64_t *off, int n, int64_t ci)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (off[mid] <= ci)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

__global__ __launch_bounds__(256) void k_calib_hist(const float *__restrict__ scores,
                                                    const int64_t *__restrict__ woff,
                                                    const int64_t *__restrict__ cal_off, int n,
                                                    int64_t n_cal, int shift,
                                                    const RadixState *__restrict__ rs,
                                                    unsigned int *__restrict__ hist)
{
    __shared__ unsigned int h[256];
    const int tid = threadIdx.x;
    const uint32_t prefix = rs->prefix;
    h[tid] = 0;
    __syncthreads();
    const int64_t start = static_cast<int64_t>(blockIdx.x) * 256 * kCalItems;
    if (start < n_cal) {
        int s = find_stream(cal_off, n, start);
        for (int j = 0; j < kCalItems; ++j) {
            const int64_t ci = start + static_cast<int64_t>(j) * 256 + tid;
            if (ci >= n_cal)
                break;
            while (cal_off[s + 1] <= ci)
                ++s;
            const uint32_t key = fkey(scores[woff[s] + (ci - cal_off[s])]);
            const bool match = shift >= 24 ? true : ((key >> (shift + 8)) == prefix);
            if (match)
                atomicAdd(&h[(key >> shift) & 255u], 1u);
        }
    }
    __syncthreads();
    if (h[tid])
        atomicAdd(&hist[tid], h[tid]);
}

// The radix state's start: no prefix, the sought rank, nothing above; the bins cleared.
__global__ __launch_bounds__(256) void k_radix_init(RadixState *__restrict__ rs, int64_t rank,
                                                    unsigned int *__restrict__ hist)
{
    hist[threadIdx.x] = 0u;
    if (threadIdx.x == 0) {
        rs->prefix = 0u;
        rs->ok = 1;
        rs->rank = rank;
        rs->n_greater = 0;
    }
}

// One block of 256 threads, thread d holding bin d: an inclusive scan of the bins (in 64-bit)
// finds the digit whose range [before, before + count) holds the rank; that thread appends the
// digit to the prefix, keeps rank - before and adds the keys of the higher digits. The bins are
// cleared for the next pass.
__global__ __launch_bounds__(256) void k_radix_pick(RadixState *__restrict__ rs, unsigned int *__restrict__ hist)
{
    __shared__ int64_t wsum[4];
    const int d = threadIdx.x, lane = d & 63, wave = d >> 6;
    const int64_t c = hist[d];
    hist[d] = 0u;
    int64_t inc = c;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int64_t o = __shfl_up(inc, off);
        if (lane >= off)
            inc += o;
    }
    if (lane == 63)
        wsum[wave] = inc;
    __syncthreads();
    int64_t base = 0, total = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w < wave)
            base += wsum[w];
        total += wsum[w];
    }
    inc += base;
    const int64_t before = inc - c;
    const int64_t rank = rs->rank;
    __syncthreads();
    if (c > 0 && rank >= before && rank < inc) {
        rs->prefix = (rs->prefix << 8) | static_cast<uint32_t>(d);
        rs->rank = rank - before;
        rs->n_greater += total - inc;
    }
    if (d == 0 && !(rank >= 0 && rank < total))
        rs->ok = 0;
}

// Peaks of the calibration set, pass 1: how many keys above key_t each block holds.
__global__ __launch_bounds__(256) void k_calib_count(const float *__restrict__ scores,
                                                     const int64_t *__restrict__ woff,
                                                     const int64_t *__restrict__ cal_off, int n,
                                                     int64_t n_cal, uint32_t key_t,
                                                     int64_t *__restrict__ block_counts)
{
    __shared__ int wsum[4];
    const int tid = threadIdx.x;
    const int64_t start = static_cast<int64_t>(blockIdx.x) * 256 * kCalItems;
    int cnt = 0;
    int s = find_stream(cal_off, n, start);
    for (int j = 0; j < kCalItems; ++j) {
        const int64_t ci = start + static_cast<int64_t>(j) * 256 + tid;
        if (ci >= n_cal)
            break;
        while (cal_off[s + 1] <= ci)
            ++s;
        cnt += fkey(scores[woff[s] + (ci - cal_off[s])]) > key_t ? 1 : 0;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        cnt += __shfl_xor(cnt, off);
    if ((tid & 63) == 0)
        wsum[tid >> 6] = cnt;
    __syncthreads();
    if (tid == 0)
        block_counts[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

// Pass 2: write the excesses y = score - t of the peaks in calibration order (stable).
__global__ __launch_bounds__(256) void k_calib_compact(const float *__restrict__ scores,
                                                       const int64_t *__restrict__ woff,
                                                       const int64_t *__restrict__ cal_off, int n,
                                                       int64_t n_cal, uint32_t key_t, double t,
                                                       const int64_t *__restrict__ block_off,
                                                       double *__restrict__ y, int64_t cap)
{
    __shared__ int wcnt[4];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int64_t start = static_cast<int64_t>(blockIdx.x) * 256 * kCalItems;
    int64_t run = block_off[blockIdx.x];
    int s = find_stream(cal_off, n, start);
    for (int j = 0; j < kCalItems; ++j) {
        const int64_t ci = start + static_cast<int64_t>(j) * 256 + tid;
        float v = 0.0f;
        bool hit = false;
        if (ci < n_cal) {
            while (cal_off[s + 1] <= ci)
                ++s;
            v = scores[woff[s] + (ci - cal_off[s])];
            hit = fkey(v) > key_t;
        }
        const uint64_t mask = __ballot(hit);
        const int below = __popcll(mask & ((1ull << lane) - 1ull));
        if (lane == 0)
            wcnt[wave] = __popcll(mask);
        __syncthreads();
        int before = 0;
        for (int k = 0; k < wave; ++k)
            before += wcnt[k];
        const int total = wcnt[0] + wcnt[1] + wcnt[2] + wcnt[3];
        const int64_t pos = run + before + below;
        if (hit && pos < cap)
            y[pos] = static_cast<double>(v) - t;
        run += total;
        __syncthreads();
    }
}

// Exclusive scan of n int64 values by one block; out[n] receives the total.
__global__ __launch_bounds__(1024) void k_scan_i64(const int64_t *__restrict__ in, int64_t n,
                                                   int64_t *__restrict__ out)
{
    __shared__ int64_t wsum[16];
    const int tid = threadIdx.x;
    const int64_t chunk = (n + 1023) / 1024;
    const int64_t a = tid * chunk;
    const int64_t b = a + chunk < n ? a + chunk : n;
    int64_t local = 0;
    for (int64_t i = a; i < b; ++i)
        local += in[i];
    int64_t total;
    int64_t r = block_scan_excl<1024>(local, wsum, total);
    if (tid == 0)
        out[n] = total;
    for (int64_t i = a; i < b; ++i) {
        out[i] = r;
        r += in[i];
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

// Likelihood sums of the excesses: block (g, j) covers chunk j of nsplit contiguous chunks of y
// at the kGpdX points xs[g*kGpdX ...] (each excess is loaded once for all of them) and writes
// pa = sum xy/(1+xy), pb = sum log1p(xy) per point in a fixed order (DER: also pda = sum
// y/(1+xy)^2 and pdb = sum y/(1+xy), their derivatives in x). The terms take the device form
// (hardware reciprocal refined by Newton steps, within a few ulps of the divided form).
constexpr int kGpdX = 8;
template <bool DER>
__global__ __launch_bounds__(256) void k_gpd_sums(const double *__restrict__ y, int64_t n,
                                                  const double *__restrict__ xs, int nx, int nsplit,
                                                  double *__restrict__ pa, double *__restrict__ pb,
                                                  double *__restrict__ pda, double *__restrict__ pdb)
{
    constexpr int NV = DER ? 4 : 2;   // sums per point
    __shared__ double red[4][NV * kGpdX];
    const int grp = blockIdx.x / nsplit;
    const int j = blockIdx.x - grp * nsplit;
    double x[kGpdX];
#pragma unroll
    for (int k = 0; k < kGpdX; ++k) {
        const int i = grp * kGpdX + k;
        x[k] = i < nx ? xs[i] : 0.0;
    }
    const int64_t chunk = (n + nsplit - 1) / nsplit;
    const int64_t lo = j * chunk;
    const int64_t hi = lo + chunk < n ? lo + chunk : n;
    double acc[NV][kGpdX];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int k = 0; k < kGpdX; ++k)
            acc[v][k] = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
        const double yi = y[i];
#pragma unroll
        for (int k = 0; k < kGpdX; ++k) {
            double ta, tb, r;
            gpd_terms_fast(x[k] * yi, ta, tb, r);
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
        for (int k = 0; k < kGpdX; ++k)
            acc[v][k] = wave_sum(acc[v][k]);
    if (lane == 0) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int k = 0; k < kGpdX; ++k)
                red[wave][v * kGpdX + k] = acc[v][k];
    }
    __syncthreads();
    if (threadIdx.x < NV * kGpdX) {
        const int v = threadIdx.x / kGpdX, k = threadIdx.x - v * kGpdX;
        const int i = grp * kGpdX + k;
        if (i < nx) {
            double *out = v == 0 ? pa : v == 1 ? pb : v == 2 ? pda : pdb;
            const int c = threadIdx.x;
            out[static_cast<int64_t>(i) * nsplit + j] = ((red[0][c] + red[1][c]) + red[2][c]) + red[3][c];
        }
    }
}

// Sum, minimum and maximum of the excesses: block j of nblk reduces chunk j (fixed order) into
// part[3j..3j+2]; one block then combines the nblk partials in order.
__global__ __launch_bounds__(256) void k_peak_partial(const double *__restrict__ y, int64_t n,
                                                      double *__restrict__ part)
{
    __shared__ double sa[256];
    __shared__ double sb[256];
    __shared__ double sc[256];
    const int tid = threadIdx.x;
    const int64_t chunk = (n + gridDim.x - 1) / gridDim.x;
    const int64_t lo = blockIdx.x * chunk;
    const int64_t hi = lo + chunk < n ? lo + chunk : n;
    double sum = 0.0, mn = INFINITY, mx = -INFINITY;
    for (int64_t i = lo + tid; i < hi; i += 256) {
        const double v = y[i];
        sum += v;
        mn = fmin(mn, v);
        mx = fmax(mx, v);
    }
    sa[tid] = sum;
    sb[tid] = mn;
    sc[tid] = mx;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (tid < w) {
            sa[tid] += sa[tid + w];
            sb[tid] = fmin(sb[tid], sb[tid + w]);
            sc[tid] = fmax(sc[tid], sc[tid + w]);
        }
        __syncthreads();
    }
    if (tid == 0) {
        part[3 * blockIdx.x + 0] = sa[0];
        part[3 * blockIdx.x + 1] = sb[0];
        part[3 * blockIdx.x + 2] = sc[0];
    }
}

__global__ __launch_bounds__(64) void k_peak_final(const double *__restrict__ part, int nblk,
                                                   double *__restrict__ out)
{
    if (threadIdx.x != 0)
        return;
    double sum = 0.0, mn = INFINITY, mx = -INFINITY;
    for (int j = 0; j < nblk; ++j) {
        sum += part[3 * j];
        mn = fmin(mn, part[3 * j + 1]);
        mx = fmax(mx, part[3 * j + 2]);
    }
    out[0] = sum;
    out[1] = mn;
    out[2] = mx;
}

}  // namespace

// Blocks per stream of the reference statistics: about 2048 in all, so that few or ragged streams
// fill the chip (64 streams of 8192 x 8 reference values: 22 -> 14 us; 512 ragged ones of up to
// 32768 x 16: 280 -> 147 us; 1024 of 2048 x 32 in bf16: 36 -> 27 us); from 1024 streams on one block
// each, without partial sums. Four times as many blocks measured slower on short streams (each
// pays its own chain of offset, first-value and reduction latencies: 27 -> 47 us in bf16) and 15%
// faster on the ragged ones only. The chunk sums of a call take at most kStatPartMax bytes.
constexpr size_t kStatPartMax = size_t{64} << 20;

static int stat_split(int n, int M)
{
    const size_t bytes = static_cast<size_t>(n) * kStatMaxChunks * M * 2 * sizeof(double);
    if (n <= 0 || bytes > kStatPartMax)
        return 1;
    const int g = 2048 / n;
    return g < 1 ? 1 : (g > kStatMaxChunks ? kStatMaxChunks : g);
}

size_t stat_part_bytes(int n, int M)
{
    return stat_split(n, M) > 1 ? static_cast<size_t>(n) * kStatMaxChunks * M * 2 * sizeof(double) : 0;
}

// Four metrics per load where a step holds whole groups of them and x is aligned for it.
static bool stat_vec(const Geometry &g, const void *x)
{
    return g.M % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0;
}

static hipError_t launch_stat_blocks(const Geometry &g, const void *x, const int64_t *soff, int n, int G, double *part,
                                     float *mean, float *std, hipStream_t st)
{
    using Kernel = void (*)(const void *, const int64_t *, int, float, int, double *, float *, float *);
    const bool vec = stat_vec(g, x);
    const Kernel k = g.dtype == ENOVA_F32 ? (vec ? static_cast<Kernel>(k_ref_stats<ENOVA_F32, 4>) : k_ref_stats<ENOVA_F32, 1>)
                                          : (vec ? static_cast<Kernel>(k_ref_stats<ENOVA_BF16, 4>) : k_ref_stats<ENOVA_BF16, 1>);
    hipLaunchKernelGGL(k, dim3(static_cast<unsigned>(n) * G), dim3(kStatThreads), 0, st, x, soff, g.M, g.ref_frac, G,
                       part, mean, std);
    return hipGetLastError();
}

hipError_t launch_ref_stats(const Geometry &g, const void *x, const int64_t *soff, int n,
                            float *mean, float *std, double *part, hipStream_t st)
{
    if (n <= 0)
        return hipSuccess;
    const int G = part ? stat_split(n, g.M) : 1;
    const hipError_t e = launch_stat_blocks(g, x, soff, n, G, part, mean, std, st);
    if (e != hipSuccess || G == 1)
        return e;
    const int64_t total = static_cast<int64_t>(n) * g.M;
    const dim3 fin(static_cast<unsigned>((total + 255) / 256));
    if (g.dtype == ENOVA_F32)
        hipLaunchKernelGGL(k_stat_finish<ENOVA_F32>, fin, dim3(256), 0, st, x, soff, total, g.M, g.ref_frac, part,
                           mean, std);
    else
        hipLaunchKernelGGL(k_stat_finish<ENOVA_BF16>, fin, dim3(256), 0, st, x, soff, total, g.M, g.ref_frac, part,
                           mean, std);
    return hipGetLastError();
}

hipError_t launch_stream_scan(const Geometry &g, const int64_t *soff, const int64_t *woff, int n,
                              int mode, int div, int64_t *out, hipStream_t st)
{
    const ScanArgs a{soff, woff, n, mode, div, g.W, g.S, g.ref_frac, out};
    hipLaunchKernelGGL(k_stream_scan, dim3(1), dim3(1024), 0, st, a);
    return hipGetLastError();
}

// Streams up to which the scan rides on the statistics launch (its one block of 256 threads then
// takes at most 16 streams a thread).
constexpr int kPrepScanMax = 4096;

hipError_t launch_prep_scan(const Geometry &g, const void *x, const int64_t *soff, const int64_t *woff, int n,
                            int div, int64_t *tile_off, float *mean, float *std, double *part, hipStream_t st)
{
    const int G = part ? stat_split(n, g.M) : 1;
    if (!mean)
        return launch_stream_scan(g, soff, woff, n, 0, div, tile_off, st);
    const ScanArgs a{soff, woff, n, 0, div, g.W, g.S, g.ref_frac, tile_off};
    if (n <= kPrepScanMax) {
        using Kernel = void (*)(ScanArgs, const void *, int, int, double *, float *, float *);
        const bool vec = stat_vec(g, x);
        const Kernel k = g.dtype == ENOVA_F32 ? (vec ? static_cast<Kernel>(k_prep<ENOVA_F32, 4>) : k_prep<ENOVA_F32, 1>)
                                              : (vec ? static_cast<Kernel>(k_prep<ENOVA_BF16, 4>) : k_prep<ENOVA_BF16, 1>);
        hipLaunchKernelGGL(k, dim3(static_cast<unsigned>(n) * G + 1), dim3(kStatThreads), 0, st, a, x, g.M, G, part,
                           mean, std);
        return hipGetLastError();
    }
    const hipError_t e = launch_stat_blocks(g, x, soff, n, G, part, mean, std, st);
    return e != hipSuccess ? e : launch_stream_scan(g, soff, woff, n, 0, div, tile_off, st);
}

hipError_t launch_prep_map(const Geometry &g, const void *x, const int64_t *soff, const int64_t *tile_off, int n,
                           int64_t grid, int *map, float *mean, float *std, const double *part, hipStream_t st)
{
    if (grid <= 0)
        return hipSuccess;
    StatFinish f{};
    int64_t items = grid;
    if (mean && part && stat_split(n, g.M) > 1) {
        f = StatFinish{part, x, soff, g.dtype, g.M, g.ref_frac, mean, std};
        items = std::max<int64_t>(items, static_cast<int64_t>(n) * g.M);
    }
    int64_t blocks = (items + 255) / 256;
    if (blocks > 65536)
        blocks = 65536;
    hipLaunchKernelGGL(k_tile_map, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, tile_off, n, grid, map, f);
    return hipGetLastError();
}

hipError_t launch_tile_map(const int64_t *tile_off, int n, int64_t grid, int *map, hipStream_t st)
{
    return launch_prep_map(Geometry{}, nullptr, nullptr, tile_off, n, grid, map, nullptr, nullptr, nullptr, st);
}

hipError_t launch_flag(const float *scores, int64_t n, float thr, uint8_t *flags, hipStream_t st)
{
    if (n <= 0)
        return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536)
        blocks = 65536;
    hipLaunchKernelGGL(k_flag, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, scores, n,
                       thr, flags);
    return hipGetLastError();
}

static unsigned cal_blocks(int64_t n_cal)
{
    return static_cast<unsigned>((n_cal + 256 * kCalItems - 1) / (256 * kCalItems));
}

hipError_t launch_radix_init(RadixState *rs, int64_t rank, unsigned int *hist, hipStream_t st)
{
    hipLaunchKernelGGL(k_radix_init, dim3(1), dim3(256), 0, st, rs, rank, hist);
    return hipGetLastError();
}

hipError_t launch_calib_hist(const float *scores, const int64_t *woff, const int64_t *cal_off,
                             int n, int64_t n_cal, int shift, RadixState *rs, unsigned int *hist,
                             hipStream_t st)
{
    if (n_cal <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_calib_hist, dim3(cal_blocks(n_cal)), dim3(256), 0, st, scores, woff,
                       cal_off, n, n_cal, shift, rs, hist);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_radix_pick, dim3(1), dim3(256), 0, st, rs, hist);
    return hipGetLastError();
}

int64_t calib_blocks(int64_t n_cal) { return (n_cal + 256 * kCalItems - 1) / (256 * kCalItems); }

hipError_t launch_calib_count(const float *scores, const int64_t *woff, const int64_t *cal_off, int n,
                              int64_t n_cal, uint32_t key, int64_t *block_counts, hipStream_t st)
{
    if (n_cal <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_calib_count, dim3(cal_blocks(n_cal)), dim3(256), 0, st, scores, woff,
                       cal_off, n, n_cal, key, block_counts);
    return hipGetLastError();
}

hipError_t launch_calib_compact(const float *scores, const int64_t *woff, const int64_t *cal_off,
                                int n, int64_t n_cal, uint32_t key, double t,
                                const int64_t *block_off, double *y, int64_t cap, hipStream_t st)
{
    if (n_cal <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_calib_compact, dim3(cal_blocks(n_cal)), dim3(256), 0, st, scores, woff,
                       cal_off, n, n_cal, key, t, block_off, y, cap);
    return hipGetLastError();
}

hipError_t launch_scan_i64(const int64_t *in, int64_t n, int64_t *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_scan_i64, dim3(1), dim3(1024), 0, st, in, n, out);
    return hipGetLastError();
}

// sa[i] = the chunk partials pa[i*nsplit + j] of point i added by one wave in a fixed order:
// lane l adds the chunks j = l, l + 64, ... in order, then a butterfly adds the lanes; likewise sb
// from pb. Four points per block.
__global__ __launch_bounds__(256) void k_gpd_reduce(const double *__restrict__ pa, const double *__restrict__ pb,
                                                    int nx, int nsplit, double *__restrict__ sa,
                                                    double *__restrict__ sb)
{
    const int i = blockIdx.x * 4 + static_cast<int>(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (i >= nx)
        return;
    const double *a = pa + static_cast<int64_t>(i) * nsplit, *b = pb + static_cast<int64_t>(i) * nsplit;
    double ta = 0.0, tb = 0.0;
    for (int j = lane; j < nsplit; j += 64) {
        ta += a[j];
        tb += b[j];
    }
    ta = wave_sum(ta);
    tb = wave_sum(tb);
    if (lane == 0) {
        sa[i] = ta;
        sb[i] = tb;
    }
}

hipError_t launch_gpd_reduce(const double *pa, const double *pb, int nx, int nsplit, double *sa, double *sb,
                             hipStream_t st)
{
    if (nx <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_gpd_reduce, dim3(static_cast<unsigned>((nx + 3) / 4)), dim3(256), 0, st, pa, pb, nx,
                       nsplit, sa, sb);
    return hipGetLastError();
}

int gpd_split(int64_t n, int nx)
{
    // about 2048 blocks in all (eight per compute unit: the fp64 division and log1p chains need
    // several waves per SIMD to hide their latency), and at least 1024 excesses per chunk
    const int64_t groups = (nx + kGpdX - 1) / kGpdX;
    int64_t s = (2048 + groups - 1) / (groups < 1 ? 1 : groups);
    const int64_t cap = n / 1024;
    if (s > cap)
        s = cap;
    return static_cast<int>(s < 1 ? 1 : s);
}

hipError_t launch_gpd_sums(const double *y, int64_t n, const double *xs, int nx, int nsplit,
                           double *pa, double *pb, double *pda, double *pdb, hipStream_t st)
{
    if (nx <= 0)
        return hipSuccess;
    if ((pda == nullptr) != (pdb == nullptr))
        return hipErrorInvalidValue;
    const unsigned groups = static_cast<unsigned>((nx + kGpdX - 1) / kGpdX);
    if (pda)
        hipLaunchKernelGGL(k_gpd_sums<true>, dim3(groups * nsplit), dim3(256), 0, st, y, n, xs, nx, nsplit, pa, pb,
                           pda, pdb);
    else
        hipLaunchKernelGGL(k_gpd_sums<false>, dim3(groups * nsplit), dim3(256), 0, st, y, n, xs, nx, nsplit, pa,
                           pb, pda, pdb);
    return hipGetLastError();
}

int peak_blocks(int64_t n)
{
    const int64_t b = (n + 8191) / 8192;
    return static_cast<int>(b < 1 ? 1 : (b > kPeakBlocks ? kPeakBlocks : b));
}

hipError_t launch_peak_stats(const double *y, int64_t n, double *out, double *work, hipStream_t st)
{
    const int nblk = peak_blocks(n);
    hipLaunchKernelGGL(k_peak_partial, dim3(nblk), dim3(256), 0, st, y, n, work);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_peak_final, dim3(1), dim3(64), 0, st, work, nblk, out);
    return hipGetLastError();
}

}  // namespace enova
