// Bandwidth-bound helper kernels: reference statistics, per-stream scans, tile maps and flags.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "block_scan.h"
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

// Single-block exclusive scan of the streams' tile counts (div windows a tile).
struct ScanArgs {
    const int64_t *soff, *woff;
    int n, div;
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
        return (g.woff[s + 1] - g.woff[s] + g.div - 1) / g.div;
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
                                                  int *__restrict__ map, unsigned *__restrict__ marks, StatFinish f)
{
    const int64_t first = blockIdx.x * 256LL + threadIdx.x, step = static_cast<int64_t>(gridDim.x) * 256;
    if (marks && first == 0)
        *marks = 0u;
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
                              int div, int64_t *out, hipStream_t st)
{
    const ScanArgs a{soff, woff, n, div, g.ref_frac, out};
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
        return launch_stream_scan(g, soff, woff, n, div, tile_off, st);
    const ScanArgs a{soff, woff, n, div, g.ref_frac, tile_off};
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
    return e != hipSuccess ? e : launch_stream_scan(g, soff, woff, n, div, tile_off, st);
}

hipError_t launch_prep_map(const Geometry &g, const void *x, const int64_t *soff, const int64_t *tile_off, int n,
                           int64_t grid, int *map, unsigned *marks, float *mean, float *std, const double *part,
                           hipStream_t st)
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
    hipLaunchKernelGGL(k_tile_map, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, tile_off, n, grid, map, marks,
                       f);
    return hipGetLastError();
}

hipError_t launch_tile_map(const int64_t *tile_off, int n, int64_t grid, int *map, hipStream_t st)
{
    return launch_prep_map(Geometry{}, nullptr, nullptr, tile_off, n, grid, map, nullptr, nullptr, nullptr, nullptr,
                           st);
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

}  // namespace enova
