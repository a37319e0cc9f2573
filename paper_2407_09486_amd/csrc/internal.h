// Internal declarations of libenova_detect: kernel parameter blocks and launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <cstddef>
#include <cstdint>

#include "enova_detect.h"

namespace enova {

// ---------------------------------------------------------------------------------------------
// Geometry of the matrix-core path.
//
// The window of W steps x M metrics is cut into Q = ceil(W/S) "super-rows" of S consecutive
// steps (S*Mp elements, Mp = M padded so a super-row is a whole number of 16-byte chunks).
// Window k of a stream consists of super-rows k .. k+Q-1 of that stream, so a tile of Nb
// consecutive windows needs only Nb+Q-1 super-rows staged in LDS: every staged element is
// normalised once and then read by up to Q windows (implicit im2col of a strided 1-D
// convolution). The reduction index is walked chunk by chunk: chunk kappa = q*CPR + c is
// 16-byte chunk c of the window's super-row q.
// ---------------------------------------------------------------------------------------------
struct Geometry {
    int M, W, S, H, L, D;   // true sizes
    int dtype, act;
    float ref_frac;
    int epc;                // elements per 16-byte chunk: 4 (f32) or 8 (bf16)
    int Mp;                 // metrics padded so that S*Mp % epc == 0
    int Q;                  // super-rows per window
    int CPR;                // chunks per super-row
    int CPRP;               // LDS row pitch in chunks (odd, so 16 consecutive rows hit distinct banks)
    int KC;                 // chunks per window, rounded up to a multiple of 2*kPrefetchSteps
    int spare;              // staged super-rows after a tile's last window's Q - 1
    int Hp;                 // hidden width padded to 32*HB
    int HB;                 // 32-row hidden blocks of the tile (Hp = 32*HB)
    int HBW;                // hidden blocks per wave
    int NBW;                // 32-window blocks per wave
    int WH;                 // waves along the hidden rows (NW/WH along the windows)
    int NW;                 // waves per block of the matrix-core kernel (4 or 8)
    bool cl;                // epilogue weights staged in LDS (else read from L2)
    int Nb;                 // windows per tile
    size_t lds_bytes;       // dynamic LDS of the matrix-core kernel
    bool mfma_ok;
    // bf16 detectors with 193..256 hidden units take the ring kernel (k_score_ring.hip) instead:
    // 128-window tiles, a ring of RR super-rows of RP chunks in LDS, two blocks per compute unit
    bool ring;
    int RP, RR;
    int ring_floats;        // floats of the ring region (at least the epilogue's 64 KiB exchange)
    size_t ring_lds;        // dynamic LDS of the ring kernel
};

constexpr int kRingNb = 128;        // windows per tile of the ring kernel
constexpr int kRingWaves = 4;       // waves per block: 64 hidden rows each
constexpr int kRingHidden = 256;    // hidden units the ring kernel is laid out for (padded)
// dynamic LDS of the ring kernel for ring slots of P chunks, Q super-rows per window
size_t ring_lds_bytes(int P, int Q, int ring_floats);

constexpr int kWaves = 4;                 // waves per block of the other kernels
constexpr int kThreads = 64 * kWaves;
constexpr size_t kLdsLimit = 160 * 1024;
// The reduction index is padded to a multiple of 2*kPrefetchSteps chunks (the matrix-core
// kernel's deepest W1 prefetch ring, in two-chunk steps); the packed W1 carries kPrefetchSteps
// zero steps after the last one, and Geometry::spare staged super-rows follow a tile's windows
// (enough for the padded chunks and kPrefetchRows steps of window-fragment prefetch), so every
// prefetch past the last step reads valid memory.
constexpr int kPrefetchSteps = 8;
constexpr int kPrefetchRows = 2;

// Fixed device scratch of the allocation-free scoring entry point: kScratchBytes per device.
// scratch_setup returns this device's copy (device must be current); the lookup happens once per
// device and is then cached.
constexpr size_t kScratchBytes = size_t{16} << 20;
hipError_t scratch_setup(int device, void **out);

// Error reporting of the C entry points: records the message returned by enova_last_error().
enova_status fail(enova_status st, const char *fmt, ...);
enova_status hip_fail(hipError_t e, const char *what);

// Keeps the caller's current device and switches to another for a call's duration.
struct DeviceGuard {
    int prev = -1;
    bool ok = false;
    explicit DeviceGuard(int dev)
    {
        if (hipGetDevice(&prev) != hipSuccess)
            return;
        ok = prev == dev || hipSetDevice(dev) == hipSuccess;
    }
    ~DeviceGuard()
    {
        if (ok && prev >= 0)
            (void)hipSetDevice(prev);
    }
};

bool plan_geometry(const enova_detect_config &cfg, Geometry *g);
// Wave layout of the matrix-core kernel for dtype and hb 32-row hidden blocks: hidden blocks and
// 32-window blocks per wave, waves along the hidden rows, waves per block.
void mfma_layout(int dtype, int hb, int *hbw, int *nbw, int *wh, int *nw);
// Lets the instantiation chosen for g use the full LDS of a compute unit.
hipError_t prepare_score_mfma(const Geometry &g);

// Parameter block of the scoring kernels (passed by value).
struct ScoreParams {
    const void *x;
    const int64_t *soff;
    const int64_t *woff;
    const int64_t *tile_off;     // matrix-core kernel only: first tile of each stream
    const int *tile_stream;      // matrix-core kernel only: stream of each block (-1: none)
    // split kernel: the tiles with windows it leaves to the fp32 kernel, marks[0] of them (cleared with
    // the tile map), each as tile << 4 | parts of kListNb windows that hold some
    unsigned *marks;
    int n_streams;
    int64_t n_windows;
    const float *mean;
    const float *std;
    // matrix-core packed weights
    const uint4 *w1p;            // [KC/2][HB][64 lanes] 16-byte A fragments
    const float *whp;            // [HB][16][64] heads (mu rows 0..15, log-var rows 16..31)
    const float *wd1p;           // [HB][8][64]  decoder hidden layer
    // vector-kernel weights
    const void *w1t;             // [D][H] transposed W1 (float or bf16 bits)
    const float *wmu, *wlv, *wd1;
    // shared small vectors (padded to Hp / 32)
    const float *b1;             // [Hp]
    const float *bh;             // [32]: bmu (padded to 16), blv (padded to 16)
    const float *bmu, *blv;      // [L]
    const float *bd1;            // [Hp]
    const float *u;              // [Hp] column sums of Wd2
    // ring kernel: W1 as 16x16x32 A fragments [steps + kPrefetchSteps][16][64 lanes], the heads as
    // bf16 hi/lo fragments [wave][2][2][hi, lo][64], the decoder hidden layer [16][hi, lo][64]
    const uint4 *w1r;
    const uint4 *whr;
    const uint2 *wdr;
    // split kernel: W1 as f16 hi/lo 32x32x16 A fragments [steps + 2][HB][hi, lo][64 lanes], the heads
    // [HB][2][3][64] and the decoder hidden layer [HB][3][64] as bf16 parts, and each hidden row's
    // accumulator scale [Hp]
    const uint4 *w1x;
    const uint4 *whx;
    const uint4 *wdx;
    const float *w1scale;
    float sum_bd2;
    float threshold;
    int write_flags;
    float *scores;
    float *md;
    uint8_t *flags;
};

// Geometry of the split-precision kernel (k_score_split.hip; fp32 detectors): super-rows of 8-element
// chunks, each as an f16 hi and lo chunk in LDS; a large and a small tile of windows.
struct SplitGeometry {
    bool ok = false;
    int Mp = 0, Q = 0, CPR = 0, P = 0, nsteps = 0, spare = 0;
    int nb_small = 0, nb_large = 0;
    size_t lds_small = 0, lds_large = 0;
    int nb(int64_t n_windows, int n_streams) const
    {
        // the large tile once it gives two blocks to every compute unit and the streams fill it
        // at least by half (the padding of a stream's last tile is computed)
        const bool large = n_windows >= 512LL * nb_large && n_windows >= static_cast<int64_t>(n_streams) * (nb_large / 2);
        return large ? nb_large : nb_small;
    }
};
constexpr int kSplitPrefetch = 2;   // zero steps after the last one in w1x

// Launchers (return the launch error).
SplitGeometry plan_split(const Geometry &g);
hipError_t prepare_score_split(const Geometry &g, const SplitGeometry &sg);
hipError_t launch_score_split(const Geometry &g, const SplitGeometry &sg, const ScoreParams &p, int nb, int64_t grid,
                              hipStream_t st);
// The fp32 kernel over the tiles (of nb windows) that the split kernel marked, writing only their
// windows outside the split's range; score_list_lds is its dynamic LDS. A mark holds four parts of
// kListNb windows and a tile index below kMaxMarked.
constexpr int kListNb = 128;
constexpr int64_t kMaxMarked = 1LL << 28;
size_t score_list_lds(const Geometry &g);
hipError_t prepare_score_list(const Geometry &g);
hipError_t launch_score_list(const Geometry &g, const ScoreParams &p, int nb, int64_t grid, hipStream_t st);
// part: stat_part_bytes(n, M) bytes for chunk sums (then about 2048 blocks share the streams), or
// NULL (one block per stream); the statistics are bit for bit the same.
size_t stat_part_bytes(int n, int M);
hipError_t launch_ref_stats(const Geometry &g, const void *x, const int64_t *soff, int n,
                            float *mean, float *std, double *part, hipStream_t st);
// The two launches that head a scoring pass: the tiles' scan (launch_stream_scan) with the
// reference statistics unless mean is NULL, then the tile map with the statistics' last step and the
// cleared count of marks (NULL: none).
hipError_t launch_prep_scan(const Geometry &g, const void *x, const int64_t *soff, const int64_t *woff, int n,
                            int div, int64_t *tile_off, float *mean, float *std, double *part, hipStream_t st);
hipError_t launch_prep_map(const Geometry &g, const void *x, const int64_t *soff, const int64_t *tile_off, int n,
                           int64_t grid, int *map, unsigned *marks, float *mean, float *std, const double *part,
                           hipStream_t st);
// out[s] = sum_{r<s} ceil(windows of stream r / div), n+1 entries.
hipError_t launch_stream_scan(const Geometry &g, const int64_t *soff, const int64_t *woff, int n,
                              int div, int64_t *out, hipStream_t st);
// map[b] = the stream whose tiles include tile b (tile_off has n+1 entries), -1 for
// tile_off[n] <= b < grid.
hipError_t launch_tile_map(const int64_t *tile_off, int n, int64_t grid, int *map, hipStream_t st);
hipError_t launch_score_valu(const Geometry &g, const ScoreParams &p, hipStream_t st);
hipError_t launch_score_mfma(const Geometry &g, const ScoreParams &p, int64_t grid, hipStream_t st);
hipError_t prepare_score_ring(const Geometry &g);
hipError_t launch_score_ring(const Geometry &g, const ScoreParams &p, int64_t grid, hipStream_t st);
hipError_t launch_flag(const float *scores, int64_t n, float thr, uint8_t *flags, hipStream_t st);

}  // namespace enova
