// Internal declarations of the peaks-over-threshold calibration (k_pot.hip).
#pragma once

#include "internal.h"

namespace enova {

constexpr int kPotPasses = 4;          // 8-bit digits of a float key
constexpr int kPotGridPoints = 512;    // grid points per admissible interval
constexpr int kPotRounds = 64;         // evaluations per bracket at most
constexpr int kPotStatBlocks = 256;
constexpr int kPotX = 8;               // points that an excess is loaded for
// Chunk sums of an evaluation: at most 4 sums of (2048 + groups) x kPotX (chunk, point) pairs, the
// points in at most 2 kPotGridPoints / kPotX groups.
constexpr int64_t kPotPartDoubles = 4LL * (2048 + 2 * kPotGridPoints / kPotX) * kPotX;

// The radix select: the key prefix chosen so far, the rank still sought among the keys that share
// it, the count of keys above it; lost if a pass did not hold the rank.
struct PotSelect {
    uint32_t prefix;
    int32_t lost;
    int64_t rank, n_greater;
};

struct PotBracket {
    double lo, hi, wlo, whi;   // w at the ends (an end kept twice in a row has its w halved: Illinois)
    double x, root;            // the point evaluated next; the root once done
    int lo_neg, done, side, evals;
};

enum { kPotGrid = 0, kPotNewton = 1, kPotLast = 2, kPotDone = 3 };
enum { kPotNoWindows = 1, kPotLost = 2, kPotLevelNotFinite = 3, kPotCount = 4, kPotNotFinite = 5 };

// Everything the launches of one call leave for the next one (device memory).
struct PotState {
    int err, phase, method, npts, n_roots, n_br;
    int64_t n_cal, n_peaks;
    double t, ysum, z, gamma, sigma;
    PotSelect sel[kPotPasses + 1];
    unsigned hist[kPotPasses][256];
    double part[3][kPotStatBlocks];
    // a sign change needs two points of one grid, so at most one root or bracket per point
    double xs[2 * kPotGridPoints], sum[4][2 * kPotGridPoints], roots[2 * kPotGridPoints];
    int owner[2 * kPotGridPoints];
    PotBracket br[2 * kPotGridPoints];
};

// What the host reads at the end.
struct PotOut {
    int err, phase, method, pad;
    int64_t n_cal, n_peaks;
    double t, z, gamma, sigma;
};

struct PotWork {
    PotState *state;
    int64_t *cal;                  // [n + 1]
    int64_t *counts, *offsets;     // [pot_blocks] each
    double *y;                     // [cap] excesses
    double *part;                  // [kPotPartDoubles]
    int64_t cap;
};

int64_t pot_blocks(int64_t n_windows);
// The calibration set and its level quantile's key; the excesses, their statistics and the fit's
// start (the whole fit below ten peaks); `rounds` pairs of an evaluation and a step of the fit; the
// result and, with flags, score > threshold once the fit has ended without an error.
hipError_t launch_pot_select(const Geometry &g, const float *scores, const int64_t *soff, const int64_t *woff, int n,
                             int64_t n_windows, double level, const PotWork &w, hipStream_t st);
hipError_t launch_pot_peaks(const float *scores, const int64_t *woff, int n, int64_t n_windows, double q,
                            const PotWork &w, hipStream_t st);
hipError_t launch_pot_rounds(int rounds, double q, const PotWork &w, hipStream_t st);
hipError_t launch_pot_flag(const float *scores, int64_t n_windows, const PotWork &w, PotOut *out, uint8_t *flags,
                           hipStream_t st);

}  // namespace enova
