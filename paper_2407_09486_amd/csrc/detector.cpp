// Host side of libenova_detect: argument validation, weight repacking, workspace management
// and kernel launches behind the C ABI of include/enova_detect.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "enova_detect.h"
#include "internal.h"
#include "pot_internal.h"
#include "stream_internal.h"
#include "variants_internal.h"

namespace {
thread_local std::string g_last_error;
}  // namespace

namespace enova {

enova_status fail(enova_status st, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return st;
}

enova_status hip_fail(hipError_t e, const char *what)
{
    return fail(ENOVA_EHIP, "%s: %s", what, hipGetErrorString(e));
}

}  // namespace enova

using namespace enova;

namespace {

float bf16_bits_to_float(uint16_t b)
{
    uint32_t u = static_cast<uint32_t>(b) << 16;
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}

// Round to nearest even; a NaN stays a (quiet) NaN.
uint16_t float_to_bf16_bits(float f)
{
    uint32_t u;
    std::memcpy(&u, &f, sizeof(u));
    if ((u & 0x7fffffffu) > 0x7f800000u)
        return static_cast<uint16_t>((u >> 16) | 0x0040u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}

}  // namespace

struct enova_detector_s {
    Geometry g{};
    int device = 0;
    int kind = 1;                 // 1 vector-ALU, 2 matrix-core
    // weights (in few allocations)
    std::vector<void *> weights;
    const uint4 *w1p = nullptr;   // matrix-core A fragments
    // ring kernel: W1, heads and decoder fragments
    const uint4 *w1r = nullptr, *whr = nullptr;
    const uint2 *wdr = nullptr;
    SplitGeometry sg;             // split kernel (fp32 detectors): its tiles and fragments
    const uint4 *w1x = nullptr, *whx = nullptr, *wdx = nullptr;
    const float *w1scale = nullptr;
    const uint4 *w1s = nullptr;   // streaming kernel: W1, heads and decoder fragments
    const float *whs = nullptr, *wds = nullptr;
    const uint4 *wd2x = nullptr;  // split variant pass: Wd2's f16 parts and the padded bd2
    const float *bd2x = nullptr;
    float wd2_unscale = 1.0f;
    const float4 *wd2p = nullptr; // fused variant pass: decoder-output fragments of Wd2
    const void *w1t = nullptr;    // [D][H] transposed W1
    float *small = nullptr;       // every small weight array
    float *b1 = nullptr, *bh = nullptr, *bmu = nullptr, *blv = nullptr, *wmu = nullptr,
          *wlv = nullptr, *wd1 = nullptr, *bd1 = nullptr, *u = nullptr, *whp = nullptr,
          *wd1p = nullptr;
    float sum_bd2 = 0.0f;
    // workspace
    float *stats = nullptr;
    size_t stats_cap = 0;         // floats
    int64_t *tiles = nullptr;
    size_t tiles_cap = 0;         // entries
    int *tile_map = nullptr;      // stream of each matrix-core block, and the split kernel's marks
    size_t tile_map_cap = 0;      // entries
    int64_t *cal = nullptr;
    size_t cal_cap = 0;
    PotState *pot = nullptr;      // the threshold call's state, and the sums of its fit's chunks
    double *pot_part = nullptr;
    size_t pot_part_cap = 0;
    double *peaks = nullptr;      // excesses over the level quantile, calibration order
    size_t peaks_cap = 0;
    int64_t *blk = nullptr;       // per-block peak counts, then their exclusive scan
    size_t blk_cap = 0;
    PotOut *pot_out = nullptr;    // its result (pinned host memory)
    // this device's fixed scratch (kScratchBytes, shared by every detector on the device), the
    // only workspace of enova_detect_score_noalloc
    void *scratch = nullptr;
    // dense fp32 weights of the output variants: W1 [H][D], [Wmu; Wlv] [2L][H], [bmu | blv] [2L],
    // Wd1 [H][L], Wd2 [D][H], bd2 [D]
    float *d_w1 = nullptr, *d_wml = nullptr, *d_bml = nullptr, *d_wd1 = nullptr, *d_wd2 = nullptr,
          *d_bd2 = nullptr;
    // workspace of the output variants (one chunk of windows; the fused pass's tile scan and map)
    float *ext_ws = nullptr;
    size_t ext_ws_cap = 0;        // floats
    // timing
    bool timing = false;
    hipEvent_t ev[4] = {nullptr, nullptr, nullptr, nullptr};
    hipEvent_t ext_ev[2] = {nullptr, nullptr};
    bool ran_stats = false, ran_score = false, ran_ext = false;
};

namespace enova {

bool plan_geometry(const enova_detect_config &cfg, Geometry *g)
{
    g->M = cfg.metrics;
    g->W = cfg.window;
    g->S = cfg.stride;
    g->H = cfg.hidden;
    g->L = cfg.latent;
    g->D = cfg.window * cfg.metrics;
    g->dtype = cfg.dtype;
    g->act = cfg.act;
    g->ref_frac = cfg.ref_frac;
    g->epc = cfg.dtype == ENOVA_F32 ? 4 : 8;
    int mp = g->M;
    while ((static_cast<int64_t>(g->S) * mp) % g->epc)
        ++mp;
    g->Mp = mp;
    g->Q = (g->W + g->S - 1) / g->S;
    const int64_t cpr = static_cast<int64_t>(g->S) * g->Mp / g->epc;
    g->CPR = static_cast<int>(cpr);
    g->CPRP = (g->CPR % 2 == 0) ? g->CPR + 1 : g->CPR;
    int64_t kc = static_cast<int64_t>(g->Q) * g->CPR;
    kc = (kc + 2 * kPrefetchSteps - 1) / (2 * kPrefetchSteps) * (2 * kPrefetchSteps);
    g->KC = static_cast<int>(kc);
    // the furthest chunk a window fragment prefetch reads: kPrefetchRows steps past the last
    const int64_t kmax = kc + 2 * kPrefetchRows - 1;
    g->spare = static_cast<int>(kmax / g->CPR - g->Q + 2);
    int hb = 1;
    while (hb < 8 && 32 * hb < g->H)
        hb *= 2;
    g->HB = hb;
    g->Hp = 32 * hb;
    mfma_layout(g->dtype, hb, &g->HBW, &g->NBW, &g->WH, &g->NW);
    g->Nb = (g->NW / g->WH) * g->NBW * 32;
    // epilogue weights (heads, decoder hidden layer, b1, bd1, u, head biases), the segment, its
    // row sums and the stream statistics
    const size_t n_const = static_cast<size_t>(hb) * (16 * 64 + 8 * 64) + 3 * static_cast<size_t>(g->Hp) + 32;
    // with several waves along the hidden rows, the segment's space later holds the exchange of
    // head and decoder partial sums
    const size_t rows = static_cast<size_t>(g->Nb + g->Q - 1 + g->spare);
    const size_t seg_bytes = rows * g->CPRP * 16;
    const size_t xchg_bytes = g->WH > 1 ? static_cast<size_t>(g->NW) * std::min(g->NBW, 2) * 17 * 64 * sizeof(float) : 0;
    // the split bf16 layout keeps its epilogue weights in L2 to leave LDS to a 256-window tile
    g->cl = g->WH == 1;
    // (without the copied block, b1, bd1, u and the head biases still get LDS of their own)
    const size_t n_small = 3 * static_cast<size_t>(g->Hp) + 32;
    g->lds_bytes = (g->cl ? n_const : n_small) * sizeof(float) + std::max(seg_bytes, xchg_bytes) +
                   rows * 2 * sizeof(float) + 3 * sizeof(float) * static_cast<size_t>(g->S) * g->Mp;
    g->mfma_ok = g->H <= 256 && g->L <= 16 && cpr < (1 << 20) && kc < (1 << 24) &&
                 g->lds_bytes <= kLdsLimit;
    // bf16 with 193..256 hidden units: the ring kernel when a block fits half a compute unit's LDS
    // (a ring slot is one super-row of at most 64 chunks, i.e. one chunk per lane of a wave)
    g->ring = false;
    g->RP = g->RR = g->ring_floats = 0;
    g->ring_lds = 0;
    if (g->mfma_ok && g->dtype == ENOVA_BF16 && g->H > 192 && g->H <= kRingHidden && g->L <= 16) {
        const int P = (g->CPR + 15) / 16 * 16;   // whole groups of four 4-chunk reduction steps
        const int R = (kRingNb + 2 + 7) / 8 * 8;
        const int64_t ring_f = std::max<int64_t>(static_cast<int64_t>(R) * P * 4,
                                                 static_cast<int64_t>(kRingWaves) * 2 * (kRingNb / 16) * 4 * 64);
        if (P <= 64) {
            const size_t lds = ring_lds_bytes(P, g->Q, static_cast<int>(ring_f));
            if (lds <= kLdsLimit / 2) {
                g->ring = true;
                g->RP = P;
                g->RR = R;
                g->ring_floats = static_cast<int>(ring_f);
                g->ring_lds = lds;
                g->Nb = kRingNb;
            }
        }
    }
    if (!g->mfma_ok) {
        g->Hp = ((g->H + 31) / 32) * 32;
    }
    return g->mfma_ok;
}

}  // namespace enova

namespace {

// Arrays that are packed on the host and then go to the device together: small ones share an allocation
// and a copy (each on its own took some 10 us, a third of a small detector's set-up). Large ones have
// theirs: 4 MB in one allocation took 80 us to free.
class Uploads {
public:
    ~Uploads()
    {
        for (const Part &q : parts_)
            std::free(q.host);
    }
    // n zeroed elements to fill; *dst is their device address once upload() has succeeded
    template <typename T, typename P>
    T *add(P **dst, size_t n)
    {
        const size_t bytes = (std::max<size_t>(n, 1) * sizeof(T) + 255) / 256 * 256;
        parts_.push_back(Part{dst, std::calloc(1, bytes), bytes});
        if (!parts_.back().host)
            throw std::bad_alloc();
        return static_cast<T *>(parts_.back().host);
    }
    enova_status upload(std::vector<void *> &owned)
    {
        std::stable_partition(parts_.begin(), parts_.end(), [](const Part &q) { return q.bytes <= kTogether; });
        std::vector<unsigned char> run;
        for (size_t i = 0; i < parts_.size();) {
            // small parts up to four times kTogether, or one large one
            size_t n = i, bytes = 0;
            run.clear();
            do {
                const Part &q = parts_[n++];
                const unsigned char *host = static_cast<const unsigned char *>(q.host);
                if (q.bytes <= kTogether)
                    run.insert(run.end(), host, host + q.bytes);
                bytes += q.bytes;
            } while (n < parts_.size() && parts_[n].bytes <= kTogether && bytes + parts_[n].bytes <= 4 * kTogether);
            owned.push_back(nullptr);
            hipError_t e = hipMalloc(&owned.back(), bytes);
            if (e != hipSuccess) {
                owned.pop_back();
                return fail(ENOVA_ENOMEM, "hipMalloc(%zu): %s", bytes, hipGetErrorString(e));
            }
            e = hipMemcpy(owned.back(), run.empty() ? parts_[i].host : run.data(), bytes, hipMemcpyHostToDevice);
            if (e != hipSuccess)
                return hip_fail(e, "hipMemcpy weights");
            for (unsigned char *at = static_cast<unsigned char *>(owned.back()); i < n; ++i) {
                std::memcpy(parts_[i].dst, &at, sizeof(at));
                at += parts_[i].bytes;
            }
        }
        return ENOVA_OK;
    }

private:
    static constexpr size_t kTogether = 128 << 10;
    struct Part {
        void *dst;     // the pointer to set
        void *host;
        size_t bytes;
    };
    std::vector<Part> parts_;
};

template <typename T>
enova_status ensure(T **buf, size_t *cap, size_t need)
{
    if (need <= *cap && *buf)
        return ENOVA_OK;
    if (*buf) {
        (void)hipFree(*buf);
        *buf = nullptr;
        *cap = 0;
    }
    size_t n = std::max<size_t>(need, 64);
    hipError_t e = hipMalloc(reinterpret_cast<void **>(buf), n * sizeof(T));
    if (e != hipSuccess)
        return fail(ENOVA_ENOMEM, "workspace hipMalloc(%zu): %s", n * sizeof(T), hipGetErrorString(e));
    *cap = n;
    return ENOVA_OK;
}

// Eight values as two f16 each, hi the nearest (ties to even; |v| below 65520) and lo the nearest to what is
// left. Written without branches, for the compiler to take four at a time.
inline uint32_t nearest_f16(float f, float *value)
{
    uint32_t u;
    std::memcpy(&u, &f, sizeof(u));
    const uint32_t sign = u & 0x80000000u, a = u ^ sign;
    // from 2^-14 on: the mantissa rounded to 10 bits; below: a multiple of 2^-24, the last place of 0.5 to 1
    const uint32_t r = (a + 0xfffu + ((a >> 13) & 1u)) & ~0x1fffu;
    float m;
    std::memcpy(&m, &a, sizeof(m));
    const bool normal = a >= 0x38800000u;
    const float low = ((normal ? 0.0f : m) + 0.75f) - 0.75f;
    float big;
    std::memcpy(&big, &r, sizeof(big));
    const float v = normal ? big : low;
    const uint32_t bits = normal ? (r - 0x38000000u) >> 13 : static_cast<uint32_t>(static_cast<int32_t>(low * 0x1p24f));
    uint32_t q;
    std::memcpy(&q, &v, sizeof(q));
    q |= sign;
    std::memcpy(value, &q, sizeof(q));
    return bits | sign >> 16;
}

inline void f16_parts(const float (&v)[8], uint16_t *hi, uint16_t *lo)
{
    uint32_t h[8], l[8];
    for (int e = 0; e < 8; ++e) {
        float a, b;
        h[e] = nearest_f16(v[e], &a);
        l[e] = nearest_f16(v[e] - a, &b);
    }
    for (int e = 0; e < 8; ++e) {
        hi[e] = static_cast<uint16_t>(h[e]);
        lo[e] = static_cast<uint16_t>(l[e]);
    }
}

// fn(src, kappa, e) for every weight src = t * M + m of a W1 row in the chunk order of super-rows of
// cpr chunks of epc elements (mp elements a step): element e of chunk kappa.
template <typename F>
void for_row(const Geometry &g, int mp, int cpr, int epc, F fn)
{
    const int sh = epc == 8 ? 3 : 2;
    for (int t = 0, q = 0, ts = 0; t < g.W; ++t) {
        for (int m = 0; m < g.M; ++m) {
            const int el = ts * mp + m;
            fn(t * g.M + m, q * cpr + (el >> sh), el & (epc - 1));
        }
        if (++ts == g.S) {
            ts = 0;
            ++q;
        }
    }
}

// W1's row h in the chunk order of g: at(kappa) is where the 16 bytes of chunk kappa go (without padded
// metrics the row's elements as they come).
template <typename F>
void pack_row(const Geometry &g, const void *w1, int h, F at)
{
    const size_t esz = g.dtype == ENOVA_BF16 ? 2 : 4;
    const unsigned char *row = static_cast<const unsigned char *>(w1) + static_cast<size_t>(h) * g.D * esz;
    if (g.Mp == g.M)
        for (int j = 0, kappa = 0; j < g.D; j += g.epc, ++kappa)
            std::memcpy(at(kappa), row + j * esz, std::min(g.epc, g.D - j) * esz);
    else
        for_row(g, g.Mp, g.CPR, g.epc, [&](int j, int kappa, int e) {
            std::memcpy(reinterpret_cast<unsigned char *>(at(kappa)) + e * esz, row + j * esz, esz);
        });
}

// Fragments of the ring kernel (bf16 detectors with 193..256 hidden units):
//  W1      step i = q * KS + sp (KS = P / 4), hidden block hb (16 rows), lane l: the 8 bf16 of
//          W1[16 hb + l % 16] at the elements of chunk 4 sp + l / 16 of super-row q (zero past the
//          window, the hidden width or the super-row's chunks); kPrefetchSteps zero steps follow.
//  heads   [wave w][m][zb][hi, lo][lane l] 8 bf16: row l % 16 of Wmu (zb = 0) or Wlv (zb = 1), zero
//          past L, at hidden rows 16 (4w + 2m) + 4 (l / 16) + t (t < 4) and
//          16 (4w + 2m + 1) + 4 (l / 16) + t - 4 (t >= 4) -- the accumulator rows the lane holds.
//  decoder [hidden block hb][hi, lo][lane l] 4 bf16: Wd1[16 hb + l % 16][4 (l / 16) + t].
// Weights of the heads and the decoder are split into bf16 hi + lo (the remainder rounded).
hipError_t pack_ring(enova_detector d, const enova_detect_weights *w, Uploads &up)
{
    const Geometry &g = d->g;
    const int H = g.H, L = g.L, D = g.D;
    const int KS = g.RP / 4, NS = g.Q * KS;
    constexpr int HBT = kRingHidden / 16;
    const size_t n_w1 = static_cast<size_t>(NS + kPrefetchSteps) * HBT * 64;   // 16-byte fragments
    const size_t n_wh = static_cast<size_t>(kRingWaves) * 2 * 2 * 2 * 64;       // 16-byte fragments
    const size_t n_wd = static_cast<size_t>(HBT) * 2 * 64;                      // 8-byte fragments
    uint16_t *w1r = up.add<uint16_t>(&d->w1r, n_w1 * 8), *whr = up.add<uint16_t>(&d->whr, n_wh * 8),
             *wdr = up.add<uint16_t>(&d->wdr, n_wd * 4);
    const uint16_t *w1 = static_cast<const uint16_t *>(w->w1);
    for (int i = 0; i < NS; ++i) {
        const int q = i / KS, sp = i - q * KS;
        for (int hb = 0; hb < HBT; ++hb)
            for (int lane = 0; lane < 64; ++lane) {
                const int h = 16 * hb + (lane & 15);
                const int c = 4 * sp + (lane >> 4);
                if (h >= H || c >= g.CPR)
                    continue;
                uint16_t *dst = w1r + ((static_cast<size_t>(i) * HBT + hb) * 64 + lane) * 8;
                for (int e = 0; e < 8; ++e) {
                    const int jj = c * 8 + e;
                    const int tt = jj / g.Mp, m = jj - (jj / g.Mp) * g.Mp;
                    const int t = q * g.S + tt;
                    if (t < g.W && m < g.M)
                        dst[e] = w1[static_cast<int64_t>(h) * D + static_cast<int64_t>(t) * g.M + m];
                }
            }
    }
    auto split = [](float v, uint16_t &hi, uint16_t &lo) {
        hi = float_to_bf16_bits(v);
        lo = float_to_bf16_bits(v - bf16_bits_to_float(hi));
    };
    for (int wv = 0; wv < kRingWaves; ++wv)
        for (int m = 0; m < 2; ++m)
            for (int zb = 0; zb < 2; ++zb) {
                const size_t base = (((static_cast<size_t>(wv) * 2 + m) * 2 + zb) * 2) * 64;
                for (int lane = 0; lane < 64; ++lane) {
                    const int row = lane & 15, grp = lane >> 4;
                    for (int t = 0; t < 8; ++t) {
                        const int h = t < 4 ? 16 * (4 * wv + 2 * m) + 4 * grp + t
                                            : 16 * (4 * wv + 2 * m + 1) + 4 * grp + (t - 4);
                        float v = 0.0f;
                        if (h < H && row < L)
                            v = zb == 0 ? w->wmu[row * H + h] : w->wlv[row * H + h];
                        uint16_t hi, lo;
                        split(v, hi, lo);
                        whr[(base + lane) * 8 + t] = hi;
                        whr[(base + 64 + lane) * 8 + t] = lo;
                    }
                }
            }
    for (int hb = 0; hb < HBT; ++hb)
        for (int lane = 0; lane < 64; ++lane)
            for (int t = 0; t < 4; ++t) {
                const int h = 16 * hb + (lane & 15);
                const int l = 4 * (lane >> 4) + t;
                float v = 0.0f;
                if (h < H && l < L)
                    v = w->wd1[h * L + l];
                uint16_t hi, lo;
                split(v, hi, lo);
                wdr[((static_cast<size_t>(hb) * 2 + 0) * 64 + lane) * 4 + t] = hi;
                wdr[((static_cast<size_t>(hb) * 2 + 1) * 64 + lane) * 4 + t] = lo;
            }
    return prepare_score_ring(g);
}

// Fragments of the streaming kernel's 16x16 matrix ops: W1 as A fragments
// [stream_w1_steps][Hp/16][64 lanes] x 16 bytes (lane l: hidden row 16 hb + l%16, chunk
// 4 step + l/16 in the detector's chunk order, zeros past the window), the heads as
// [Hp/16][4][2][64] floats (op (hb, r) of head 0 = mean, 1 = log-variance: lane l holds the head
// row l%16 at hidden unit 16 hb + 4 (l/16) + r) and the decoder's hidden layer as [Hp/16][4][64]
// floats (op (hb, r): lane l holds Wd1[16 hb + l%16][4 (l/16) + r]).
hipError_t pack_stream(enova_detector d, const enova_detect_weights *w, Uploads &up)
{
    const Geometry &g = d->g;
    const int H = g.H, L = g.L, D = g.D, NHB = g.Hp / 16;
    const bool bf = g.dtype == ENOVA_BF16;
    const int steps = stream_w1_steps(g);
    const size_t n_w1 = static_cast<size_t>(steps) * NHB * 64;   // 16-byte fragments
    const size_t n_wh = static_cast<size_t>(NHB) * 4 * 2 * 64;   // floats
    const size_t n_wd = static_cast<size_t>(NHB) * 4 * 64;       // floats
    uint32_t *buf = up.add<uint32_t>(&d->w1s, n_w1 * 4);
    float *wh = up.add<float>(&d->whs, n_wh), *wd = up.add<float>(&d->wds, n_wd);
    for (int h = 0; h < H; ++h) {
        uint32_t *dst = buf + (static_cast<size_t>(h >> 4) * 64 + (h & 15)) * 4;
        pack_row(g, w->w1, h, [&](int kappa) {
            return dst + (static_cast<size_t>(kappa >> 2) * NHB * 64 + (kappa & 3) * 16) * 4;
        });
    }
    for (int hb = 0; hb < NHB; ++hb)
        for (int r = 0; r < 4; ++r)
            for (int lane = 0; lane < 64; ++lane) {
                const int row = lane & 15;
                const int hh = 16 * hb + 4 * (lane >> 4) + r;
                if (hh < H && row < L) {
                    wh[((hb * 4 + r) * 2 + 0) * 64 + lane] = w->wmu[row * H + hh];
                    wh[((hb * 4 + r) * 2 + 1) * 64 + lane] = w->wlv[row * H + hh];
                }
                const int hd = 16 * hb + row;
                const int l = 4 * (lane >> 4) + r;
                if (hd < H && l < L)
                    wd[(hb * 4 + r) * 64 + lane] = w->wd1[hd * L + l];
            }
    return prepare_stream_score(g);
}

// Row of register r for lane half g inside a 32x32 matrix-op accumulator block.
int crow(int r, int g) { return 8 * (r >> 2) + 4 * g + (r & 3); }

// Decoder-output fragments of the fused variant pass (32x32x2 fp32 ops whose B operand is the
// decoder hidden layer's accumulator): Wd2 as [D/32][HB][4][64 lanes] x 4 floats, where lane l,
// component e of (ob, hb, r4) holds Wd2[32 ob + l%32][32 hb + crow(4 r4 + e, l/32)] (zero past
// H).
hipError_t pack_ext_fused(enova_detector d, const enova_detect_weights *w, Uploads &up)
{
    const Geometry &g = d->g;
    const int H = g.H, D = g.D, HB = g.HB, nob = D / 32;
    const size_t n_w = static_cast<size_t>(nob) * HB * 4 * 64 * 4;
    float *buf = up.add<float>(&d->wd2p, n_w);
    for (int ob = 0; ob < nob; ++ob)
        for (int hb = 0; hb < HB; ++hb)
            for (int r4 = 0; r4 < 4; ++r4)
                for (int lane = 0; lane < 64; ++lane)
                    for (int e = 0; e < 4; ++e) {
                        const int j = 32 * ob + (lane & 31);
                        const int h = 32 * hb + crow(4 * r4 + e, lane >> 5);
                        if (h < H)
                            buf[((((static_cast<size_t>(ob) * HB + hb) * 4 + r4) * 64 + lane) * 4) + e] =
                                w->wd2[static_cast<int64_t>(j) * H + h];
                    }
    return prepare_ext_fused(g);
}

// Weights the split kernel can take: all finite, none so large that a product of three layers could
// leave the fp32 range, and no input whose weight stands out. An input's f16 parts hold it to 2^-29
// whatever its size, and a window is only known to have one input of kSplitMin (split.h) or more, at any
// place. With e_j = sum_h g_h |W1[h][j]|, g_h the heads' weights of hidden unit h, the heads err by
// some 2^-30 sqrt(sum e_j^2) where they are of the order of 2^-2 e_j or more for that place j: not above
// fp32's own rounding while all e_j are alike, but without a bound where small inputs have large
// weights (half the metrics at 1e-6 under weights of 9e5: scores off by 6e-4, and 4e-3 at 1e-8; in fp32
// 1e-6). So the places may differ by kSplitPlaces and the metrics, over all steps, by kSplitMetrics: that
// keeps the error of such a window below 2^-28 sqrt(D) 16, 1.3e-6 at D = 512 (places: 5e-6). Randomly
// drawn weights differ by 2 to 3 (64 hidden units) and by 1.1.
constexpr float kSplitPlaces = 64.0f, kSplitMetrics = 16.0f;

bool split_weights_ok(const Geometry &g, const enova_detect_weights *w)
{
    const size_t H = g.H, L = g.L, D = g.D;
    auto ok = [](const void *p, size_t n) {
        const float *f = static_cast<const float *>(p);
        bool good = true;
        for (size_t i = 0; i < n; ++i)
            good &= std::fabs(f[i]) < 0x1p20f;   // false for NaN
        return good;
    };
    if (!(ok(w->w1, H * D) && ok(w->b1, H) && ok(w->wmu, L * H) && ok(w->bmu, L) && ok(w->wlv, L * H) &&
          ok(w->blv, L) && ok(w->wd1, H * L) && ok(w->bd1, H)))
        return false;
    std::vector<float> e(D, 0.0f);
    for (size_t h = 0; h < H; ++h) {
        float gh = 0.0f;
        for (size_t l = 0; l < L; ++l)
            gh += std::fabs(w->wmu[l * H + h]) + std::fabs(w->wlv[l * H + h]);
        const float *row = static_cast<const float *>(w->w1) + h * D;
        for (size_t j = 0; j < D; ++j)
            e[j] += gh * std::fabs(row[j]);
    }
    float lo = e[0], hi = e[0];
    for (const float v : e) {
        lo = std::min(lo, v);
        hi = std::max(hi, v);
    }
    if (hi > kSplitPlaces * lo)
        return false;
    std::vector<double> em(g.M, 0.0);
    for (size_t j = 0; j < D; ++j)
        em[j % g.M] += e[j];
    const auto mm = std::minmax_element(em.begin(), em.end());
    return *mm.second <= kSplitMetrics * *mm.first;
}

// Fragments of the split kernel:
//  W1      step i, hidden block hb, part (hi, lo), lane l: the 8 f16 of W1[32 hb + l % 32] at chunk
//          2i + l / 32 (8 elements; zero past the window, the hidden width or the row), each row
//          scaled by 2^e with its largest |w| in [2^13, 2^14); kSplitPrefetch zero steps follow.
//  heads   [hb][m][part][lane] 8 bf16 and decoder [hb][part][lane] 8 bf16: the slots of the bf16
//          detectors' fragments (reduction slot t of lane half g is hidden row crow(8m + t, g),
//          latent crow(t, g)), three parts of each weight.
//  scale   2^-e / kSplitScale of each hidden row.
hipError_t pack_split(enova_detector d, const enova_detect_weights *w, Uploads &up)
{
    const Geometry &g = d->g;
    const SplitGeometry &sg = d->sg;
    const int H = g.H, L = g.L, HB = g.HB;
    const float *w1 = static_cast<const float *>(w->w1);
    const size_t n_w1 = static_cast<size_t>(sg.nsteps + kSplitPrefetch) * HB * 2 * 64;   // 16-byte fragments
    const size_t n_wh = static_cast<size_t>(HB) * 2 * 3 * 64, n_wd = static_cast<size_t>(HB) * 3 * 64;
    uint16_t *w1x = up.add<uint16_t>(&d->w1x, n_w1 * 8), *whx = up.add<uint16_t>(&d->whx, n_wh * 8),
             *wdx = up.add<uint16_t>(&d->wdx, n_wd * 8);
    float *scale = up.add<float>(&d->w1scale, g.Hp);
    // the weight of every element of every chunk (g.D: none)
    const int chunks = sg.Q * sg.CPR;
    std::vector<int> at(static_cast<size_t>(chunks) * 8, g.D);
    for_row(g, sg.Mp, sg.CPR, 8, [&](int j, int kappa, int e) { at[static_cast<size_t>(kappa) * 8 + e] = j; });
    std::vector<float> row(g.D + 1, 0.0f);
    for (int h = 0; h < H; ++h) {
        const float *src = w1 + static_cast<size_t>(h) * g.D;
        float big = 0.0f;
        for (int j = 0; j < g.D; ++j)
            big = std::max(big, std::fabs(src[j]));
        const int e = big > 0.0f ? std::min(13 - std::ilogb(big), 100) : 0;
        const float scaled = std::ldexp(1.0f, e);
        scale[h] = std::ldexp(1.0f, -e - 4);
        for (int j = 0; j < g.D; ++j)
            row[j] = src[j] * scaled;
        uint16_t *dst = w1x + (static_cast<size_t>(h >> 5) * 2 * 64 + (h & 31)) * 8;
        for (int kappa = 0; kappa < chunks; ++kappa) {
            float v[8];
            for (int i = 0; i < 8; ++i)
                v[i] = row[at[static_cast<size_t>(kappa) * 8 + i]];
            uint16_t *to = dst + (static_cast<size_t>(kappa >> 1) * HB * 2 * 64 + (kappa & 1) * 32) * 8;
            f16_parts(v, to, to + 64 * 8);
        }
    }
    auto parts = [](float v, uint16_t *dst, size_t stride) {
        for (int q = 0; q < 3; ++q) {
            const uint16_t b = float_to_bf16_bits(v);
            dst[q * stride] = b;
            v -= bf16_bits_to_float(b);
        }
    };
    for (int hb = 0; hb < HB; ++hb)
        for (int lane = 0; lane < 64; ++lane)
            for (int t = 0; t < 8; ++t) {
                for (int m = 0; m < 2; ++m) {
                    const int row = lane & 31, h = hb * 32 + crow(8 * m + t, lane >> 5);
                    float v = 0.0f;
                    if (h < H && (row & 15) < L)
                        v = row < 16 ? w->wmu[row * H + h] : w->wlv[(row - 16) * H + h];
                    parts(v, whx + (((static_cast<size_t>(hb) * 2 + m) * 3) * 64 + lane) * 8 + t, 64 * 8);
                }
                const int h = hb * 32 + (lane & 31), l = crow(t, lane >> 5);
                parts(h < H && l < L ? w->wd1[h * L + l] : 0.0f,
                      wdx + ((static_cast<size_t>(hb) * 3) * 64 + lane) * 8 + t, 64 * 8);
            }
    const hipError_t e = prepare_score_split(g, d->sg);
    return e == hipSuccess ? prepare_score_list(g) : e;
}

// Fragments of the split variant pass: Wd2's rows in the padded order j' = t Mp + m as two f16 parts,
// scaled by the power of two that puts the largest |weight| into [2^13, 2^14): [Dp/32][HB][2][hi,
// lo][64 lanes] x 8, where slot t of (ob, hb, m), lane l is the weight of row 32 ob + l % 32 at hidden
// unit 32 hb + crow(8 m + t, l / 32); bd2 padded the same way follows.
hipError_t pack_ext_split(enova_detector d, const enova_detect_weights *w, Uploads &uploads)
{
    const Geometry &g = d->g;
    const int H = g.H, HB = g.HB, Mp = d->sg.Mp, Dp = ext_split_rows(g, d->sg);
    float big = 0.0f;
    for (size_t i = 0; i < static_cast<size_t>(g.D) * H; ++i)
        big = std::max(big, std::fabs(w->wd2[i]));
    const int e = big > 0.0f ? std::min(13 - std::ilogb(big), 100) : 0;
    const float up = std::ldexp(1.0f, e);
    d->wd2_unscale = std::ldexp(1.0f, -e);
    const size_t n_w = static_cast<size_t>(Dp / 32) * HB * 2 * 2 * 64;   // 16-byte fragments
    uint16_t *buf = uploads.add<uint16_t>(&d->wd2x, n_w * 8);
    float *bd = uploads.add<float>(&d->bd2x, Dp);
    std::vector<float> units(g.Hp, 0.0f);
    for (int t = 0; t < g.W; ++t)
        for (int m = 0; m < g.M; ++m) {
            const int j = t * Mp + m;
            bd[j] = w->bd2[t * g.M + m];
            const float *row = w->wd2 + static_cast<int64_t>(t * g.M + m) * H;
            for (int h = 0; h < H; ++h)
                units[h] = row[h] * up;
            uint16_t *dst = buf + (static_cast<size_t>(j >> 5) * HB * 2 * 2 * 64 + (j & 31)) * 8;
            for (int f = 0; f < HB * 2; ++f)          // hidden block f / 2, fragment f % 2 of it
                for (int half = 0; half < 2; ++half) {
                    // crow(8 (f % 2) + t, half), t < 8: two runs of four
                    const float *from = &units[16 * f + 4 * half];
                    float v[8];
                    for (int i = 0; i < 8; ++i)
                        v[i] = from[8 * (i >> 2) + (i & 3)];
                    uint16_t *to = dst + (static_cast<size_t>(f) * 2 * 64 + half * 32) * 8;
                    f16_parts(v, to, to + 64 * 8);
                }
        }
    return prepare_ext_split(g, d->sg);
}

// Weights of the decoder's output that the split variant pass can take: finite and below 2^20 (as
// split_weights_ok), and neither a row nor a column whose largest is under kSplitOutput times the largest of
// all (but for zeros). One power of two scales them all, and one a window's hidden activations, which so
// are held to 2^-38 of the largest: rows 1e6 apart, or columns that activations 1e6 apart make up for,
// put the rms error of the other metrics' md at 2.6e-7 to 3.6e-7, against 5e-8 in fp32.
constexpr float kSplitOutput = 0x1p-10f;

bool split_output_ok(const Geometry &g, const enova_detect_weights *w)
{
    const size_t H = g.H, D = g.D;
    std::vector<float> col(H, 0.0f);
    float big = 0.0f, least = INFINITY;
    for (size_t j = 0; j < D; ++j) {
        float row = 0.0f;
        for (size_t h = 0; h < H; ++h) {
            const float a = std::fabs(w->wd2[j * H + h]);
            if (!(a < 0x1p20f))   // also for NaN
                return false;
            row = std::max(row, a);
            col[h] = std::max(col[h], a);
        }
        big = std::max(big, row);
        if (row > 0.0f)
            least = std::min(least, row);
    }
    for (const float c : col)
        if (c > 0.0f)
            least = std::min(least, c);
    return !(least < kSplitOutput * big);
}

void free_detector(enova_detector d)
{
    if (!d)
        return;
    for (void *p : d->weights)
        (void)hipFree(p);
    void *ptrs[] = {d->stats, d->tiles, d->tile_map, d->cal, d->pot,
                    d->peaks, d->blk, d->pot_part, d->ext_ws};
    for (void *p : ptrs)
        if (p)
            (void)hipFree(p);
    if (d->pot_out)
        (void)hipHostFree(d->pot_out);
    for (hipEvent_t e : d->ev)
        if (e)
            (void)hipEventDestroy(e);
    for (hipEvent_t e : d->ext_ev)
        if (e)
            (void)hipEventDestroy(e);
    delete d;
}

enova_status check_config(const enova_detect_config *c)
{
    if (!c)
        return fail(ENOVA_EINVAL, "config is NULL");
    if (c->metrics < 1 || c->window < 1 || c->stride < 1 || c->hidden < 1 || c->latent < 1)
        return fail(ENOVA_EINVAL, "metrics, window, stride, hidden and latent must be >= 1");
    if (c->latent > 64)
        return fail(ENOVA_EINVAL, "latent %d > 64", c->latent);
    if (static_cast<int64_t>(c->window) * c->metrics > 65536)
        return fail(ENOVA_EINVAL, "window*metrics = %lld > 65536",
                    static_cast<long long>(c->window) * c->metrics);
    if (c->dtype != ENOVA_F32 && c->dtype != ENOVA_BF16)
        return fail(ENOVA_EINVAL, "unknown dtype %d", c->dtype);
    if (c->act != ENOVA_RELU && c->act != ENOVA_TANH)
        return fail(ENOVA_EINVAL, "unknown activation %d", c->act);
    if (c->kernel < ENOVA_KERNEL_AUTO || c->kernel > ENOVA_KERNEL_MFMA)
        return fail(ENOVA_EINVAL, "unknown kernel choice %d", c->kernel);
    if (!(c->ref_frac > 0.0f && c->ref_frac <= 1.0f))
        return fail(ENOVA_EINVAL, "ref_frac must be in (0, 1]");
    return ENOVA_OK;
}

}  // namespace

extern "C" {

const char *enova_status_str(enova_status s)
{
    switch (s) {
    case ENOVA_OK: return "ok";
    case ENOVA_EINVAL: return "invalid argument";
    case ENOVA_ESHAPE: return "nothing to act on for this shape";
    case ENOVA_ENOMEM: return "out of memory";
    case ENOVA_EHIP: return "HIP runtime error";
    case ENOVA_EUNSUPPORTED: return "unsupported request";
    case ENOVA_ENUMERIC: return "non-finite values";
    }
    return "unknown status";
}

const char *enova_last_error(void) { return g_last_error.c_str(); }

static enova_status fill_detector(enova_detector d, const enova_detect_weights *w);

enova_status enova_detect_init(const enova_detect_config *config, const enova_detect_weights *w,
                               enova_detector *out)
{
    if (!out)
        return fail(ENOVA_EINVAL, "out is NULL");
    *out = nullptr;
    enova_status st = check_config(config);
    if (st != ENOVA_OK)
        return st;
    if (!w || !w->w1 || !w->b1 || !w->wmu || !w->bmu || !w->wlv || !w->blv || !w->wd1 || !w->bd1 ||
        !w->wd2 || !w->bd2)
        return fail(ENOVA_EINVAL, "a weight pointer is NULL");

    enova_detector d = new (std::nothrow) enova_detector_s();
    if (!d)
        return fail(ENOVA_ENOMEM, "host allocation");
    Geometry &g = d->g;
    plan_geometry(*config, &g);
    if (config->kernel == ENOVA_KERNEL_MFMA && !g.mfma_ok) {
        // the message reads the geometry, which the detector owns: format it before the free
        st = fail(ENOVA_EUNSUPPORTED,
                  "matrix-core kernel needs hidden <= 256, latent <= 16 and a tile that fits LDS "
                  "(H=%d L=%d LDS=%zu)", g.H, g.L, g.lds_bytes);
        free_detector(d);
        return st;
    }
    if (config->kernel == ENOVA_KERNEL_VALU || !g.mfma_ok) {
        if (g.H > 1024) {
            st = fail(ENOVA_EUNSUPPORTED, "hidden width %d > 1024 is not supported", g.H);
            free_detector(d);
            return st;
        }
        d->kind = 1;
    } else {
        d->kind = 2;
    }
    if (hipGetDevice(&d->device) != hipSuccess) {
        free_detector(d);
        return fail(ENOVA_EHIP, "no current HIP device");
    }
    {
        // the device address of this device's fixed scratch, looked up with the device current
        const hipError_t e = scratch_setup(d->device, &d->scratch);
        if (e != hipSuccess) {
            free_detector(d);
            return hip_fail(e, "device scratch lookup");
        }
    }
    try {
        st = fill_detector(d, w);
    } catch (const std::bad_alloc &) {
        st = fail(ENOVA_ENOMEM, "host allocation");
    }
    if (st != ENOVA_OK) {
        free_detector(d);
        return st;
    }
    *out = d;
    return ENOVA_OK;
}

// Packs the weights for the kernels that the shape takes and uploads them.
static enova_status fill_detector(enova_detector d, const enova_detect_weights *w)
{
    const Geometry &g = d->g;
    const int H = g.H, L = g.L, D = g.D, Hp = g.Hp;
    const bool bf = g.dtype == ENOVA_BF16;
    Uploads up;
    // small arrays: b1[Hp] bd1[Hp] u[Hp] bh[32] bmu[L] blv[L] wmu[L*H] wlv[L*H] wd1[H*L]
    //               whp[HB*16*64] wd1p[HB*8*64]
    const size_t n_whp = d->kind == 2 ? static_cast<size_t>(g.HB) * 16 * 64 : 0;
    const size_t n_wd1p = d->kind == 2 ? static_cast<size_t>(g.HB) * 8 * 64 : 0;
    // every sub-array starts on a 16-byte boundary (the kernels copy them with 16-byte loads)
    size_t o = 0;
    auto take = [&o](size_t n) {
        const size_t at = o;
        o += (n + 3) / 4 * 4;
        return at;
    };
    // the matrix-core kernel copies whp, wd1p, b1, bd1, u, bh as one contiguous block into LDS
    const size_t o_whp = take(n_whp);
    const size_t o_wd1p = take(n_wd1p);
    const size_t o_b1 = take(Hp);
    const size_t o_bd1 = take(Hp);
    const size_t o_u = take(Hp);
    const size_t o_bh = take(32);
    const size_t o_bmu = take(L);
    const size_t o_blv = take(L);
    const size_t o_wmu = take(static_cast<size_t>(L) * H);
    const size_t o_wlv = take(static_cast<size_t>(L) * H);
    const size_t o_wd1 = take(static_cast<size_t>(H) * L);
    float *small = up.add<float>(&d->small, o);

    std::vector<double> cs(H, 0.0);
    for (int j = 0; j < D; ++j)
        for (int h = 0; h < H; ++h)
            cs[h] += static_cast<double>(w->wd2[static_cast<int64_t>(j) * H + h]);
    for (int h = 0; h < H; ++h) {
        small[o_b1 + h] = w->b1[h];
        small[o_bd1 + h] = w->bd1[h];
        small[o_u + h] = static_cast<float>(cs[h]);
    }
    double sb = 0.0;
    for (int j = 0; j < D; ++j)
        sb += static_cast<double>(w->bd2[j]);
    d->sum_bd2 = static_cast<float>(sb);
    for (int l = 0; l < L; ++l) {
        small[o_bmu + l] = w->bmu[l];
        small[o_blv + l] = w->blv[l];
        if (l < 16) {
            small[o_bh + l] = w->bmu[l];
            small[o_bh + 16 + l] = w->blv[l];
        }
    }
    std::memcpy(&small[o_wmu], w->wmu, sizeof(float) * L * H);
    std::memcpy(&small[o_wlv], w->wlv, sizeof(float) * L * H);
    std::memcpy(&small[o_wd1], w->wd1, sizeof(float) * H * L);
    if (d->kind == 2 && bf) {
        // bf16 workload: the heads and decoder weights as bf16 hi + lo fragments of the
        // 32x32x16 matrix op; reduction slot (g, t) of heads op m is hidden row crow(8m + t, g),
        // of the decoder op latent crow(t, g)
        uint16_t *whb = reinterpret_cast<uint16_t *>(&small[o_whp]);
        uint16_t *wdb = reinterpret_cast<uint16_t *>(&small[o_wd1p]);
        for (int hb = 0; hb < g.HB; ++hb)
            for (int m = 0; m < 2; ++m)
                for (int lane = 0; lane < 64; ++lane)
                    for (int t = 0; t < 8; ++t) {
                        const int row = lane & 31;          // 0..15 mean head, 16..31 log-variance
                        const int h = hb * 32 + crow(8 * m + t, lane >> 5);
                        float v = 0.0f;
                        if (h < H) {
                            if (row < 16 && row < L)
                                v = w->wmu[row * H + h];
                            else if (row >= 16 && row - 16 < L)
                                v = w->wlv[(row - 16) * H + h];
                        }
                        const uint16_t hi = float_to_bf16_bits(v);
                        const uint16_t lo = float_to_bf16_bits(v - bf16_bits_to_float(hi));
                        whb[((((static_cast<size_t>(hb) * 2 + m) * 2 + 0) * 64 + lane) * 8) + t] = hi;
                        whb[((((static_cast<size_t>(hb) * 2 + m) * 2 + 1) * 64 + lane) * 8) + t] = lo;
                    }
        for (int hb = 0; hb < g.HB; ++hb)
            for (int lane = 0; lane < 64; ++lane)
                for (int t = 0; t < 8; ++t) {
                    const int h = hb * 32 + (lane & 31);
                    const int l = crow(t, lane >> 5);
                    float v = 0.0f;
                    if (h < H && l < L)
                        v = w->wd1[h * L + l];
                    const uint16_t hi = float_to_bf16_bits(v);
                    const uint16_t lo = float_to_bf16_bits(v - bf16_bits_to_float(hi));
                    wdb[(((static_cast<size_t>(hb) * 2 + 0) * 64 + lane) * 8) + t] = hi;
                    wdb[(((static_cast<size_t>(hb) * 2 + 1) * 64 + lane) * 8) + t] = lo;
                }
    } else if (d->kind == 2) {
        for (int hb = 0; hb < g.HB; ++hb)
            for (int r = 0; r < 16; ++r)
                for (int lane = 0; lane < 64; ++lane) {
                    const int row = lane & 31;              // 0..15 mean head, 16..31 log-variance head
                    const int h = hb * 32 + crow(r, lane >> 5);
                    float v = 0.0f;
                    if (h < H) {
                        if (row < 16 && row < L)
                            v = w->wmu[row * H + h];
                        else if (row >= 16 && row - 16 < L)
                            v = w->wlv[(row - 16) * H + h];
                    }
                    small[o_whp + (static_cast<size_t>(hb) * 16 + r) * 64 + lane] = v;
                }
        for (int hb = 0; hb < g.HB; ++hb)
            for (int r = 0; r < 8; ++r)
                for (int lane = 0; lane < 64; ++lane) {
                    const int h = hb * 32 + (lane & 31);
                    const int l = crow(r, lane >> 5);
                    float v = 0.0f;
                    if (h < H && l < L)
                        v = w->wd1[h * L + l];
                    small[o_wd1p + (static_cast<size_t>(hb) * 8 + r) * 64 + lane] = v;
                }
    }
    // dense fp32 copies for the output variants (16-byte aligned sub-arrays)
    float *w1 = up.add<float>(&d->d_w1, static_cast<size_t>(H) * D);
    if (bf) {
        const uint16_t *src = static_cast<const uint16_t *>(w->w1);
        for (size_t i = 0; i < static_cast<size_t>(H) * D; ++i)
            w1[i] = bf16_bits_to_float(src[i]);
    } else {
        std::memcpy(w1, w->w1, sizeof(float) * static_cast<size_t>(H) * D);
    }
    float *wml = up.add<float>(&d->d_wml, 2 * static_cast<size_t>(L) * H), *bml = up.add<float>(&d->d_bml, 2 * L);
    std::memcpy(wml, w->wmu, sizeof(float) * L * H);
    std::memcpy(wml + static_cast<size_t>(L) * H, w->wlv, sizeof(float) * L * H);
    std::memcpy(bml, w->bmu, sizeof(float) * L);
    std::memcpy(bml + L, w->blv, sizeof(float) * L);
    std::memcpy(up.add<float>(&d->d_wd1, static_cast<size_t>(H) * L), w->wd1, sizeof(float) * H * L);
    std::memcpy(up.add<float>(&d->d_wd2, static_cast<size_t>(D) * H), w->wd2, sizeof(float) * static_cast<size_t>(D) * H);
    std::memcpy(up.add<float>(&d->d_bd2, D), w->bd2, sizeof(float) * D);

    hipError_t e = hipSuccess;
    const char *what = "";
    auto pack = [&](hipError_t (*fn)(enova_detector, const enova_detect_weights *, Uploads &), const char *kernel) {
        if (e == hipSuccess) {
            e = fn(d, w, up);
            what = kernel;
        }
    };
    if (d->kind == 1) {
        // transposed W1 [D][H] in the storage type
        const size_t esz = bf ? 2 : 4;
        unsigned char *wt = up.add<unsigned char>(&d->w1t, static_cast<size_t>(D) * H * esz);
        for (int h = 0; h < H; ++h)
            for (int j = 0; j < D; ++j) {
                const size_t dst = (static_cast<size_t>(j) * H + h) * esz;
                const size_t src = (static_cast<size_t>(h) * D + j) * esz;
                std::memcpy(&wt[dst], static_cast<const unsigned char *>(w->w1) + src, esz);
            }
    } else {
        // A fragments: step i, hidden block hb, lane -> 16 bytes of W1[h][chunk 2i + lane/32]
        // kPrefetchSteps zero steps follow the last one: the kernel's W1 prefetch runs past it
        const int steps = g.KC / 2;
        const size_t frag = static_cast<size_t>(steps + kPrefetchSteps) * g.HB * 64;
        uint32_t *pk = up.add<uint32_t>(&d->w1p, frag * 4);
        for (int h = 0; h < H; ++h) {
            uint32_t *dst = pk + (static_cast<size_t>(h >> 5) * 64 + (h & 31)) * 4;
            pack_row(g, w->w1, h, [&](int kappa) {
                return dst + (static_cast<size_t>(kappa >> 1) * g.HB * 64 + (kappa & 1) * 32) * 4;
            });
        }
        pack([](enova_detector q, const enova_detect_weights *, Uploads &) { return prepare_score_mfma(q->g); },
             "configure matrix-core kernel");
        if (g.ring)
            pack(pack_ring, "configure the ring scoring kernel");
        d->sg = plan_split(g);
        d->sg.ok = d->sg.ok && score_list_lds(g) <= kLdsLimit && split_weights_ok(g, w);
        if (d->sg.ok)
            pack(pack_split, "configure the split scoring kernel");
        if (stream_score_supported(g))
            pack(pack_stream, "configure the streaming scoring kernel");
        if (ext_split_supported(g, d->sg) && split_output_ok(g, w))
            pack(pack_ext_split, "configure the split variant kernel");
        else if (ext_fused_supported(g))
            pack(pack_ext_fused, "configure the fused variant kernel");
    }
    if (e != hipSuccess)
        return hip_fail(e, what);
    const enova_status st = up.upload(d->weights);
    if (st != ENOVA_OK)
        return st;
    d->b1 = d->small + o_b1;
    d->bd1 = d->small + o_bd1;
    d->u = d->small + o_u;
    d->bh = d->small + o_bh;
    d->bmu = d->small + o_bmu;
    d->blv = d->small + o_blv;
    d->wmu = d->small + o_wmu;
    d->wlv = d->small + o_wlv;
    d->wd1 = d->small + o_wd1;
    d->whp = d->small + o_whp;
    d->wd1p = d->small + o_wd1p;
    return ENOVA_OK;
}

enova_status enova_detect_destroy(enova_detector det)
{
    if (!det)
        return ENOVA_OK;
    DeviceGuard dg(det->device);
    (void)hipDeviceSynchronize();
    free_detector(det);
    return ENOVA_OK;
}

enova_status enova_detect_window_offsets(enova_detector det, const int64_t *soff, int32_t n,
                                         int64_t *woff)
{
    if (!det || !soff || !woff)
        return fail(ENOVA_EINVAL, "NULL argument");
    if (n < 0)
        return fail(ENOVA_EINVAL, "n_streams < 0");
    if (soff[0] != 0)
        return fail(ENOVA_EINVAL, "stream_offsets[0] must be 0");
    const int64_t W = det->g.W, S = det->g.S;
    woff[0] = 0;
    for (int32_t s = 0; s < n; ++s) {
        const int64_t T = soff[s + 1] - soff[s];
        if (T < 0)
            return fail(ENOVA_EINVAL, "stream_offsets decrease at stream %d", s);
        woff[s + 1] = woff[s] + (T >= W ? (T - W) / S + 1 : 0);
    }
    return ENOVA_OK;
}

enova_status enova_detect_ref_stats(enova_detector det, const void *x, const int64_t *soff,
                                    int32_t n, float *out_mean, float *out_std, hipStream_t stream)
{
    if (!det)
        return fail(ENOVA_EINVAL, "detector is NULL");
    if (n < 0)
        return fail(ENOVA_EINVAL, "n_streams < 0");
    if (n == 0)
        return ENOVA_OK;
    if (!x || !soff || !out_mean || !out_std)
        return fail(ENOVA_EINVAL, "NULL argument");
    DeviceGuard dg(det->device);
    hipError_t e = launch_ref_stats(det->g, x, soff, n, out_mean, out_std, nullptr, stream);
    if (e != hipSuccess)
        return hip_fail(e, "reference statistics kernel");
    return ENOVA_OK;
}

namespace {

// The scoring path's workspace: reference statistics [2][n][M] floats (when the caller gives
// none) and their chunk sums, the matrix-core kernel's first tile of each stream [n+1] and stream
// of each block [grid], with the split kernel's marks behind it.
struct ScoreWork {
    float *stats = nullptr;
    double *part = nullptr;
    int64_t *tiles = nullptr;
    int *tile_map = nullptr;
};

// Entries of the tile map (and of the marks: a tile holds a window at the least).
size_t map_ints(int64_t grid, int64_t n_windows, bool split)
{
    const size_t map = static_cast<size_t>(grid > 0 ? grid : 1);
    return split ? map + 1 + static_cast<size_t>(std::min(grid, n_windows)) : map;
}

// Floats of the statistics and of their chunk sums behind them (on a 16-byte boundary).
size_t stats_floats(int32_t n, int M, size_t *o_part)
{
    *o_part = (2 * static_cast<size_t>(n) * M + 3) / 4 * 4;
    return *o_part + stat_part_bytes(n, M) / sizeof(float);
}

// Bytes of the fixed-scratch layout of that workspace, each part on a 256-byte boundary. The chunk
// sums come last and only where they still fit the scratch (*o_part = 0: one block per stream).
size_t noalloc_bytes(const Geometry &g, int kind, int32_t n, int64_t grid, int64_t n_windows, bool split, bool stats,
                     size_t *o_tiles, size_t *o_map, size_t *o_part)
{
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    size_t o = stats ? up(2 * static_cast<size_t>(n) * g.M * sizeof(float)) : 0;
    *o_tiles = o;
    if (kind == 2)
        o += up((static_cast<size_t>(n) + 1) * sizeof(int64_t));
    *o_map = o;
    if (kind == 2)
        o += up(map_ints(grid, n_windows, split) * sizeof(int));
    *o_part = 0;
    const size_t part = stats ? stat_part_bytes(n, g.M) : 0;
    if (part > 0 && o > 0 && o + part <= kScratchBytes) {
        *o_part = o;
        o += part;
    }
    return o;
}

// Windows of fewer values than this are scored by the fp32 kernel. Of independent normal values a share of
// 0.2^D windows has them all below kSplitMin (split.h), which the split kernel leaves to its list: one in
// five of a single value, and every wave has some up to three. 200 streams x 8000 steps, H = 32, 64, 128,
// 200, split and fp32 in us: D = 1 274, 435, 882, 1702 and 159, 271, 476, 923; D = 3 212, 327, 639, 1029 and 162,
// 276, 480, 926; D = 4 158, 238, 401, 650 and 163, 279, 482, 925.
constexpr int kSplitLeastD = 4;

// Both scoring entry points. noalloc: the workspace is carved from the device's fixed scratch
// (no allocation, no timing events); otherwise it is the detector's grow-only workspace.
enova_status score_common(enova_detector det, const void *x, const int64_t *soff, const int64_t *woff, int32_t n,
                          int64_t n_windows, const float *ref_mean, const float *ref_std, float threshold,
                          float *out_scores, float *out_md, uint8_t *out_flags, hipStream_t stream, bool noalloc)
{
    if (!det)
        return fail(ENOVA_EINVAL, "detector is NULL");
    if (n < 0 || n_windows < 0)
        return fail(ENOVA_EINVAL, "n_streams and n_windows must be >= 0");
    if ((ref_mean == nullptr) != (ref_std == nullptr))
        return fail(ENOVA_EINVAL, "ref_mean and ref_std must both be given or both be NULL");
    det->ran_stats = det->ran_score = false;
    if (n == 0 || n_windows == 0)
        return ENOVA_OK;
    if (!x || !soff || !woff || !out_scores)
        return fail(ENOVA_EINVAL, "NULL argument");
    const bool want_flags = out_flags != nullptr && !std::isnan(threshold);
    const Geometry &g = det->g;
    // windows per tile: the split kernel's where it applies, unless its smaller tiles need more
    // blocks or workspace than a call may have
    bool split = det->kind == 2 && det->sg.ok && g.D >= kSplitLeastD;
    int nb = split ? det->sg.nb(n_windows, n) : g.Nb;
    int64_t grid = det->kind == 2 ? (n_windows + nb - 1) / nb + n : 0;
    size_t o_tiles = 0, o_map = 0, o_part = 0;
    auto layout = [&]() {
        return noalloc ? noalloc_bytes(g, det->kind, n, grid, n_windows, split, !ref_mean, &o_tiles, &o_map, &o_part) : 0;
    };
    size_t need = layout();
    if (split && (grid > kMaxMarked || need > kScratchBytes)) {
        split = false;
        nb = g.Nb;
        grid = (n_windows + nb - 1) / nb + n;
        need = layout();
    }
    if (grid > 0x7fffffffLL)
        return fail(ENOVA_EUNSUPPORTED, "too many tiles (%lld)", static_cast<long long>(grid));
    if (det->kind != 2 && (n_windows + 15) / 16 > 0x7fffffffLL)
        return fail(ENOVA_EUNSUPPORTED, "too many windows");
    ScoreWork wk;
    if (noalloc) {
        if (need > kScratchBytes)
            return fail(ENOVA_ESHAPE,
                        "the allocation-free call needs %zu bytes of device scratch for %d streams and %lld "
                        "windows; it has %zu",
                        need, n, static_cast<long long>(n_windows), kScratchBytes);
        if (!det->scratch)
            return fail(ENOVA_EHIP, "device scratch unavailable");
        unsigned char *base = static_cast<unsigned char *>(det->scratch);
        wk.stats = reinterpret_cast<float *>(base);
        wk.tiles = reinterpret_cast<int64_t *>(base + o_tiles);
        wk.tile_map = reinterpret_cast<int *>(base + o_map);
        wk.part = o_part ? reinterpret_cast<double *>(base + o_part) : nullptr;
    }
    DeviceGuard dg(det->device);
    if (!dg.ok)
        return fail(ENOVA_EHIP, "cannot select the detector's device");
    hipError_t e;
    const bool timing = det->timing && !noalloc;
    if (timing && !det->ev[0]) {
        for (auto &ev : det->ev)
            if ((e = hipEventCreate(&ev)) != hipSuccess)
                return hip_fail(e, "hipEventCreate");
    }
    if (!noalloc) {
        enova_status st = ENOVA_OK;
        size_t o_part = 0;
        if (!ref_mean)
            st = ensure(&det->stats, &det->stats_cap, stats_floats(n, g.M, &o_part));
        if (st == ENOVA_OK && det->kind == 2) {
            st = ensure(&det->tiles, &det->tiles_cap, static_cast<size_t>(n) + 1);
            if (st == ENOVA_OK)
                st = ensure(&det->tile_map, &det->tile_map_cap, map_ints(grid, n_windows, split));
        }
        if (st != ENOVA_OK)
            return st;
        wk.stats = det->stats;
        if (!ref_mean && stat_part_bytes(n, g.M) > 0)
            wk.part = reinterpret_cast<double *>(det->stats + o_part);
        wk.tiles = det->tiles;
        wk.tile_map = det->tile_map;
    }
    const bool own = !ref_mean;
    float *own_mean = own ? wk.stats : nullptr, *own_std = own ? wk.stats + static_cast<size_t>(n) * g.M : nullptr;
    if (own) {
        ref_mean = own_mean;
        ref_std = own_std;
    }
    if (timing && own)
        (void)hipEventRecord(det->ev[0], stream);
    if (det->kind == 2) {
        e = launch_prep_scan(g, x, soff, woff, n, nb, wk.tiles, own_mean, own_std, wk.part, stream);
        if (e != hipSuccess)
            return hip_fail(e, "tile scan and reference statistics kernels");
    } else if (own) {
        e = launch_ref_stats(g, x, soff, n, own_mean, own_std, wk.part, stream);
        if (e != hipSuccess)
            return hip_fail(e, "reference statistics kernel");
    }
    // chunk sums are closed by the tile map's launch
    const bool stats_in_map = own && det->kind == 2 && wk.part;
    if (timing && own && !stats_in_map)
        (void)hipEventRecord(det->ev[1], stream);
    det->ran_stats = timing && own;
    ScoreParams p{};
    p.x = x;
    p.soff = soff;
    p.woff = woff;
    p.n_streams = n;
    p.n_windows = n_windows;
    p.mean = ref_mean;
    p.std = ref_std;
    p.w1p = det->w1p;
    p.whp = det->whp;
    p.wd1p = det->wd1p;
    p.w1t = det->w1t;
    p.wmu = det->wmu;
    p.wlv = det->wlv;
    p.wd1 = det->wd1;
    p.b1 = det->b1;
    p.bh = det->bh;
    p.bmu = det->bmu;
    p.blv = det->blv;
    p.bd1 = det->bd1;
    p.u = det->u;
    p.w1r = det->w1r;
    p.whr = det->whr;
    p.wdr = det->wdr;
    p.w1x = det->w1x;
    p.whx = det->whx;
    p.wdx = det->wdx;
    p.w1scale = det->w1scale;
    p.sum_bd2 = det->sum_bd2;
    p.threshold = threshold;
    p.write_flags = want_flags ? 1 : 0;
    p.scores = out_scores;
    p.md = out_md;
    p.flags = out_flags;
    if (det->kind == 2) {
        p.tile_off = wk.tiles;
        p.marks = split ? reinterpret_cast<unsigned *>(wk.tile_map + grid) : nullptr;
        e = launch_prep_map(g, x, soff, wk.tiles, n, grid, wk.tile_map, p.marks, own_mean, own_std, wk.part, stream);
        if (e != hipSuccess)
            return hip_fail(e, "tile map kernel");
        if (timing && stats_in_map)
            (void)hipEventRecord(det->ev[1], stream);
        p.tile_stream = wk.tile_map;
        if (timing)
            (void)hipEventRecord(det->ev[2], stream);
        if (split) {
            e = launch_score_split(g, det->sg, p, nb, grid, stream);
            if (e == hipSuccess)
                e = launch_score_list(g, p, nb, grid, stream);
        } else {
            e = g.ring ? launch_score_ring(g, p, grid, stream) : launch_score_mfma(g, p, grid, stream);
        }
    } else {
        if (timing)
            (void)hipEventRecord(det->ev[2], stream);
        e = launch_score_valu(g, p, stream);
    }
    if (e != hipSuccess)
        return hip_fail(e, "scoring kernel");
    if (timing)
        (void)hipEventRecord(det->ev[3], stream);
    det->ran_score = timing;
    return ENOVA_OK;
}

}  // namespace

enova_status enova_detect_score(enova_detector det, const void *x, const int64_t *soff,
                                const int64_t *woff, int32_t n, int64_t n_windows,
                                const float *ref_mean, const float *ref_std, float threshold,
                                float *out_scores, float *out_md, uint8_t *out_flags,
                                hipStream_t stream)
{
    return score_common(det, x, soff, woff, n, n_windows, ref_mean, ref_std, threshold, out_scores, out_md,
                        out_flags, stream, false);
}

enova_status enova_detect_score_noalloc(enova_detector det, const void *x, const int64_t *soff,
                                        const int64_t *woff, int32_t n, int64_t n_windows,
                                        const float *ref_mean, const float *ref_std, float threshold,
                                        float *out_scores, float *out_md, uint8_t *out_flags,
                                        hipStream_t stream)
{
    return score_common(det, x, soff, woff, n, n_windows, ref_mean, ref_std, threshold, out_scores, out_md,
                        out_flags, stream, true);
}

}  // extern "C"

namespace {

// Tiles of a fused pass over n streams, its grid.
int64_t ext_tiles(int32_t n, int64_t n_windows) { return (n_windows + kExtFusedNb - 1) / kExtFusedNb + n; }

// The evaluation of a variants call (ENOVA_EXT_*). A shape that only the split pass takes goes to the
// chunked evaluation also where its tiles are more than a launch can have.
int ext_route(enova_detector d, int32_t n, int64_t n_windows, int norm)
{
    if (d->wd2x && (ext_fused_supported(d->g) ||
                    (ext_tiles(n, n_windows) <= 0x7fffffffLL && ext_split_pays(d->g, d->sg, n_windows, norm))))
        return ENOVA_EXT_SPLIT;
    return d->wd2p ? ENOVA_EXT_FUSED : ENOVA_EXT_CHUNKED;
}

}  // namespace

extern "C" {

enova_status enova_detect_score_ext(enova_detector det, const void *x, const int64_t *soff, const int64_t *woff,
                                    int32_t n, int64_t n_windows, const float *ref_mean, const float *ref_std,
                                    int32_t norm, float *out_scores, float *out_md, float *out_md_metric,
                                    float *out_recon, hipStream_t stream)
{
    if (!det)
        return fail(ENOVA_EINVAL, "detector is NULL");
    if (n < 0 || n_windows < 0)
        return fail(ENOVA_EINVAL, "n_streams and n_windows must be >= 0");
    if (norm != ENOVA_NORM_REFERENCE && norm != ENOVA_NORM_WINDOW)
        return fail(ENOVA_EINVAL, "bad normalisation mode");
    if ((ref_mean == nullptr) != (ref_std == nullptr))
        return fail(ENOVA_EINVAL, "ref_mean and ref_std must both be given or both be NULL");
    det->ran_ext = false;
    if (n == 0 || n_windows == 0)
        return ENOVA_OK;
    if (!x || !soff || !woff)
        return fail(ENOVA_EINVAL, "NULL argument");
    const Geometry &g = det->g;
    if (g.M > kExtMaxM)
        return fail(ENOVA_EUNSUPPORTED, "output variants support at most %d metrics", kExtMaxM);
    DeviceGuard dg(det->device);
    if (!dg.ok)
        return fail(ENOVA_EHIP, "cannot select the detector's device");
    hipError_t e;
    if (det->timing && !det->ext_ev[0]) {
        for (auto &ev : det->ext_ev)
            if ((e = hipEventCreate(&ev)) != hipSuccess)
                return hip_fail(e, "hipEventCreate");
    }
    const int D = g.D, H = g.H, L = g.L, M = g.M;
    const int route = ext_route(det, n, n_windows, norm);
    if (route != ENOVA_EXT_CHUNKED) {
        // fused pass: one block per 256-window tile, every output written directly
        const bool split = route == ENOVA_EXT_SPLIT;
        const int64_t grid = ext_tiles(n, n_windows);
        if (grid > 0x7fffffffLL)
            return fail(ENOVA_EUNSUPPORTED, "too many tiles (%lld)", static_cast<long long>(grid));
        const bool stats = norm == ENOVA_NORM_REFERENCE && !ref_mean;
        // workspace: reference statistics [2][n][M] floats and their chunk sums, first tile of each
        // stream [n+1] int64, the split pass's masks [grid][4] int64, stream of each block [grid] ints, its
        // marks (a tile holds a window at the least)
        size_t o_part = 0;
        const size_t n_st = stats ? stats_floats(n, M, &o_part) : 0;
        const size_t n_tiles = 2 * (static_cast<size_t>(n) + 1);
        const size_t n_masks = split ? 8 * static_cast<size_t>(grid) : 0;
        const size_t n_marks = split ? 1 + static_cast<size_t>(std::min(grid, n_windows)) : 0;
        enova_status st = ensure(&det->ext_ws, &det->ext_ws_cap,
                                 n_st + n_tiles + n_masks + static_cast<size_t>(grid) + n_marks + 4);
        if (st != ENOVA_OK)
            return st;
        int64_t *tiles = reinterpret_cast<int64_t *>(det->ext_ws + n_st);
        uint64_t *masks = reinterpret_cast<uint64_t *>(tiles + n + 1);
        int *tmap = reinterpret_cast<int *>(masks + n_masks / 2);
        unsigned *marks = split ? reinterpret_cast<unsigned *>(tmap + grid) : nullptr;
        if (det->timing)
            (void)hipEventRecord(det->ext_ev[0], stream);
        float *own_mean = stats ? det->ext_ws : nullptr;
        float *own_std = stats ? det->ext_ws + static_cast<size_t>(n) * M : nullptr;
        double *part = stats && stat_part_bytes(n, M) > 0 ? reinterpret_cast<double *>(det->ext_ws + o_part) : nullptr;
        if (stats) {
            ref_mean = own_mean;
            ref_std = own_std;
        }
        if ((e = launch_prep_scan(g, x, soff, woff, n, kExtFusedNb, tiles, own_mean, own_std, part, stream)) !=
            hipSuccess)
            return hip_fail(e, "tile scan and reference statistics kernels");
        if ((e = launch_prep_map(g, x, soff, tiles, n, grid, tmap, marks, own_mean, own_std, part, stream)) != hipSuccess)
            return hip_fail(e, "tile map kernel");
        const int decode = (out_md || out_md_metric || out_recon) ? 1 : 0;
        ExtFusedParams fp{};
        fp.x = static_cast<const float *>(x);
        fp.soff = soff;
        fp.woff = woff;
        fp.tile_off = tiles;
        fp.tile_stream = tmap;
        fp.mean = ref_mean;
        fp.std = ref_std;
        fp.w1p = det->w1p;
        fp.cst = det->whp;
        fp.wd2p = det->wd2p;
        fp.bd2 = det->d_bd2;
        fp.scores = out_scores;
        fp.md = out_md;
        fp.mdm = out_md_metric;
        fp.rec = out_recon;
        fp.norm = norm;
        fp.decode = decode;
        if (split) {
            ExtSplitParams sp{};
            sp.x = static_cast<const float *>(x);
            sp.soff = soff;
            sp.woff = woff;
            sp.tile_off = tiles;
            sp.tile_stream = tmap;
            sp.marks = marks;
            sp.masks = masks;
            sp.mean = ref_mean;
            sp.std = ref_std;
            sp.w1x = det->w1x;
            sp.whx = det->whx;
            sp.wdx = det->wdx;
            sp.w1scale = det->w1scale;
            sp.wd2x = det->wd2x;
            sp.bd2 = det->bd2x;
            sp.b1 = det->b1;
            sp.bd1 = det->bd1;
            sp.bh = det->bh;
            sp.w1 = det->d_w1;
            sp.wml = det->d_wml;
            sp.bml = det->d_bml;
            sp.wd1 = det->d_wd1;
            sp.wd2 = det->d_wd2;
            sp.bd2d = det->d_bd2;
            sp.scores = out_scores;
            sp.md = out_md;
            sp.mdm = out_md_metric;
            sp.rec = out_recon;
            sp.norm = norm;
            sp.decode = decode;
            e = launch_ext_split(g, det->sg, sp, det->wd2_unscale, grid, stream);
            if (e == hipSuccess && ext_fused_list_supported(g)) {
                fp.marks = marks;
                fp.masks = masks;
                fp.wd2 = det->d_wd2;
                e = launch_ext_fused_list(g, fp, grid, stream);
            } else if (e == hipSuccess) {
                e = launch_ext_list(g, det->sg, sp, grid, stream);
            }
            if (e != hipSuccess)
                return hip_fail(e, "split variant kernels");
            if (det->timing)
                (void)hipEventRecord(det->ext_ev[1], stream);
            det->ran_ext = true;
            return ENOVA_OK;
        }
        if ((e = launch_ext_fused(g, fp, grid, stream)) != hipSuccess)
            return hip_fail(e, "fused variant kernel");
        if (det->timing)
            (void)hipEventRecord(det->ext_ev[1], stream);
        det->ran_ext = true;
        return ENOVA_OK;
    }
    const int B = variants_chunk(D, n_windows);
    // workspace: V, out [B][D]; a1, h, a2, hd [B][H]; ml [B][2L]; the products' split partials,
    // for a full chunk and for the last, shorter one
    const int last = variants_last_rows(n_windows, B);
    const int64_t wsg = variants_gemm_workspace(B, last, D, H, L);
    // With M a power of two <= 32 the decoder-output product reduces v - m' in its epilogue
    // (per window, metric and column slot) instead of writing m'; `out` then holds those sums.
    const bool fused = M <= 32 && (M & (M - 1)) == 0;
    const bool decode = out_md || out_md_metric || out_recon;
    const int slots = fused ? std::max(gemm_reduce_slots(B, D), gemm_reduce_slots(last, D)) : 0;
    auto up4 = [](size_t v) { return (v + 3) / 4 * 4; };   // every sub-buffer 16-byte aligned
    const size_t nBD = up4(static_cast<size_t>(B) * D), nBH = up4(static_cast<size_t>(B) * H),
                 nML = up4(static_cast<size_t>(B) * 2 * L);
    const size_t nP = up4(static_cast<size_t>(B) * slots * M), nQ = up4(static_cast<size_t>(B) * slots);
    const size_t nOut = fused ? nP + nQ : nBD;
    const size_t nMap = up4(static_cast<size_t>(B));   // the chunk's window -> stream map (ints)
    const size_t need = nBD + nOut + 4 * nBH + nML + nMap + static_cast<size_t>(wsg) + 16;
    enova_status st = ensure(&det->ext_ws, &det->ext_ws_cap, need);
    if (st != ENOVA_OK)
        return st;
    float *V = det->ext_ws, *out = V + nBD, *a1 = out + nOut, *h = a1 + nBH, *a2 = h + nBH, *hd = a2 + nBH,
          *ml = hd + nBH, *mapf = ml + nML, *gw = mapf + nMap;
    int *wmap = reinterpret_cast<int *>(mapf);
    if (det->timing)
        (void)hipEventRecord(det->ext_ev[0], stream);
    if (norm == ENOVA_NORM_REFERENCE && !ref_mean) {
        size_t o_part = 0;
        st = ensure(&det->stats, &det->stats_cap, stats_floats(n, M, &o_part));
        if (st != ENOVA_OK)
            return st;
        ref_mean = det->stats;
        ref_std = det->stats + static_cast<size_t>(n) * M;
        double *part = stat_part_bytes(n, M) > 0 ? reinterpret_cast<double *>(det->stats + o_part) : nullptr;
        if ((e = launch_ref_stats(g, x, soff, n, det->stats, det->stats + static_cast<size_t>(n) * M, part,
                                  stream)) != hipSuccess)
            return hip_fail(e, "reference statistics kernel");
    }
    GemmEpilogue plain{};
    GemmEpilogue enc;
    enc.kind = kEpiBiasAct;
    enc.act = g.act;
    enc.bias = det->b1;
    enc.out2 = h;
    GemmEpilogue dec = enc;
    dec.bias = det->bd1;
    dec.out2 = hd;
    GemmEpilogue red;   // fused reductions of d = v - (product + bd2)
    red.kind = kEpiRowReduce;
    red.bias = det->d_bd2;
    red.pre = V;
    red.ldv = D;
    red.groups = M;
    red.out2 = out;
    red.sq = out + nP;
    for (int64_t w0 = 0; w0 < n_windows; w0 += B) {
        const int rows = static_cast<int>(std::min<int64_t>(B, n_windows - w0));
        e = launch_ext_stage(x, g.dtype, soff, woff, n, w0, rows, M, g.W, g.S, norm, ref_mean, ref_std, wmap, V,
                             stream);
        if (e == hipSuccess)   // a1 = V W1^T + b1, h = act(a1)
            e = launch_gemm(enc, V, D, 1, det->d_w1, 1, D, a1, H, rows, H, D, nullptr, gw, wsg, stream);
        if (e == hipSuccess)   // [mu | lv] = h [Wmu; Wlv]^T
            e = launch_gemm(plain, h, H, 1, det->d_wml, 1, H, ml, 2 * L, rows, 2 * L, H, nullptr, gw, wsg, stream);
        if (e == hipSuccess)
            e = launch_ext_latent(ml, det->d_bml, rows, L, out_scores ? out_scores + w0 : nullptr, stream);
        if (e != hipSuccess)
            return hip_fail(e, "output-variant kernels");
        if (!decode)   // only scores requested: the decoder is not needed
            continue;
        if (e == hipSuccess)   // a2 = mu Wd1^T + bd1, hd = act(a2)
            e = launch_gemm(dec, ml, 2 * L, 1, det->d_wd1, 1, L, a2, H, rows, H, L, nullptr, gw, wsg, stream);
        float *o_md = out_md ? out_md + w0 : nullptr, *o_mdm = out_md_metric ? out_md_metric + w0 * M : nullptr,
              *o_rec = out_recon ? out_recon + w0 : nullptr;
        if (fused) {
            if (e == hipSuccess)   // decoder output, reduced against V in the epilogue
                e = launch_gemm(red, hd, H, 1, det->d_wd2, 1, H, out, D, rows, D, H, nullptr, gw, wsg, stream);
            if (e == hipSuccess)
                e = launch_ext_finish(out, out + nP, rows, gemm_reduce_slots(rows, D), M, g.W, o_md, o_mdm, o_rec,
                                      stream);
        } else {
            if (e == hipSuccess)   // decoder output without bd2
                e = launch_gemm(plain, hd, H, 1, det->d_wd2, 1, H, out, D, rows, D, H, nullptr, gw, wsg, stream);
            if (e == hipSuccess)
                e = launch_ext_reduce(V, out, det->d_bd2, rows, M, g.W, o_md, o_mdm, o_rec, stream);
        }
        if (e != hipSuccess)
            return hip_fail(e, "output-variant kernels");
    }
    if (det->timing)
        (void)hipEventRecord(det->ext_ev[1], stream);
    det->ran_ext = true;
    return ENOVA_OK;
}

enova_status enova_detect_ext_time(enova_detector det, double *ms)
{
    if (!det || !ms)
        return fail(ENOVA_EINVAL, "NULL argument");
    *ms = 0.0;
    if (!det->timing || !det->ran_ext || !det->ext_ev[1])
        return ENOVA_OK;
    DeviceGuard dg(det->device);
    hipError_t e = hipEventSynchronize(det->ext_ev[1]);
    float f = 0.0f;
    if (e == hipSuccess)
        e = hipEventElapsedTime(&f, det->ext_ev[0], det->ext_ev[1]);
    if (e != hipSuccess)
        return hip_fail(e, "event timing");
    *ms = f;
    return ENOVA_OK;
}

enova_status enova_detect_flag(enova_detector det, const float *scores, int64_t n_windows,
                               float threshold, uint8_t *out_flags, hipStream_t stream)
{
    if (!det)
        return fail(ENOVA_EINVAL, "detector is NULL");
    if (n_windows < 0)
        return fail(ENOVA_EINVAL, "n_windows < 0");
    if (n_windows == 0)
        return ENOVA_OK;
    if (!scores || !out_flags)
        return fail(ENOVA_EINVAL, "NULL argument");
    DeviceGuard dg(det->device);
    hipError_t e = launch_flag(scores, n_windows, threshold, out_flags, stream);
    if (e != hipSuccess)
        return hip_fail(e, "flag kernel");
    return ENOVA_OK;
}

enova_status enova_detect_threshold(enova_detector det, const float *scores, const int64_t *soff,
                                    const int64_t *woff, int32_t n, int64_t n_windows, double level,
                                    double q, float *out_threshold, double *out_info,
                                    uint8_t *out_flags, hipStream_t stream)
{
    if (!det)
        return fail(ENOVA_EINVAL, "detector is NULL");
    if (!out_threshold)
        return fail(ENOVA_EINVAL, "out_threshold is NULL");
    if (!(level > 0.0 && level < 1.0) || !(q > 0.0 && q < 1.0))
        return fail(ENOVA_EINVAL, "level and q must lie in (0, 1)");
    if (n < 0 || n_windows < 0)
        return fail(ENOVA_EINVAL, "n_streams and n_windows must be >= 0");
    if (n == 0 || n_windows == 0)
        return fail(ENOVA_ESHAPE, "no windows to calibrate on");
    if (!scores || !soff || !woff)
        return fail(ENOVA_EINVAL, "NULL argument");
    DeviceGuard dg(det->device);
    const Geometry &g = det->g;
    enova_status st = ensure(&det->cal, &det->cal_cap, static_cast<size_t>(n) + 1);
    const size_t nblk = static_cast<size_t>(pot_blocks(n_windows));
    if (st == ENOVA_OK)
        st = ensure(&det->blk, &det->blk_cap, 2 * nblk);
    if (st == ENOVA_OK && !det->pot) {
        const hipError_t e = hipMalloc(reinterpret_cast<void **>(&det->pot), sizeof(PotState));
        if (e != hipSuccess) {
            det->pot = nullptr;
            return fail(ENOVA_ENOMEM, "hipMalloc(%zu): %s", sizeof(PotState), hipGetErrorString(e));
        }
    }
    if (st == ENOVA_OK && !det->pot_out &&
        hipHostMalloc(reinterpret_cast<void **>(&det->pot_out), sizeof(PotOut)) != hipSuccess) {
        det->pot_out = nullptr;
        return fail(ENOVA_ENOMEM, "pinned host memory of the threshold's result");
    }
    if (st != ENOVA_OK)
        return st;
    PotWork w{det->pot, det->cal, det->blk, det->blk + nblk, nullptr, nullptr, 0};
    hipError_t e = launch_pot_select(g, scores, soff, woff, n, n_windows, level, w, stream);
    if (e != hipSuccess)
        return hip_fail(e, "level quantile kernels");
    // at most (1 - level) of the calibration scores lie above the level quantile; the windows bound
    // their number, and where that would be much memory the number itself is read back
    int64_t n_cal = n_windows;
    if ((1.0 - level) * static_cast<double>(n_windows) > 0x1p24) {
        if ((e = hipMemcpyAsync(&n_cal, &det->pot->n_cal, sizeof(int64_t), hipMemcpyDeviceToHost, stream)) != hipSuccess ||
            (e = hipStreamSynchronize(stream)) != hipSuccess)
            return hip_fail(e, "calibration count");
        if (n_cal <= 0)
            return fail(ENOVA_ESHAPE, "no window lies inside a reference prefix");
    }
    w.cap = static_cast<int64_t>((1.0 - level) * static_cast<double>(n_cal)) + 2;
    if ((st = ensure(&det->peaks, &det->peaks_cap, static_cast<size_t>(w.cap))) != ENOVA_OK ||
        (st = ensure(&det->pot_part, &det->pot_part_cap, static_cast<size_t>(kPotPartDoubles))) != ENOVA_OK)
        return st;
    w.y = det->peaks;
    w.part = det->pot_part;
    if ((e = launch_pot_peaks(scores, woff, n, n_windows, q, w, stream)) != hipSuccess)
        return hip_fail(e, "peak kernels");
    // the grid, Newton steps and the candidates: five rounds end nearly every fit, the flags then
    // follow at once; a fit that needs more gets them two at a time
    PotOut *r = det->pot_out;
    for (int rounds = 5;; rounds = 2) {
        if ((e = launch_pot_rounds(rounds, q, w, stream)) != hipSuccess ||
            (e = launch_pot_flag(scores, n_windows, w, r, out_flags, stream)) != hipSuccess ||
            (e = hipStreamSynchronize(stream)) != hipSuccess)
            return hip_fail(e, "tail fit kernels");
        switch (r->err) {
        case 0: break;
        case kPotNoWindows: return fail(ENOVA_ESHAPE, "no window lies inside a reference prefix");
        case kPotLost: return fail(ENOVA_EHIP, "radix select lost the order statistic");
        case kPotLevelNotFinite:
            return fail(ENOVA_ENUMERIC, "non-finite calibration score at the level quantile");
        case kPotCount: return fail(ENOVA_EHIP, "peak count mismatch (%lld)", static_cast<long long>(r->n_peaks));
        default: return fail(ENOVA_ENUMERIC, "non-finite calibration score");
        }
        if (r->phase == kPotDone)
            break;
    }
    *out_threshold = static_cast<float>(r->z);
    if (out_info) {
        out_info[0] = r->t;
        out_info[1] = static_cast<double>(r->n_cal);
        out_info[2] = static_cast<double>(r->n_peaks);
        out_info[3] = r->gamma;
        out_info[4] = r->sigma;
        out_info[5] = r->method;
    }
    return ENOVA_OK;
}

enova_status enova_detect_set_timing(enova_detector det, int32_t enable)
{
    if (!det)
        return fail(ENOVA_EINVAL, "detector is NULL");
    det->timing = enable != 0;
    return ENOVA_OK;
}

enova_status enova_detect_kernel_times(enova_detector det, double *score_ms, double *stats_ms)
{
    if (!det)
        return fail(ENOVA_EINVAL, "detector is NULL");
    DeviceGuard dg(det->device);
    float a = 0.0f, b = 0.0f;
    hipError_t e;
    if (det->timing && det->ran_score && det->ev[2]) {
        if ((e = hipEventSynchronize(det->ev[3])) != hipSuccess ||
            (e = hipEventElapsedTime(&a, det->ev[2], det->ev[3])) != hipSuccess)
            return hip_fail(e, "score kernel timing");
    }
    if (det->timing && det->ran_stats && det->ev[0]) {
        if ((e = hipEventSynchronize(det->ev[1])) != hipSuccess ||
            (e = hipEventElapsedTime(&b, det->ev[0], det->ev[1])) != hipSuccess)
            return hip_fail(e, "stats kernel timing");
    }
    if (score_ms)
        *score_ms = a;
    if (stats_ms)
        *stats_ms = b;
    return ENOVA_OK;
}

enova_status enova_detect_ext_mode(enova_detector det, int32_t *fused)
{
    if (!det || !fused)
        return fail(ENOVA_EINVAL, "NULL argument");
    *fused = ext_fused_supported(det->g) && det->kind == 2 ? 1 : 0;
    return ENOVA_OK;
}

enova_status enova_detect_ext_route(enova_detector det, int32_t n_streams, int64_t n_windows, int32_t norm,
                                    int32_t *route)
{
    if (!det || !route)
        return fail(ENOVA_EINVAL, "NULL argument");
    if (n_streams < 0 || n_windows < 0)
        return fail(ENOVA_EINVAL, "n_streams and n_windows must be >= 0");
    if (norm != ENOVA_NORM_REFERENCE && norm != ENOVA_NORM_WINDOW)
        return fail(ENOVA_EINVAL, "bad normalisation mode");
    *route = ext_route(det, n_streams, n_windows, norm);
    return ENOVA_OK;
}

enova_status enova_detect_kernel_kind(enova_detector det, int32_t *kind)
{
    if (!det || !kind)
        return fail(ENOVA_EINVAL, "NULL argument");
    *kind = det->kind;
    return ENOVA_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------------------------
// Streaming detection
// ---------------------------------------------------------------------------------------------
struct enova_stream_s {
    enova_detector det = nullptr;
    int n = 0;
    int64_t steps = 0;            // steps pushed so far (the same for every stream)
    double q = 1e-3;
    void *ring = nullptr;         // [n][2W][M]
    float *mean = nullptr, *std = nullptr;   // [n][M]
    float *scores = nullptr;      // [n] when the caller does not ask for scores
    SpotState spot{};
    hipEvent_t ev[3] = {nullptr, nullptr, nullptr};   // score start, score end / spot start, spot end
    bool timed = false;           // the last scoring push recorded ev
    // the threshold update and the refit run on the set's own stream (default priority), so a
    // push's refit overlaps the next push's append and scoring: the update waits for the push's
    // scores (score_ev), `stream` waits for the update (upd_ev: flags written, scores read), and
    // a state read waits for the refit (fit_ev)
    hipStream_t fit_stream = nullptr;
    hipEvent_t score_ev = nullptr, upd_ev = nullptr, fit_ev = nullptr;
    bool fit_pending = false;
};

namespace {

void free_stream(enova_stream s)
{
    if (!s)
        return;
    void *ptrs[] = {s->ring, s->mean, s->std, s->scores, s->spot.t, s->spot.z, s->spot.cnt,
                    s->spot.npk, s->spot.peaks, s->spot.mark, s->spot.err, s->spot.list,
                    s->spot.count};
    for (void *p : ptrs)
        if (p)
            (void)hipFree(p);
    for (hipEvent_t e : s->ev)
        if (e)
            (void)hipEventDestroy(e);
    if (s->score_ev)
        (void)hipEventDestroy(s->score_ev);
    if (s->upd_ev)
        (void)hipEventDestroy(s->upd_ev);
    if (s->fit_ev)
        (void)hipEventDestroy(s->fit_ev);
    if (s->fit_stream)
        (void)hipStreamDestroy(s->fit_stream);
    delete s;
}

template <typename T>
enova_status dev_alloc(T **dst, size_t count)
{
    hipError_t e = hipMalloc(reinterpret_cast<void **>(dst), std::max<size_t>(count, 1) * sizeof(T));
    if (e != hipSuccess) {
        *dst = nullptr;
        return fail(ENOVA_ENOMEM, "hipMalloc(%zu): %s", count * sizeof(T), hipGetErrorString(e));
    }
    return ENOVA_OK;
}

}  // namespace

extern "C" {

enova_status enova_stream_create(enova_detector det, int32_t n, const float *ref_mean, const float *ref_std,
                                 const float *calib_scores, const int64_t *calib_offsets, double level,
                                 double q, int32_t peak_cap, enova_stream *out, hipStream_t stream)
{
    if (!det || !ref_mean || !ref_std || !calib_offsets || !out)
        return fail(ENOVA_EINVAL, "NULL argument");
    *out = nullptr;
    if (n < 1)
        return fail(ENOVA_EINVAL, "n_streams must be >= 1");
    if (!(level > 0.0 && level < 1.0) || !(q > 0.0 && q < 1.0))
        return fail(ENOVA_EINVAL, "level and q must lie in (0, 1)");
    if (peak_cap < 1)
        return fail(ENOVA_EINVAL, "peak_cap must be >= 1");
    if (calib_offsets[0] != 0)
        return fail(ENOVA_EINVAL, "calib_offsets[0] must be 0");
    for (int32_t i = 0; i < n; ++i)
        if (calib_offsets[i + 1] < calib_offsets[i])
            return fail(ENOVA_EINVAL, "calib_offsets must be non-decreasing");
    const int64_t n_cal = calib_offsets[n];
    if (n_cal > 0 && !calib_scores)
        return fail(ENOVA_EINVAL, "calib_scores is NULL");
    const Geometry &g = det->g;
    if (det->kind != 2 || !det->w1s)
        return fail(ENOVA_EUNSUPPORTED, "streaming needs the matrix-core kernel's shapes");
    DeviceGuard dg(det->device);
    hipError_t e = hipSuccess;

    enova_stream s = new (std::nothrow) enova_stream_s;
    if (!s)
        return fail(ENOVA_ENOMEM, "host allocation");
    s->det = det;
    s->n = n;
    s->q = q;
    const size_t esz = g.dtype == ENOVA_F32 ? 4 : 2;
    const size_t nm = static_cast<size_t>(n) * g.M;
    enova_status st = ENOVA_OK;
    int64_t *d_off = nullptr;
    if ((st = dev_alloc(reinterpret_cast<unsigned char **>(&s->ring), nm * 2 * g.W * esz)) != ENOVA_OK ||
        (st = dev_alloc(&s->mean, nm)) != ENOVA_OK || (st = dev_alloc(&s->std, nm)) != ENOVA_OK ||
        (st = dev_alloc(&s->scores, n)) != ENOVA_OK || (st = dev_alloc(&s->spot.t, n)) != ENOVA_OK ||
        (st = dev_alloc(&s->spot.z, n)) != ENOVA_OK || (st = dev_alloc(&s->spot.cnt, n)) != ENOVA_OK ||
        (st = dev_alloc(&s->spot.npk, n)) != ENOVA_OK ||
        (st = dev_alloc(&s->spot.peaks, static_cast<size_t>(n) * peak_cap)) != ENOVA_OK ||
        (st = dev_alloc(&s->spot.mark, n)) != ENOVA_OK || (st = dev_alloc(&s->spot.err, 1)) != ENOVA_OK ||
        (st = dev_alloc(&s->spot.list, n)) != ENOVA_OK || (st = dev_alloc(&s->spot.count, 2)) != ENOVA_OK ||
        (st = dev_alloc(&d_off, static_cast<size_t>(n) + 1)) != ENOVA_OK) {
        (void)hipFree(d_off);
        free_stream(s);
        return st;
    }
    s->spot.cap = peak_cap;
    int err = 0;
    if ((e = hipMemsetAsync(s->ring, 0, nm * 2 * g.W * esz, stream)) != hipSuccess ||
        (e = hipMemcpyAsync(s->mean, ref_mean, nm * sizeof(float), hipMemcpyDeviceToDevice, stream)) != hipSuccess ||
        (e = hipMemcpyAsync(s->std, ref_std, nm * sizeof(float), hipMemcpyDeviceToDevice, stream)) != hipSuccess ||
        (e = hipMemsetAsync(s->spot.err, 0, sizeof(int), stream)) != hipSuccess ||
        (e = hipMemsetAsync(s->spot.count, 0, 2 * sizeof(int), stream)) != hipSuccess ||
        (e = hipMemcpyAsync(d_off, calib_offsets, (static_cast<size_t>(n) + 1) * sizeof(int64_t),
                            hipMemcpyHostToDevice, stream)) != hipSuccess ||
        (e = launch_spot_init(n_cal > 0 ? calib_scores : s->scores, d_off, n, level, s->spot, stream)) != hipSuccess ||
        (e = hipMemcpyAsync(&err, s->spot.err, sizeof(int), hipMemcpyDeviceToHost, stream)) != hipSuccess ||
        (e = hipStreamSynchronize(stream)) != hipSuccess) {
        (void)hipFree(d_off);
        free_stream(s);
        return hip_fail(e, "streaming set start");
    }
    (void)hipFree(d_off);
    if (err == 2) {
        free_stream(s);
        return fail(ENOVA_ENUMERIC, "non-finite calibration score");
    }
    if (err == 1) {
        free_stream(s);
        return fail(ENOVA_EINVAL, "a stream's calibration peaks exceed peak_cap");
    }
    if ((e = launch_spot_fit(n, q, s->spot, true, stream)) != hipSuccess || (e = hipStreamSynchronize(stream)) != hipSuccess) {
        free_stream(s);
        return hip_fail(e, "streaming threshold fit");
    }
    *out = s;
    return ENOVA_OK;
}

enova_status enova_stream_push(enova_stream s, const void *x_step, float *out_scores, float *out_md,
                               uint8_t *out_flags, int32_t *out_due, hipStream_t stream)
{
    if (!s || !x_step)
        return fail(ENOVA_EINVAL, "NULL argument");
    enova_detector det = s->det;
    const Geometry &g = det->g;
    DeviceGuard dg(det->device);
    hipError_t e = launch_stream_append(g, x_step, s->n, s->steps, s->ring, stream);
    if (e != hipSuccess)
        return hip_fail(e, "streaming append kernel");
    s->steps += 1;
    const bool due = s->steps >= g.W && (s->steps - g.W) % g.S == 0;
    if (out_due)
        *out_due = due ? 1 : 0;
    if (!due)
        return ENOVA_OK;
    StreamScoreParams p{};
    p.ring = s->ring;
    p.n_streams = s->n;
    p.first_slot = static_cast<int>(s->steps % g.W);
    p.mean = s->mean;
    p.std = s->std;
    p.w1p = det->w1s;
    p.whp = det->whs;
    p.wd1p = det->wds;
    p.b1 = det->b1;
    p.bd1 = det->bd1;
    p.u = det->u;
    p.bh = det->bh;
    p.sum_bd2 = det->sum_bd2;
    p.scores = out_scores ? out_scores : s->scores;
    p.md = out_md;
    const bool timed = det->timing;
    if (timed && !s->ev[0]) {
        for (hipEvent_t &ev : s->ev)
            if ((e = hipEventCreate(&ev)) != hipSuccess)
                return hip_fail(e, "timing events");
    }
    if (timed)
        (void)hipEventRecord(s->ev[0], stream);
    if ((e = launch_stream_score(g, p, stream)) != hipSuccess)
        return hip_fail(e, "streaming scoring kernel");
    if (timed)
        (void)hipEventRecord(s->ev[1], stream);
    if (!s->fit_stream) {
        if ((e = hipStreamCreateWithFlags(&s->fit_stream, hipStreamNonBlocking)) != hipSuccess ||
            (e = hipEventCreateWithFlags(&s->score_ev, hipEventDisableTiming)) != hipSuccess ||
            (e = hipEventCreateWithFlags(&s->upd_ev, hipEventDisableTiming)) != hipSuccess ||
            (e = hipEventCreateWithFlags(&s->fit_ev, hipEventDisableTiming)) != hipSuccess)
            return hip_fail(e, "streaming refit stream");
    }
    // on the set's stream, behind the previous push's refit (whose thresholds it compares with,
    // and whose peaks, counts and list it rewrites): this push's update, then its refit, which
    // overlaps the next push's append and scoring on `stream`
    if ((e = hipEventRecord(s->score_ev, stream)) != hipSuccess ||
        (e = hipStreamWaitEvent(s->fit_stream, s->score_ev, 0)) != hipSuccess)
        return hip_fail(e, "streaming threshold order");
    s->spot.cur ^= 1;   // this push's list counter (cleared by the previous push's refit)
    if ((e = launch_spot_update(p.scores, s->n, s->spot, out_flags, s->fit_stream)) != hipSuccess)
        return hip_fail(e, "streaming threshold update");
    if ((e = hipEventRecord(s->upd_ev, s->fit_stream)) != hipSuccess ||
        (e = launch_spot_fit(s->n, s->q, s->spot, false, s->fit_stream)) != hipSuccess ||
        (e = hipEventRecord(s->fit_ev, s->fit_stream)) != hipSuccess)
        return hip_fail(e, "streaming refit");
    if (timed)
        (void)hipEventRecord(s->ev[2], s->fit_stream);
    // later work on `stream` sees this push's flags, and may overwrite the scores the update read
    if ((e = hipStreamWaitEvent(stream, s->upd_ev, 0)) != hipSuccess)
        return hip_fail(e, "streaming threshold order");
    s->fit_pending = true;
    s->timed = timed;
    return ENOVA_OK;
}

enova_status enova_stream_state(enova_stream s, double *t, double *z, int64_t *n, int32_t *n_peaks,
                                hipStream_t stream)
{
    if (!s)
        return fail(ENOVA_EINVAL, "NULL argument");
    DeviceGuard dg(s->det->device);
    const size_t k = static_cast<size_t>(s->n);
    hipError_t e = hipSuccess;
    if (s->fit_pending && (e = hipStreamWaitEvent(stream, s->fit_ev, 0)) != hipSuccess)
        return hip_fail(e, "streaming refit wait");
    if ((t && (e = hipMemcpyAsync(t, s->spot.t, k * sizeof(double), hipMemcpyDeviceToHost, stream)) != hipSuccess) ||
        (z && (e = hipMemcpyAsync(z, s->spot.z, k * sizeof(double), hipMemcpyDeviceToHost, stream)) != hipSuccess) ||
        (n && (e = hipMemcpyAsync(n, s->spot.cnt, k * sizeof(int64_t), hipMemcpyDeviceToHost, stream)) != hipSuccess) ||
        (n_peaks && (e = hipMemcpyAsync(n_peaks, s->spot.npk, k * sizeof(int32_t), hipMemcpyDeviceToHost, stream)) != hipSuccess) ||
        (e = hipStreamSynchronize(stream)) != hipSuccess)
        return hip_fail(e, "streaming state copy");
    return ENOVA_OK;
}

enova_status enova_stream_kernel_times(enova_stream s, double *score_ms, double *spot_ms)
{
    if (!s)
        return fail(ENOVA_EINVAL, "NULL argument");
    DeviceGuard dg(s->det->device);
    float a = 0.0f, b = 0.0f;
    hipError_t e;
    if (s->timed) {
        if ((e = hipEventSynchronize(s->ev[2])) != hipSuccess ||
            (e = hipEventElapsedTime(&a, s->ev[0], s->ev[1])) != hipSuccess ||
            (e = hipEventElapsedTime(&b, s->ev[1], s->ev[2])) != hipSuccess)
            return hip_fail(e, "streaming kernel timing");
    }
    if (score_ms)
        *score_ms = a;
    if (spot_ms)
        *spot_ms = b;
    return ENOVA_OK;
}

enova_status enova_stream_destroy(enova_stream s)
{
    if (!s)
        return ENOVA_OK;
    DeviceGuard dg(s->det->device);
    (void)hipDeviceSynchronize();
    free_stream(s);
    return ENOVA_OK;
}

}  // extern "C"
