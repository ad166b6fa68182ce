// C ABI of the library (see include/rtn.h): argument validation, kernel-plan selection,
// selective-precision dispatch.  No device code here.
#include "../../include/rtn.h"
#include "rtn_internal.h"
#include <vector>
#include <algorithm>
#include <cmath>
#include <mutex>

#include <stdlib.h>
#include <string.h>

using rtn::LinearArgs;
using rtn::LinearPlan;

namespace {

constexpr size_t kWorkspaceCap = (size_t)16 << 20;     // split-K partials never exceed this ...
constexpr size_t kWorkspaceCapTall = (size_t)64 << 20; // ... except under the plans of path 3 from 64 rows (and the tile kernel's)
constexpr int kMaxSplitK = 16;

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }

int chunk_k(int bits) { return bits == 4 ? 512 : 256; }
int tile_k(int bits) { return bits == 4 ? 128 : 64; }

// Normalises group_size (<= 0 or K means per-channel) and checks it.
rtn_status check_problem(int64_t N, int64_t K, int bits, int group_size, int64_t* g_out) {
    if (bits != 4 && bits != 8) return RTN_ERR_BITS;
    if (N <= 0 || K <= 0 || N % 16 != 0 || K % chunk_k(bits) != 0) return RTN_ERR_SHAPE;
    // K < 2^23: the kernels divide k-step and chunk indices by the group length with a multiply-high by
    // floor(2^32 / d) + 1, exact while index * d < 2^32
    if (N > (int64_t)1 << 30 || K >= (int64_t)1 << 23) return RTN_ERR_SHAPE;
    int64_t g = (group_size <= 0) ? K : group_size;
    if (g > K || K % g != 0) return RTN_ERR_GROUP;
    const int ck = chunk_k(bits), tk = tile_k(bits);
    if (g < ck) {                                   // 32, 64, ... up to a k-chunk: a power-of-two number of groups per chunk
        if (g != 32 && g != 64 && g != tk && g != 2 * tk && g != 4 * tk) return RTN_ERR_GROUP;
    } else if (g % ck != 0) {
        return RTN_ERR_GROUP;
    }
    *g_out = g;
    return RTN_OK;
}

size_t workspace_bound(int64_t M, int64_t N) {
    size_t one = (size_t)M * (size_t)N * sizeof(float);
    size_t want = one * kMaxSplitK;
    if (want > kWorkspaceCap) want = kWorkspaceCap;
    if (want < 256) want = 256;
    return (want + 255) & ~(size_t)255;
}

int device_max_lds() {
    static int cached = 0;
    if (cached == 0) {
        int v = 0, dev = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess && v > 0)
            cached = v < (int)rtn::kMaxLdsBytes ? v : (int)rtn::kMaxLdsBytes;
        else
            cached = (int)rtn::kMaxLdsBytes;   // no device to ask (host-only planning): the gfx950 figure
    }
    return cached;
}

int round_pow2(int64_t v, int lo, int hi) {
    int p = lo;
    while (p * 2 <= hi && (int64_t)p * 3 / 2 <= v) p *= 2;     // nearest power of two in the log sense
    return p;
}

// Default plan, from configuration sweeps on MI355X.  Short-lived wavefronts at high
// occupancy stream best: a wavefront gets 1-4 k-chunks (4-16 KiB of packed weights) of one tile-row
// and K is split inside the workgroup (reduced through LDS).  With more than two activation rows the
// staged slice grows, so workgroups widen along N (sharing it) and, for long K, K is also split across
// workgroups so that a slice stays a few chunks long; those partials go through the workspace.
// (That is modelled_plan's last part, for the skinny kernel; before it come the models of the other kernels.)

// A fixed shape of path 3 for more than 16 rows: the candidate (wavefronts per workgroup, tile-rows per wavefront, K
// splits) with the lowest time in a model of a wide kernel that walked K in steps of its own for every shape.  Automatic
// plans come from block_or_wide_plan below.  This one stands where a caller's program would notice if it moved: it completes
// explicit configurations that leave fields open, it draws the line up to which a problem keeps its exact codes and
// what rtn_linear_noalloc accepts (wide_or_tile_plan), and the small groups' models were fitted to its shapes.
// The model is the larger of three streaming / arithmetic times -- activations re-read from L2 once per workgroup column
// plus the weights, the weights from HBM, the MFMA work -- derated by how evenly the workgroups fill the compute units, plus
// fixed per-launch, per-round and split-K reduction costs.
double wide_model_us(int64_t M, int64_t N, int64_t K, int bits, int mb, int wv, int nbw, int s) {
    const double kL2 = 11.26e12, kHbm = 6.96e12, kMfma = 1.02e15, kSmallTile = 0.767, kFix = 2e-6, kRound = 1.5e-6;
    const double kReduce0 = 2.5e-6, kReduceBw = 4.55e12, kUtilExp = 0.662;
    const int64_t rows = 16 * mb, ZB = (M + rows - 1) / rows, n_wg = 16 * nbw * wv, XB = (N + n_wg - 1) / n_wg;
    const int64_t wgs = XB * ZB * s, slots = 256 * (wv == 4 ? 3 : 1);
    const int64_t rounds = (wgs + slots - 1) / slots;
    const double util = (double)wgs / (double)(rounds * slots);
    const double Mp = (double)(ZB * rows), wbytes = (double)N * K * bits / 8.0;
    const double t_l2 = (2.0 * Mp * K * XB + wbytes * std::sqrt((double)ZB)) / kL2;
    const double t_hbm = wbytes * 1.03 / kHbm;
    const double t_mfma = 2.0 * Mp * N * K / (kMfma * (nbw * mb >= 8 ? 1.0 : kSmallTile));
    double t = std::max(t_l2, std::max(t_hbm, t_mfma)) / std::pow(util, kUtilExp) + kFix + rounds * kRound;
    if (s > 1) t += kReduce0 + 2.0 * s * M * N * 4.0 / kReduceBw;
    return t * 1e6;
}

void wide_plan(int64_t M, int64_t N, int64_t K, int bits, int64_t g, LinearPlan* p) {
    p->path = 3;
    p->m_rows16 = M <= 32 ? 2 : (M <= 48 ? 3 : 4);
    // 48-row blocks above 64 rows where they save a fifth of the padded rows (65-96 and 129-144 rows: 96 against 128,
    // 144 against 192).
    // Workgroup shape and K split are still the ones modelled for 64-row blocks.
    const bool blocks48 = M > 64 && ((M + 47) / 48) * 48 * 5 <= ((M + 63) / 64) * 64 * 4;
    p->m_blocks = (int)((M + 16 * p->m_rows16 - 1) / (16 * p->m_rows16));
    p->prefetch = 1; p->waves_k = 1;
    const int64_t KS = K / 128;
    // groups under 128 columns keep to the small bound at every M: rtn_linear_noalloc serves them all
    int64_t smax = (int64_t)((M >= 64 && g % 128 == 0 ? kWorkspaceCapTall : kWorkspaceCap) / ((size_t)M * N * sizeof(float)));
    if (smax > kMaxSplitK) smax = kMaxSplitK;
    if (smax > KS / 4) smax = KS / 4;
    if (smax < 1) smax = 1;
    // three splits (they fill the compute units where two leave a third idle and four start a second round) compete
    // with the powers of two; other splits are taken only when the model puts them 5 % ahead
    double best = 1e30, best_any = 1e30;
    LinearPlan any = *p;
    for (int wv = 4; wv <= 16; wv *= 2)
        for (int nbw = 1; nbw <= 4; nbw *= 2) {
            if (p->m_rows16 * nbw > 8 || (wv == 16 && nbw > 1)) continue;
            if (g % 128 != 0 && (wv != 8 || nbw > 2)) continue;     // the shapes built for groups of 32 and 64 columns
            for (int s = 1; s <= smax; ++s) {
                const double t = wide_model_us(M, N, K, bits, p->m_rows16, wv, nbw, s);
                if (((s & (s - 1)) == 0 || s == 3) && t < best) {
                    best = t;
                    p->waves_n = wv; p->n_tiles16 = nbw; p->split_k = s;
                }
                if (t < best_any) {
                    best_any = t;
                    any.waves_n = wv; any.n_tiles16 = nbw; any.split_k = s;
                }
            }
        }
    if (best_any < 0.95 * best) {
        p->waves_n = any.waves_n; p->n_tiles16 = any.n_tiles16; p->split_k = any.split_k;
    }
    if (blocks48) {
        p->m_rows16 = 3;
        p->m_blocks = (int)((M + 47) / 48);
    }
}

// The block kernel's time, as two models have it.  The first: a workgroup has a fixed start, so much per unit of four packed tiles
// that each of its wavefronts along K runs (by 32-row blocks; the scales cost per group and block), the sum over the wavefronts along
// K; slower by up to a third on a busy chip, whose clock falls.  Workgroups come in rounds of one per compute unit (two of the 32-row
// ones), of the fullest XCD.  Against it the stream of weights at 6.8 TB/s and of activations from L2 at 17 TB/s.  Fitted to 5300
// launches on sixteen shapes of 1024 to 57344 columns, 20 to 512 rows, int4 and int8, groups of 64, 128 and K.
struct BlockTimes {
    int mb;             // row blocks of 32 rows
    int64_t wgs;        // workgroups
    double wg_us;       // one workgroup on an idle chip
    double stream_us;   // its weights and activations at the rates above
};

double block_wg_us(int mb, int64_t K, int bits, int64_t g, int wk, int s) {
    static const double kUnit[4] = {1.93, 2.25, 2.49, 2.77}, kGroup[4] = {0.044, 0.123, 0.269, 0.382};
    const int64_t unit = bits == 4 ? 512 : 256, units = K / unit;
    const double per = (double)(((units + s - 1) / s + wk - 1) / wk), groups = g >= unit ? 1.0 : (double)(unit / g);
    return 1.33 + per * (kUnit[mb - 1] * (bits == 8 ? 0.675 : 1.0) + kGroup[mb - 1] * groups) + (wk > 1 ? 0.73 * mb : 0.0);
}

BlockTimes block_times(int64_t M, int64_t N, int64_t K, int bits, int64_t g, int rows16, int wk, int s) {
    const int64_t cols = 256 / wk;
    const int64_t ZB = (M + 16 * rows16 - 1) / (16 * rows16), XB = (N + cols - 1) / cols;
    BlockTimes b;
    b.mb = (int)((M + 32 * ZB - 1) / (32 * ZB));
    b.wgs = XB * ZB * s;
    b.wg_us = block_wg_us(b.mb, K, bits, g, wk, s);
    b.stream_us = (double)N * K * bits / 8.0 / 6.83e6 + (double)XB * ZB * 32 * b.mb * K * 2.0 / 1.71e7;
    return b;
}

// Rounds of workgroups (slots of them on the fullest XCD at once) in times of the tallest ones, of mb blocks; those of a block less take
// `low` of that and start last: whole rounds and the mean.  As if all were tall 28672 x 4096 at 300 rows, 128 + 96 + 96, went out in
// 64-row tiles: 88 us, 83 this way; 20000 x 5120 at 400 rows 108 and 93, 57344 x 8192 at 200 rows 215 and 193.  A 32-row tile is taken as
// long as a 64-row one: it unpacks as much, and where the model had it shorter a round that low tiles began looked cheap (16384 x 16384
// int8 group 64 at 160 rows in 384 workgroups 172 us, in 192 of twice the length 142; 8192 x 8192 int4 at 521 rows 97 and 84).
// Of 250 plans that two heights change in 12000 drawn problems 111 are more than 2 % faster than the plan for one, 4 more than 2 %
// slower (5 % at most); with the models' own ratio 67 were, up to 22 %.
// How the model has had row tiles.  The earlier ones draw the line to the tile kernel alone: a problem that ran on exact codes by any
// of them keeps them (modelled_plan).
enum Picture : int { kLaunched, kOneHeight, kTwoHeights };      // kTwoHeights: 32-row tiles shorter too, an order over the XCDs for each part
void block_rounds(int64_t M, int64_t N, int mb, int wk, int s, double slots, double low, Picture picture, double equal, double* whole, double* mean) {
    if (picture == kOneHeight) {
        *mean = equal;
        *whole = std::ceil(equal);
        return;
    }
    const rtn::BlockTiles tiles = rtn::block_tiles(M, N, mb, wk, s);
    const rtn::BlockParts p = rtn::block_parts(tiles, mb, tiles.workgroups() <= 256);
    auto on_xcd = [&](int i) {                                                    // (none in a part that is not there)
        if (picture == kLaunched || p.n == 1) return (double)p.part[i].on_xcd;
        const int64_t rows = p.part[i].rows, sliced = (tiles.columns * rows + 7) / 8 * s, dealt = (tiles.columns + 7) / 8 * rows * s;
        return (double)(rtn::xcd_slices_save_a_round(tiles.columns, rows, s) ? sliced : dealt);
    };
    const double t = on_xcd(0), l = on_xcd(1), of_tall = std::ceil(t / slots);
    *whole = of_tall + (std::ceil((t + l) / slots) - of_tall) * low;
    *mean = (t + l * low) / slots;
}

double block_near_us(int64_t M, int64_t N, int64_t K, int bits, int64_t g, int rows16, int wk, int s, Picture picture) {
    const BlockTimes b = block_times(M, N, K, bits, g, rows16, wk, s);
    const double wg = b.wg_us * (1.0 + 0.36 * std::min(1.0, (double)b.wgs / 256.0) * b.mb / 4.0);
    const double slots = 32.0 * (b.mb == 1 && wk <= 4 ? 2 : 1), low = b.mb <= (picture == kTwoHeights ? 1 : 2) ? 1.0 : block_wg_us(b.mb - 1, K, bits, g, wk, s) / b.wg_us;
    double whole, mean;
    block_rounds(M, N, b.mb, wk, s, slots, low, picture, std::ceil((double)b.wgs / 8.0) / slots, &whole, &mean);
    double serial = wg * std::max(1.0, 0.91 * whole + 0.09 * mean);
    if (slots > 32.0 && b.wgs > 256) serial *= 1.78;
    return 2.93 + std::cbrt(serial * serial * serial + b.stream_us * b.stream_us * b.stream_us) +
           (s > 1 ? 1.12 + (double)M * N * s * 8.0 / 4.19e6 : 0.0);
}

// The second, for few columns, long rows and many rows too: a workgroup has a start, and the larger part (a 3/2-norm) of what its
// wavefronts along K run and of what one compute unit can fetch, which holds back few columns under long rows (each of eight
// wavefronts along K has activations of its own); two 32-row ones on a compute unit are each slower by two thirds.  Against it
// (a 4-norm) the stream from HBM, what the XCDs that have a workgroup fetch (all activations each: a matrix of few columns
// leaves most of them idle) and what they read from their L2.  The reduce pass of a K split costs more above eight splits (its
// kernel goes round).  Fitted to 78000 launches: 1394 problems of 17 to 4096 rows, 128 to 106496 columns of 512 to 53248.
double block_far_us(int64_t M, int64_t N, int64_t K, int bits, int64_t g, int rows16, int wk, int s, Picture picture) {
    static const double kUnit[4][4] = {{1.791, 1.971, 2.149, 2.810}, {2.437, 2.819, 3.048, 3.392}, {3.418, 3.411, 4.144, 4.144}, {3.948, 4.007, 4.956, 4.956}};
    static const double kGroup[4] = {0.062, 0.091, 0.044, 0.103};
    const int64_t unit = bits == 4 ? 512 : 256, units = K / unit, cols = 256 / wk;
    const int64_t ZB = (M + 16 * rows16 - 1) / (16 * rows16), XB = (N + cols - 1) / cols;
    const int mb = (int)((M + 32 * ZB - 1) / (32 * ZB));
    const bool sliced = rtn::xcd_slices_save_a_round(XB, ZB, s), two = mb == 1 && wk <= 4;
    const double on_xcd = (double)((sliced ? (XB * ZB + 7) / 8 : (XB + 7) / 8 * ZB) * s), xcds = sliced ? 8.0 : (double)std::min<int64_t>(XB, 8);
    const int64_t share = (units + s - 1) / s, per = (share + wk - 1) / wk;
    const double groups = g >= unit ? 1.0 : (double)(unit / g), weights = (double)N * K * bits / 8.0, rows = (double)M * K * 2.0;
    const double run = (double)per * (kUnit[mb - 1][wk == 1 ? 0 : wk == 2 ? 1 : wk == 4 ? 2 : 3] * (bits == 8 ? 0.541 : 1.0) + kGroup[mb - 1] * groups) *
                       (1.0 + 0.376 * std::min(1.0, (double)(XB * ZB * s) / 256.0) * mb / 4.0);
    const double a_bytes = 32.0 * mb * share * unit * 2.0, w_bytes = (double)cols * share * unit * bits / 8.0;
    const double fetch = 0.543 * (a_bytes + w_bytes) / 1e5, both = run * std::sqrt(run) + fetch * std::sqrt(fetch);
    const double wg = 0.511 + std::cbrt(both * both) + (wk > 1 ? 0.484 * mb : 0.0);
    double whole, mean;
    const int w = wk == 1 ? 0 : wk == 2 ? 1 : wk == 4 ? 2 : 3;
    // (8 bit: no less than the other model has it, which the measurements agree with: 16480 x 10752 at 147 rows 100 us split in three, 84 unsplit)
    const double other = bits == 8 && mb > 2 && picture == kLaunched ? block_wg_us(mb - 1, K, bits, g, wk, s) / block_wg_us(mb, K, bits, g, wk, s) : 0.0;
    const double low = mb <= (picture == kTwoHeights ? 1 : 2) ? 1.0 : std::max(kUnit[mb - 2][w] / kUnit[mb - 1][w], other);
    block_rounds(M, N, mb, wk, s, two ? 64.0 : 32.0, low, picture, on_xcd / (two ? 64.0 : 32.0), &whole, &mean);
    const double serial = wg * std::max(1.0, 0.774 * whole + 0.226 * mean) * (two && on_xcd > 32.0 ? 1.667 : 1.0);
    const double hbm = 1.195 * (weights + rows) / 6.83e6, fabric = 0.530 * (rows + weights / xcds) / 1e6;
    const double l2 = 0.812 * on_xcd * (a_bytes + 1.550 * w_bytes) / 2e6;
    auto to4 = [](double x) { return x * x * x * x; };
    double t = 3.218 + std::sqrt(std::sqrt(to4(serial) + to4(hbm) + to4(fabric) + to4(l2))) + 3.413 * (double)M * N * 2.0 / 1e7;
    if (s > 1) t += 2.394 + 0.734 * (double)M * N * s * 8.0 / 4.19e6 + (s > 8 ? 1.971 : 0.0);
    return t;
}

// Below 1024 columns and above 512 rows the second alone: the best measured plan is 1.5 % and 0.7 % ahead of its pick on average
// (of the first's 6 % and 3 %, up to 64 % on few columns under long rows: 394 rows of 400 x 43008 66 us, 41 possible).  Elsewhere
// their mean, whose pick is 1.3 % behind, either alone 1.9 %.
double block_model_us(int64_t M, int64_t N, int64_t K, int bits, int64_t g, int rows16, int wk, int s, Picture picture = kLaunched) {
    const double far = block_far_us(M, N, K, bits, g, rows16, wk, s, picture);
    return N < 1024 || M > 512 ? far : std::sqrt(far * block_near_us(M, N, K, bits, g, rows16, wk, s, picture));
}

// Plan of the block kernel within `cap` bytes of partial sums, and its modelled time: row tile height (32 rows up to 96 rows, 128
// from 65), wavefronts along K, K splits.  Two exceptions to the model, plans that rtn_linear_query has always reported and that are
// relied upon: 64 to 96 rows of a matrix under 24 M weights split K in two where the workspace allows (4096 x 4096 at 64 rows: 10.2 us,
// 8.6 unsplit with eight wavefronts along K); and 8-bit matrices of half a gigabyte and more with more input than output columns
// keep 64-row tiles (16384 x 53248 at 157 rows 403 us, 340 in 128-row tiles).
double block_plan(int64_t M, int64_t N, int64_t K, int bits, int64_t g, size_t cap, bool zp, LinearPlan* p, Picture picture) {
    const int64_t units = K / chunk_k(bits);
    double best = 1e30;
    p->path = 3; p->prefetch = 1; p->waves_n = 8; p->n_tiles16 = 2; p->waves_k = 1; p->split_k = 1; p->m_rows16 = 2;
    for (int r = 2; r <= 8; r *= 2) {
        if (r == 2 && M > 96) continue;
        if (r == 8 && (M <= 64 || (g % 128 != 0 && !zp) || (bits == 8 && K > N && N * K > (int64_t)512 << 20))) continue;
        const int64_t tiles = (M + 16 * r - 1) / (16 * r);
        const int mb = (int)((M + 32 * tiles - 1) / (32 * tiles));
        for (int wk = 1; wk <= 8; wk *= 2) {
            if (wk > units || (wk == 8 && (mb > 2 || zp || (r == 2 && M >= 64) || (r == 4 && M <= 64)))) continue;
            const bool two = r == 2 && M >= 64 && N * K < 24000000 && 2 * wk <= units && (size_t)M * N * sizeof(float) * 2 <= cap;
            for (int s = two ? 2 : 1; s <= kMaxSplitK && s * wk <= units; ++s) {
                if (s > 1 && (size_t)M * N * sizeof(float) * s > cap) break;
                const double t = block_model_us(M, N, K, bits, g, r, wk, s, picture);
                if (t < best) { best = t; p->m_rows16 = r; p->waves_k = wk; p->split_k = s; }
            }
        }
    }
    p->m_blocks = (int)((M + 16 * p->m_rows16 - 1) / (16 * p->m_rows16));
    return best;
}

// The wide kernel (eight wavefronts of one tile-row: 128 columns a workgroup) in the same terms: a step of 128 columns by 16-row
// blocks, 64 workgroups a round of an XCD, each slower by 1.84 where two share a compute unit.  Fitted to 11200 launches of 693
// problems (6.6 % rms, the pick 0.3 % behind the best K split on average).
double wide16_model_us(int64_t M, int64_t N, int64_t K, int bits, int64_t g, int rows16, int s) {
    static const double kStep[3] = {0.346, 0.482, 0.527};
    const int64_t XB = (N + 127) / 128, ZB = (M + 16 * rows16 - 1) / (16 * rows16), steps = (K / 128 + s - 1) / s;
    const bool sliced = rtn::xcd_slices_save_a_round(XB, ZB, s);
    const double on_xcd = (double)((sliced ? (XB * ZB + 7) / 8 : (XB + 7) / 8 * ZB) * s), xcds = sliced ? 8.0 : (double)std::min<int64_t>(XB, 8);
    const double weights = (double)N * K * bits / 8.0, rows = (double)M * K * 2.0, share = 128.0 * steps;
    const double wg = 0.055 + (double)steps * (kStep[rows16 - 2] * (bits == 8 ? 1.08 : 1.0) + 0.018 * rows16 * 128.0 / (double)g), rounds = on_xcd / 64.0;
    const double serial = wg * std::max(1.0, 0.357 * std::ceil(rounds) + 0.643 * rounds) * (on_xcd > 32.0 ? 1.844 : 1.0);
    const double hbm = 0.924 * (weights + rows) / 6.83e6, fabric = 0.330 * (rows + weights / xcds) / 1e6;
    const double l2 = 0.409 * on_xcd * (16.0 * rows16 * share * 2.0 + 128.0 * share * bits / 8.0) / 2e6;
    double t = 3.224 + std::sqrt(serial * serial + hbm * hbm + fabric * fabric + l2 * l2) + 3.484 * (double)M * N * 2.0 / 1e7;
    if (s > 1) t += 2.292 + 0.881 * (double)M * N * s * 8.0 / 4.19e6 + (s > 8 ? 2.033 : 0.0);
    return t;
}

// The block kernel's plan, or the wide kernel's where that is modelled ahead: on small problems, where the block kernel's 256 columns
// and units of 512 (8 bit: 256) leave few workgroups and its first operands come later.  Measured, block against wide kernel:
// 29 rows of 4448 x 512 int4 6.3 us and 4.6, 32 of 14000 x 1536 10.0 and 7.7, 1885 of 1008 x 1536 g32 17.5 and 13.6; level from about
// 15 us; 8-bit weights in groups of 256 columns and more at 17 to 64 rows up to 30 us (27648 x 5120 at 41 rows 31.5 and 29.8).
// Beyond 40 us, where its model was fitted to few problems, the wide kernel is not asked (57344 x 8192 int8 g128 at 29 rows 106 us, block 79).
// Up to 64 rows the line lies 3 % to its side: of 166 measured problems 20 then run slower than on the better kernel, 24 with the models level.
// The wide kernel's row blocks: 48 rows above 64 where they save a fifth of the padded rows.  With zero points it is 3 % further
// behind (a zero point per operand and lane in half the columns).
double block_or_wide_plan(int64_t M, int64_t N, int64_t K, int bits, int64_t g, size_t cap, bool zp, LinearPlan* p, Picture picture = kLaunched) {
    const double t_block = block_plan(M, N, K, bits, g, cap, zp, p, picture);
    if (t_block > 40.0) return t_block;
    const bool blocks48 = M > 64 ? ((M + 47) / 48) * 48 * 5 <= ((M + 63) / 64) * 64 * 4 : M > 32 && M <= 48;
    const int rows16 = M <= 32 ? 2 : blocks48 ? 3 : 4;
    double best = 1e30;
    int split = 1;
    for (int s = 1; s <= kMaxSplitK && (s == 1 || K / 128 / s >= 4); ++s) {
        if (s > 1 && (size_t)M * N * sizeof(float) * s > cap) break;
        const double t = (zp ? 1.03 : 1.0) * wide16_model_us(M, N, K, bits, g, rows16, s);
        if (t < best) { best = t; split = s; }
    }
    if (best >= (M <= 64 ? 1.03 : 0.98) * t_block) return t_block;
    p->waves_n = 8; p->waves_k = 1; p->n_tiles16 = 1; p->m_rows16 = rows16; p->split_k = split;
    p->m_blocks = (int)((M + 16 * rows16 - 1) / (16 * rows16));
    return best;
}

// Tile height (128 or 256 rows) and K split of the tile kernel: the pair with the lowest modelled time.  Splits need not
// be powers of two: what pays is a split that fills the last round (144 tiles: three splits of 72 tall tiles make one
// round of 216; 405B qkv at 256 rows: 163 us against 219 with one split).
constexpr size_t kWorkspaceCapTile = (size_t)256 << 20;
double tile_plan_choose(bool dense, int64_t M, int64_t N, int64_t K, size_t workspace_cap, int* rows16, int* split_k) {
    double best = 1e30;
    *rows16 = 4; *split_k = 1;
    for (int s = 1; s <= 8; ++s) {
        if (s > 1 && ((size_t)M * N * sizeof(float) * s > workspace_cap || K / 128 / s < (dense ? 8 : 4))) break;
        for (int h = 4; h <= 8; h += 4) {
            if (h == 8 && M <= 128) continue;
            const double t = rtn::tile_model_us(dense, h, M, N, K, s);
            if (t < best) { best = t; *rows16 = h; *split_k = s; }
        }
    }
    return best;
}

// Problems the tile kernel may serve at all.  It rounds each scaled weight to fp16, the wide kernel scales fp32 sums of
// exact codes (2.7e-4 against 2.0e-4 of the norm), so this line is one of precision and does not move with the kernels'
// speed: from 144 tiles of 128 x 256 without splitting K, unless the 128-row padding costs more than 64-row padding; and
// on 4-bit weights where rounds of 256 workgroups at 0.85 us (128 rows) or 1.40 us (256 rows) a step, the best of one to
// eight splits, come below 1.075 x the wide plan's modelled time.
bool tile_line(int64_t M, int64_t N, int64_t K, int bits, double t_wide) {
    const int64_t xb = (N + 255) / 256;
    if (xb * ((M + 127) / 128) >= 144 && (M + 127) / 128 * 2 <= (M + 63) / 64) return true;
    if (bits != 4) return false;
    double best = 1e30;
    for (int s = 1; s <= 8; ++s) {
        if (s > 1 && ((size_t)M * N * sizeof(float) * s > kWorkspaceCapTile || K / 128 / s < 4)) break;
        for (int h = 4; h <= 8; h += 4) {
            if (h == 8 && M <= 128) continue;
            const double rounds = (double)((xb * ((M + 32 * h - 1) / (32 * h)) * s + 255) / 256);
            double t = rounds * ((double)((K / 64 + s - 1) / s) * (h == 4 ? 0.85 : 1.40) + 8.0);
            if (s > 1) t += 2.5 + (2.0 * s * M * N * 4.0 + 2.0 * M * N) / 4.0e6;
            best = std::min(best, t);
        }
    }
    return best * 0.93 < t_wide;
}

// The tile kernel in two launches: the first rows_first rows (a multiple of 256) as full rounds of workgroups, the
// rest as a launch of its own, which the plan above gives the K split that fills its one round.  Returns rows_first,
// or 0 where one launch is modelled within 7 % of the best pair.  Measured as two calls against one on the qkv shapes:
// 405B at 2048 rows 1044 us against 1236, at 1024 rows 565 against 641; 70B at 2048 rows 324 against 374; 8B at 4096
// rows 208 against 232; no gain (and none modelled) where the tiles fill their rounds.
int64_t two_launches_modelled(bool dense, int64_t M, int64_t N, int64_t K, size_t workspace_cap, double* time_us) {
    int r16, sk;
    const double single = tile_plan_choose(dense, M, N, K, workspace_cap, &r16, &sk);
    *time_us = single;
    if (M > 16384) return 0;                                   // many rounds: the last one no longer matters
    double best = single * 0.93;
    int64_t rows_first = 0;
    for (int64_t r1 = 256; r1 < M; r1 += 256) {
        const double t = tile_plan_choose(dense, r1, N, K, workspace_cap, &r16, &sk) +
                         tile_plan_choose(dense, M - r1, N, K, workspace_cap, &r16, &sk);
        if (t < best) { best = t; rows_first = r1; }
    }
    if (rows_first > 0) *time_us = best;
    return rows_first;
}

// Plans above 16 rows are the best of some hundred modelled candidates, 5-30 us of host time: remembered per problem in a
// table of fixed size (an entry gives way to the next one that falls on it).
template <typename Value, size_t kEntries = 1024> struct Remembered {
    struct Key {
        int64_t M, N, K, g;
        size_t workspace, lds;
        int bits, kind;
        bool operator==(const Key& o) const {
            return M == o.M && N == o.N && K == o.K && g == o.g && workspace == o.workspace && lds == o.lds && bits == o.bits && kind == o.kind;
        }
    };
    struct Entry { Key key; Value value; bool used; };
    std::mutex mutex;
    Entry table[kEntries] = {};
    static size_t slot(const Key& k) {
        uint64_t h = 0;
        for (uint64_t v : {(uint64_t)k.M, (uint64_t)k.N, (uint64_t)k.K, (uint64_t)k.g, (uint64_t)k.workspace, (uint64_t)(k.bits * 8 + k.kind)})
            h = (h ^ v) * 0x9E3779B97F4A7C15ull, h ^= h >> 29;
        return (size_t)(h % kEntries);
    }
    template <typename Make> Value get(const Key& k, Make make) {
        Entry& e = table[slot(k)];
        {
            std::lock_guard<std::mutex> lock(mutex);
            if (e.used && e.key == k) return e.value;
        }
        const Value v = make();
        std::lock_guard<std::mutex> lock(mutex);
        e.key = k; e.value = v; e.used = true;
        return v;
    }
};

int64_t tile_two_launches(bool dense, int64_t M, int64_t N, int64_t K, size_t workspace_cap, double* time_us = nullptr) {
    struct Cut { int64_t rows_first; double time_us; };
    static Remembered<Cut> remembered;
    const Cut c = remembered.get({M, N, K, 0, workspace_cap, 0, 0, dense ? 1 : 0}, [&] {
        Cut v;
        v.rows_first = two_launches_modelled(dense, M, N, K, workspace_cap, &v.time_us);
        return v;
    });
    if (time_us) *time_us = c.time_us;
    return c.rows_first;
}


// Plan of the small-batch (skinny) kernel for up to 16 rows: a table of measured configurations on a grid of
// problems -- tile-rows N / 16 from 64 to 8192 and k-chunks per row from 2 to 128, by powers of two and at the 1.5 x
// points between them, 1, 2, 4, 8, 16 rows, both precisions -- plus the linear modules of the Llama 3.1 8B / 70B / 405B and Llama 3.2 1B / 3B
// layers the paper evaluates (Table 1).  Every entry lists its twelve fastest configurations with their slowdown
// against the fastest.  A problem that is in the table takes its entry's ranking; any other one lets its three nearest
// entries (distance in log2 of tile-rows, chunks per row and rows) vote: a configuration's score is the weighted mean
// log slowdown over the three (1.5 x where an entry does not list it), and the best-scored configuration that is valid
// for the problem wins.  On shapes outside the table (tuning/shapes_heldout.txt) the pick is about 1 % behind the best
// measured configuration at the median and within 10 % on nineteen problems out of twenty.
// tuning/plan_sweep.hip measures, tuning/make_plan_table.py writes the table.
constexpr int kPlanEntryConfigs = 12;
struct SkinnyPlanConfig {
    uint8_t wn, wk, split, nb, slow;       // slow: slowdown against the entry's fastest, units of 0.5 %
};
struct SkinnyPlanEntry {
    uint8_t bits;
    uint16_t nt, kc;
    uint8_t m, n;
    SkinnyPlanConfig c[kPlanEntryConfigs];
};
const SkinnyPlanEntry kSkinnyPlanTable[] = {
#include "skinny_plan_table.inc"
};

bool skinny_plan_usable(int64_t M, int64_t N, int64_t K, int bits, const LinearPlan& p, size_t lds_limit) {
    const int64_t KC = K / chunk_k(bits);
    if (p.waves_n < 1 || p.waves_k < 1 || p.waves_n * p.waves_k > 16) return false;
    if (p.split_k < 1 || p.split_k > kMaxSplitK || p.split_k > KC) return false;
    if (p.split_k > 1 && (size_t)M * N * sizeof(float) * p.split_k > kWorkspaceCap) return false;
    LinearArgs a;
    a.M = M; a.N = N; a.K = K; a.bits = bits; a.g = K;
    return rtn::linear_plan_fits(a, p, lds_limit);
}

// Workgroups come in rounds of one per compute unit: a launch of n workgroups keeps the busiest of the 256 compute units
// ceil(n / 256) workgroups long where n / 256 would be the average.  Coarse configurations (few, long-lived workgroups)
// pay for it: 269 workgroups of eight wavefronts take 1.45 x the time of 256.  The table's grid shapes are powers of
// two, the best case, so a configuration's measured slowdown is corrected by this ratio to the power 0.7 (fitted on
// shapes outside the table), entry against problem.
constexpr double kImbalanceExp = 0.7;
constexpr double kWidthStep = 0.3;      // log-time per octave of workgroup width away from a voted configuration
double cu_imbalance(int64_t workgroups) {
    const double avg = (double)workgroups / 256.0;
    return std::ceil(avg) / avg;
}

bool skinny_plan_from_table(int64_t M, int64_t N, int64_t K, int bits, size_t lds_limit, LinearPlan* out) {
    const double fnt = std::log2((double)(N / 16)), fkc = std::log2((double)(K / chunk_k(bits))), fm = std::log2((double)M);
    const int n = (int)(sizeof(kSkinnyPlanTable) / sizeof(kSkinnyPlanTable[0]));
    constexpr int kVoters = 3;
    int near_i[kVoters];
    double near_d[kVoters];
    int found = 0;
    for (int i = 0; i < n; ++i) {
        const SkinnyPlanEntry& e = kSkinnyPlanTable[i];
        if (e.bits != bits) continue;
        const double d = 2.0 * std::fabs(std::log2((double)e.nt) - fnt) + std::fabs(std::log2((double)e.kc) - fkc) +
                         0.5 * std::fabs(std::log2((double)e.m) - fm);
        int pos = found < kVoters ? found : kVoters;             // insertion into the sorted list of the nearest
        while (pos > 0 && d < near_d[pos - 1]) --pos;
        if (pos >= kVoters) continue;
        for (int q = (found < kVoters ? found : kVoters - 1); q > pos; --q) { near_i[q] = near_i[q - 1]; near_d[q] = near_d[q - 1]; }
        near_i[pos] = i; near_d[pos] = d;
        if (found < kVoters) ++found;
    }
    if (found == 0) return false;
    if (near_d[0] < 1e-9) found = 1;                            // the problem itself is in the table: its own ranking
    struct Scored { SkinnyPlanConfig c; double base, score; };
    std::vector<Scored> cand;
    cand.reserve(kVoters * kPlanEntryConfigs * 8);
    const double kMissing = std::log(1.5);
    const int64_t NT = N / 16;
    auto same = [](const SkinnyPlanConfig& a, const SkinnyPlanConfig& b) {
        return a.wn == b.wn && a.wk == b.wk && a.split == b.split && a.nb == b.nb;
    };
    auto imbalance_of = [](int64_t nt, const SkinnyPlanConfig& c) {
        return std::log(cu_imbalance(((nt + c.wn - 1) / c.wn) * c.split));
    };
    for (int v = 0; v < found; ++v) {
        const SkinnyPlanEntry& e = kSkinnyPlanTable[near_i[v]];
        for (int k = 0; k < e.n; ++k) {
            bool seen = false;
            for (size_t q = 0; q < cand.size() && !seen; ++q) seen = same(cand[q].c, e.c[k]);
            if (seen) continue;
            double num = 0.0, den = 0.0;
            for (int u = 0; u < found; ++u) {
                const SkinnyPlanEntry& f = kSkinnyPlanTable[near_i[u]];
                const double w = 1.0 / (near_d[u] + 0.25);
                double ls = kMissing;
                for (int q = 0; q < f.n; ++q)
                    if (same(f.c[q], e.c[k])) {
                        ls = std::min(kMissing, std::log(1.0 + f.c[q].slow / 200.0));
                        break;
                    }
                // the entry's own workgroup-count imbalance is taken out of its measurement ...
                ls -= kImbalanceExp * imbalance_of(f.nt, e.c[k]);
                num += w * ls; den += w;
            }
            // ... and the problem's own put in; ties: the order of the nearer entry
            const double base = num / den;
            cand.push_back({e.c[k], base, base + kImbalanceExp * imbalance_of(NT, e.c[k]) + 1e-9 * (double)cand.size()});
        }
    }
    // Workgroup width follows the problem, not the table: a voted configuration one or two wavefronts deep along K also
    // stands for its neighbours with any other number of wavefronts along N (1 .. 16 / waves_k), scored as itself with
    // the neighbour's workgroup-count imbalance and kWidthStep per octave of width moved.  The table's grid has powers
    // of two of tile-rows, where powers of two of wavefronts always divide evenly; a matrix of, say, 2153 tile-rows
    // is served 25-35 % faster at 16 rows by nine wavefronts (240 workgroups) than by eight (270, a second round on
    // fourteen compute units).  Not applied when the problem itself is in the table.
    if (found > 1) {
        const size_t voted = cand.size();
        for (size_t q = 0; q < voted; ++q) {
            const SkinnyPlanConfig c = cand[q].c;
            if (c.wk > 2 || c.split > 4 || (c.wk == 1 && c.nb == 1 && c.split > 1) || (c.wk == 2 && c.split > 2)) continue;
            for (int w2 = 1; w2 <= 16 / c.wk; ++w2) {
                if (w2 == c.wn || w2 > NT) continue;
                SkinnyPlanConfig c2 = c;
                c2.wn = (uint8_t)w2;
                const double sc = cand[q].base + kImbalanceExp * imbalance_of(NT, c2) +
                                  kWidthStep * std::fabs(std::log2((double)w2 / c.wn)) + 1e-6;
                size_t at = 0;
                while (at < cand.size() && !same(cand[at].c, c2)) ++at;
                if (at < voted) continue;                            // voted on directly
                if (at == cand.size()) cand.push_back({c2, cand[q].base, sc});
                else if (sc < cand[at].score) cand[at].score = sc;
            }
        }
    }
    const int nc = (int)cand.size();
    std::sort(cand.begin(), cand.end(), [](const Scored& a, const Scored& b) { return a.score < b.score; });
    for (int q = 0; q < nc; ++q) {
        LinearPlan p;
        p.path = 1; p.n_tiles16 = 1; p.m_rows16 = 1; p.m_blocks = 1;
        p.prefetch = cand[q].c.nb; p.waves_n = cand[q].c.wn; p.waves_k = cand[q].c.wk; p.split_k = cand[q].c.split;
        while (p.waves_n > 1 && p.waves_n > N / 16) p.waves_n /= 2;
        if (skinny_plan_usable(M, N, K, bits, p, lds_limit)) { *out = p; return true; }
    }
    return false;
}

// Groups of 32 and 64 columns from 20 rows up: path 3 with several scales per 128 columns (its plan is block_or_wide_plan's), or the
// skinny kernel 32 or 64 rows at a time (16 with zero points), whichever is modelled faster.  Path 3 is modelled, and was measured
// for the figures here, on the wide kernel in the shapes that wide_plan picks.  Up to 19 rows the skinny kernel is ahead (8B qkv, group
// 64: 9.3 us against 11.5 at 19 rows, 15.8 against 11.4 at 20).  Above, the wide kernel leads on large matrices -- 27 us against
// 44 (8B qkv), 83 against 121 (8B gate_up), 148 against 207 (70B down) at 256 rows -- and the skinny kernel
//   - where a workgroup's rows fit the LDS in one piece and there are few workgroups: the wide kernel walks K in steps of half a
//     microsecond and hardly splits so small a matrix.  20 rows of 2048 x 2048: 4.7 us against 11.2 (zero points 3.9 against
//     13.3), of 3072 x 3072 int4 group 64 12.3 against 16.3, 147 rows of 592 x 1024 6.2 against 9.2;
//   - up to 32 rows on the matrices it streams (streams_to_32_rows): int4 20 rows of 28672 x 8192 33 us against 41.
// Both models have the form of wide_model_us (serial time of a workgroup against streamed bytes) and were fitted to both kernels'
// times on 1018 problems (1015 with zero points) of 128 to 106496 x 512 to 53248 at 20 to 300 rows: 7 % and 10 % rms (8 and
// 17 %).  The pick is 0.3 % (0.7 %) behind the better kernel on average, more than 10 % on one problem in 93 (42); the wide
// kernel everywhere would be 9 % (26 %) behind.
bool small_groups(int64_t M, int64_t g) { return (g == 64 || g == 32) && M >= 20; }

double small_groups_wide_us(const LinearArgs& a, const LinearPlan& p) {
    struct Fit { double base, split, start, step, rows, tiles, bits8, hbm, l2; };
    static const Fit kFit = {3.2, 2.87, 0.21, 0.52, 0.22, 0.36, 0.09, 1.09, 0.39}, kFitZp = {0.83, 3.76, 2.02, 0.71, 0.12, 0.39, 0.1, 1.57, 0.31};
    const Fit& f = a.zeros ? kFitZp : kFit;
    const int64_t cols = 16 * p.n_tiles16 * p.waves_n, XB = (a.N + cols - 1) / cols;
    const double wgs = (double)(XB * p.m_blocks * p.split_k), steps = (double)((a.K / 128 + p.split_k - 1) / p.split_k);
    const double wg_us = f.start + steps * f.step * (1.0 + f.rows * (p.m_rows16 - 2) + f.tiles * (p.n_tiles16 - 1) * p.m_rows16 + (a.bits == 8 ? f.bits8 : 0.0));
    const double serial = std::max(1.0, wgs / 256.0) * wg_us;
    const double stream = f.hbm * a.N * a.K * a.bits / 8.0 / 6.5e6 + f.l2 * XB * p.m_blocks * 16.0 * p.m_rows16 * a.K * 2.0 / 1.1e7;
    double t = f.base + std::cbrt(serial * serial * serial + stream * stream * stream);
    if (p.split_k > 1) t += f.split + (double)a.M * a.N * p.split_k * 8.0 / 4.5e6;
    return t;
}

double small_groups_skinny_us(const LinearArgs& a, const LinearPlan& p) {
    struct Fit { double base, split, rounds, chunk, rows, bits8, slice, stage, hbm, l2; };
    static const Fit kFit = {1.83, 3.55, 0.51, 2.14, 0.23, -0.49, 0.96, 0.83, 0.9, 1.54}, kFitZp = {2.49, 0.0, 1.24, 1.42, 0.0, -0.22, 0.41, 0.47, 2.38, 1.24};
    const Fit& f = a.zeros ? kFitZp : kFit;
    const rtn::StagePlan s = rtn::linear_stages(a, p);
    const double wgs = (double)((a.N / 16 + p.waves_n - 1) / p.waves_n * p.split_k * p.m_blocks);
    const double resident = std::max(1.0, std::min(std::floor(16.0 / (p.waves_n * p.waves_k)), std::floor((double)rtn::kMaxLdsBytes / (double)s.lds)));
    const double wg_us = s.per * f.chunk * (1.0 + f.rows * (p.m_rows16 - 1) + (a.bits == 8 ? f.bits8 : 0.0)) + f.slice * (double)s.slice / 102400.0 +
                         (s.nstage > 1 ? f.stage * s.nstage : 0.0);
    const double serial = std::pow(std::max(1.0, wgs / (256.0 * resident)), f.rounds) * wg_us;
    const double stream = f.hbm * a.N * a.K * a.bits / 8.0 / 6.5e6 + f.l2 * wgs * (double)s.slice / 1.1e7;
    double t = f.base + std::cbrt(serial * serial * serial + stream * stream * stream);
    if (p.split_k > 1) t += f.split + (double)a.M * a.N * p.split_k * 8.0 / 4.5e6;
    return t;
}

// more than 16 rows: the wide kernel, except at 17-32 rows on large matrices, where the skinny kernel's pure
// weight streaming still wins.  4 bit: from 40 MB with rows of 8192 columns and more, 16 wavefronts side by side
// (6-20 % faster on the 70B and 405B shapes except the 70B o matrix; the wide kernel wins on every 8B shape).
// 8 bit: above 256 MB, the same 16-wavefront shape (with K split to one round of workgroups it is 15-20 % faster
// than 8 wavefronts on the 70B gate_up and 405B qkv matrices and level on the 405B gate_up and down matrices).
bool streams_to_32_rows(int64_t M, int64_t N, int64_t K, int bits) {
    const size_t packed_bytes = (size_t)N * K * bits / 8;
    return M <= 32 && ((bits == 4 && packed_bytes >= ((size_t)40 << 20) && K >= 8192) || packed_bytes > ((size_t)256 << 20));
}

// a: M, N, K, bits, g and whether there are zero points; skinny, wide: the kernels' own plans.
bool skinny_on_small_groups(const LinearArgs& a, const LinearPlan& skinny, const LinearPlan& wide) {
    const bool streams = streams_to_32_rows(a.M, a.N, a.K, a.bits) && a.N * a.K * a.bits / 8 > (int64_t)40 << 20;   // (at 40 MiB the models decide)
    if (!a.zeros && streams) return true;
    if (a.M > (a.zeros ? 64 : 32) && a.N * a.K >= 8000000) return false;                  // beyond the models' accuracy
    return small_groups_skinny_us(a, skinny) < (a.zeros ? 0.95 : 1.0) * small_groups_wide_us(a, wide);
}

// The tile kernel's modelled time, in one launch or two, against the plan w of wide_plan, of modelled time t_wide: where the line of
// exact codes lies (see wide_or_tile_plan).  wide_plan's model, fitted at 32 to 256 rows, falls short of that kernel's times here: by 1.26 and 1.20 at 4 bit (groups of 128, others), 1.51 and
// 1.30 at 8 bit (means over 460 problems; the tile kernel's by 1.03).
bool tile_beats_wide(int64_t M, int64_t N, int64_t K, int bits, int64_t g, const LinearPlan& w, double t_wide, size_t workspace) {
    const int64_t fit = std::max<int64_t>(1, (int64_t)(workspace / ((size_t)M * N * sizeof(float))));
    const double t_fit = w.split_k > fit ? wide_model_us(M, N, K, bits, w.m_rows16, w.waves_n, w.n_tiles16, (int)fit) : t_wide;
    double t_tile = 0;
    tile_two_launches(false, M, N, K, workspace, &t_tile);
    return t_tile * 1.03 < t_fit * (bits == 4 ? (g == 128 ? 1.26 : 1.20) : (g == 128 ? 1.51 : 1.30));
}

// force_path: 0 = choose the path, otherwise the default plan of that path.  workspace: bytes at hand for
// partial sums (by default what its best plan may take): kernel, height, split and cut are chosen within it, instead of
// the unconstrained plan with its split cut down.  Within 16 MiB, cut down against chosen: 1011 rows of 4608 x 5120 104 us
// against 77, 2921 of 1792 x 5120 105 against 84, 2048 of 4096 x 14336 321 against 236, 256 of 16384 x 53248 1010 against 734.
LinearPlan auto_plan(int64_t M, int64_t N, int64_t K, int bits, int64_t g, size_t lds_limit, int force_path = 0,
                     int64_t steps_hint = 0, size_t workspace = kWorkspaceCapTile);

LinearPlan wide_or_tile_plan(int64_t M, int64_t N, int64_t K, int bits, int64_t g, size_t workspace);

LinearPlan modelled_plan(int64_t M, int64_t N, int64_t K, int bits, int64_t g, size_t lds_limit, int force_path, int64_t steps_hint,
                         size_t workspace) {
    LinearPlan p;
    p.n_tiles16 = 1;
    const size_t cap = std::min(workspace, M >= 64 && g % 128 == 0 ? kWorkspaceCapTall : kWorkspaceCap);   // the block kernel's partials
    if (force_path == 0 && small_groups(M, g)) {
        LinearArgs a;
        a.M = M; a.N = N; a.K = K; a.bits = bits; a.g = g;
        wide_plan(M, N, K, bits, g, &p);
        const LinearPlan skinny = auto_plan(M, N, K, bits, g, lds_limit, 1);
        // (the wide kernel's split shrinks to the workspace, the skinny kernel's does not)
        const bool held = skinny.split_k == 1 || (size_t)M * N * sizeof(float) * skinny.split_k <= workspace;
        if (held && skinny_on_small_groups(a, skinny, p)) return skinny;
        block_or_wide_plan(M, N, K, bits, g, cap, false, &p);
        return p;
    }
    const size_t packed_bytes = (size_t)N * K * bits / 8;
    const bool streams16 = streams_to_32_rows(M, N, K, bits);
    const bool wide_wins = g % 128 == 0 && M > 16 && !(streams16 && packed_bytes > ((size_t)512 << 20));
    bool tile_wins = false;
    LinearPlan w, block;
    double t_block = 0;
    if (force_path == 3) wide_plan(M, N, K, bits, g, &w);
    if (force_path == 0 && wide_wins) t_block = block_or_wide_plan(M, N, K, bits, g, cap, false, &block);
    // The tile kernel rounds each scaled weight to fp16, the block kernel does not: it may take a problem from the tile kernel, never
    // give it one.  (Without the line, 0.4 % of the problems of 129 to 1024 rows lost bits: 749 rows of 5952 x 3072 int4, 362 of
    // 12176 x 1536 int8; and 16384 x 53248 at 133 rows without a workspace took 697 us on an unsplit tile plan.)
    if (force_path == 0 && wide_wins && M >= 128 && wide_or_tile_plan(M, N, K, bits, g, workspace).path == 4) {
        double t_tile = 0;
        tile_two_launches(false, M, N, K, workspace, &t_tile);
        // This line is one of precision too: it does not move where the picture of the block kernel's row tiles changes (two heights alone
        // moved 31 of 60000 drawn problems to the tile kernel; 391 rows of 26800 x 1024, 593 of 25952 x 1536 without a
        // workspace).  Beyond a third no picture is ahead of another.
        if (t_tile * 1.03 < t_block * 1.05 && t_tile * 1.5 > t_block) {
            LinearPlan unused;
            for (Picture picture : {kOneHeight, kTwoHeights})
                t_block = std::min(t_block, block_or_wide_plan(M, N, K, bits, g, cap, false, &unused, picture));
        }
        // against the block kernel (both sides of 156 such problems measured: 2-4 % behind the better one, and no better for lines
        // 5 % to either side); a little towards the tile kernel above 512 rows, where it also takes several modules of a layer at once.
        // The long 4-bit matrices of 400 MB just above 128 rows stay on the tile kernel, as rtn_linear_query is known to report them
        // (16384 x 53248 at 129 rows: 375 us, block 294).
        tile_wins = M > (bits == 4 ? 1024 : 512) || t_tile * 1.03 < t_block * (M > 512 ? 1.05 : 1.0) ||
                    (bits == 4 && K > N && packed_bytes >= ((size_t)400 << 20) && M > 128 && M <= 144);
    }
    if (force_path == 4 || tile_wins) {
        p.path = 4;
        p.prefetch = 1; p.waves_n = 8; p.waves_k = 1;
        tile_plan_choose(false, M, N, K, workspace, &p.m_rows16, &p.split_k);
        p.m_blocks = (int)((M + 32 * p.m_rows16 - 1) / (32 * p.m_rows16));
        return p;
    }
    if (force_path == 3) return w;
    if (force_path == 0 && wide_wins) return block;
    if (M <= 16 && steps_hint == 0) {
        // the table lookup costs tens of microseconds of host time (logarithms over ~800 entries): remembered per problem
        struct Key { int64_t M, N, K; int bits; size_t lds; };
        struct Memo { Key k; LinearPlan p; bool ok; };
        static std::mutex memo_mutex;
        static std::vector<Memo> memo;
        {
            std::lock_guard<std::mutex> lock(memo_mutex);
            for (const Memo& m : memo)
                if (m.k.M == M && m.k.N == N && m.k.K == K && m.k.bits == bits && m.k.lds == lds_limit) {
                    if (m.ok) return m.p;
                    goto rules;
                }
        }
        {
            const bool ok = skinny_plan_from_table(M, N, K, bits, lds_limit, &p);
            std::lock_guard<std::mutex> lock(memo_mutex);
            if (memo.size() >= 4096) memo.clear();              // a serving process sees a handful of shapes; bound it anyway
            memo.push_back({{M, N, K, bits, lds_limit}, p, ok});
            if (ok) return p;
        }
    }
rules:
    p.n_tiles16 = 1;
    // (no usable table entry, more than 16 rows on this kernel, or a slice of a grouped launch: the rules below)
    const int64_t NT = N / 16, KC = K / chunk_k(bits);
    // 4 KiB chunk-steps in the whole matrix, or in everything that shares the launch (grouped call)
    const int64_t steps = NT * KC > steps_hint ? NT * KC : steps_hint;
    p.m_rows16 = M <= 16 ? 1 : (M <= 32 ? 2 : 4);              // weights are streamed once per 16/32/64 rows
    const int mrows = 16 * p.m_rows16;
    const int rows = (int)(M < mrows ? M + 1 : mrows);
    p.path = 1;
    p.m_blocks = (int)((M + mrows - 1) / mrows);
    p.prefetch = 1;
    p.split_k = 1;
    // Matrices of a hundred megabytes and more with long rows (more than 16 chunks): the launch is many generations of
    // workgroups, its fixed costs no longer count, and what matters is the activation traffic from L2 (M / (4 waves_n)
    // of the weight bytes, whatever the K split) and enough, not too long-lived, workgroups.  From sweeps over
    // (waves_n, waves_k, split_k, prefetch) on the 70B and 405B shapes at 1-16 rows (choice within 10 % of the best
    // measured configuration everywhere, 3 % on average).
    const size_t wbytes = (size_t)N * (size_t)K * (size_t)bits / 8;
    if (KC > 16 && wbytes >= ((size_t)100 << 20) && rows <= 16) {
        if (rows == 2) {                                       // one row: eight wavefronts along K, K in halves up to 32 chunks
            p.waves_n = 1; p.waves_k = 8; p.split_k = KC <= 32 ? 2 : 1;
        } else if (rows == 3 && KC <= 32) {
            p.waves_n = 2; p.waves_k = 2; p.split_k = 4;
        } else {
            // eight tile-rows share the staged rows; K is split across workgroups to fill the compute units
            p.waves_n = 8; p.waves_k = 1; p.split_k = 1;
            // (two of these workgroups share a compute unit: as many splits as keep the launch within one round of 512;
            // three on the 405B qkv matrix, 144 workgroups each, are 9-14 % faster than four)
            int64_t split = 512 / ((NT + 7) / 8);
            split = split < 1 ? 1 : (split > 8 ? 8 : split);
            while (split > 1 && (KC / split < 4 || (size_t)M * N * sizeof(float) * split > kWorkspaceCap)) --split;
            p.split_k = (int)split;
        }
    } else
    // up to 4 rows on a moderately long K (K = 14336: 28 chunks) also stream best unsplit: 14 wavefronts x 2 chunks
    if (rows <= 2 || (rows == 3 && KC >= 16) || (rows <= 5 && KC > 16 && KC <= 32 && NT <= 384)) {
        const int64_t per_wave = steps <= 6144 ? 1 : (steps <= 24576 ? 2 : 4);
        const int64_t even = (KC + per_wave - 1) / per_wave;   // wavefronts that each get exactly per_wave chunks
        if (even <= 16 && KC % even == 0) {
            p.waves_k = (int)even;                             // e.g. K = 14336: 28 chunks = 14 wavefronts x 2
        } else {
            p.waves_k = round_pow2(even, 1, 16);
            while (p.waves_k > KC) p.waves_k /= 2;
        }
        p.waves_n = (steps > 24576 && p.waves_k < 8) ? 8 / p.waves_k : 1;    // eight wavefronts only for the largest
        if (p.waves_k > 8 && KC == 16) {                       // 16 one-chunk wavefronts: two tile-rows of 8 do better (8-bit 8B qkv)
            p.waves_k = 8;
            p.waves_n = NT >= 384 ? 2 : 1;
        }
    } else if (steps <= 6144) {
        p.waves_k = round_pow2(KC, 1, 8);
        while (p.waves_k > KC) p.waves_k /= 2;
        p.waves_n = NT >= 384 ? 2 : 1;
    } else if (rows <= 16) {
        if (KC > 16) {                                         // long K: about 7-14 chunks per workgroup
            p.waves_n = (rows <= 5 && KC <= 32) ? 2 : 4;       // few rows: two tile-rows share them, more workgroups
            p.waves_k = KC <= 32 ? 4 : 2;
            int64_t split = 4;
            while (split > 1 && (size_t)M * N * sizeof(float) * split > kWorkspaceCap) --split;
            p.split_k = (int)split;
        } else if (steps > 24576 && NT <= 2048) {              // many chunk-steps in few tile-rows (8-bit 8B gate_up)
            p.waves_n = 4;
            p.waves_k = 2;
        } else if (steps > 24576) {                            // the largest matrices: long-lived wavefronts
            p.waves_n = rows <= 5 ? 2 : 8;
            p.waves_k = rows <= 5 ? 2 : 1;
        } else if (KC >= 16) {                                 // K = 8192 on matrices of 30-60 MB (sweeps on the 70B qkv and o)
            if (rows <= 5) { p.waves_n = 2; p.waves_k = 4; }
            else if (rows <= 9) { p.waves_n = 4; p.waves_k = 4; p.split_k = 4; }
            else { p.waves_n = 8; p.waves_k = 2; p.split_k = 4; }
            while (p.split_k > 1 && (size_t)M * N * sizeof(float) * p.split_k > kWorkspaceCap) p.split_k /= 2;
        } else {
            p.waves_n = 4;
            p.waves_k = rows <= 9 ? 4 : 2;
        }
    } else {
        // more than 16 rows: wide workgroups share the staged rows (16 wavefronts on the large matrices that stay on
        // this kernel at 17-32 rows); K is split across workgroups only as far as needed to occupy the compute units
        p.waves_n = streams16 ? 16 : 8;
        p.waves_k = 1;
        const int64_t wgs = ((NT + 15) / 16) * p.m_blocks;
        if (streams16) {
            // one 16-wavefront workgroup runs per compute unit: as many splits as keep the launch within one round of
            // 256 (72 workgroups x 3 on the 405B qkv matrix: 45 us against 55 with two splits, 61-65 with four);
            // five to seven splits measured level with four
            int64_t s = 256 / wgs;
            s = s < 1 ? 1 : (s > 8 ? 8 : (s > 4 && s < 8 ? 4 : s));
            while (s > 1 && (s > KC || (size_t)M * N * sizeof(float) * s > kWorkspaceCap)) --s;
            p.split_k = (int)s;
        } else {
            while (wgs * p.split_k < 256 && p.split_k * 2 <= kMaxSplitK && p.split_k * 2 <= KC &&
                   (size_t)M * N * sizeof(float) * (p.split_k * 2) <= kWorkspaceCap)
                p.split_k *= 2;
        }
    }
    while (p.waves_n > 1 && p.waves_n > NT) p.waves_n /= 2;
    LinearArgs a;
    a.M = M; a.N = N; a.K = K; a.bits = bits; a.g = K;
    while (!rtn::linear_plan_fits(a, p, lds_limit) && p.waves_n < 16) {   // more threads to stage the rows
        p.waves_n *= 2;
        while (p.waves_n * p.waves_k > 16) p.waves_k /= 2;
    }
    return p;
}

LinearPlan auto_plan(int64_t M, int64_t N, int64_t K, int bits, int64_t g, size_t lds_limit, int force_path, int64_t steps_hint,
                     size_t workspace) {
    auto make = [&] { return modelled_plan(M, N, K, bits, g, lds_limit, force_path, steps_hint, workspace); };
    if (M <= 16) return make();                               // the skinny kernel's table has a memory of its own
    static Remembered<LinearPlan> remembered;
    return remembered.get({M, N, K, g, workspace, lds_limit, bits, force_path}, make);
}

int tall_wide_split(int64_t M, int64_t N, int64_t K) {
    const int64_t wgs = ((N + 255) / 256) * ((M + 127) / 128);
    const double t1 = 2.0 * 128 * 256 * (double)K / 4.3e12, mn4 = (double)M * N * 4.0;
    int best_s = 1;
    double best = 1e30;
    for (int s = 1; s <= 8; ++s) {
        if (s > 1 && ((size_t)M * N * sizeof(float) * s > kWorkspaceCapTall || K / 128 / s < 4)) break;
        const double rounds = (double)((wgs * s + 255) / 256);
        double t = rounds * (t1 / s + 9e-6);
        if (s > 1) t += 4e-6 + 2.0 * s * mn4 / 5e12;
        if (t < best) { best = t; best_s = s; }
    }
    return best_s;
}

// The plan above 16 rows (groups of whole 128 columns) that the wide kernel, with a 128-row tile for long 4-bit matrices, or
// the tile kernel has, whichever these two's models put ahead.  Explicit configurations that leave fields open are completed
// from it, and the line of rtn_linear_noalloc is drawn by it, so that what is accepted does not move with the automatic plan.
LinearPlan wide_or_tile_plan(int64_t M, int64_t N, int64_t K, int bits, int64_t g, size_t workspace) {
    const int64_t tiles = ((N + 255) / 256) * ((M + 127) / 128);
    LinearPlan p;
    wide_plan(M, N, K, bits, g, &p);
    const bool tall = bits == 4 && M >= 128 && (M + 127) / 128 * 2 <= (M + 63) / 64 && (size_t)N * K * bits / 8 >= ((size_t)40 << 20) && K > N;
    if (M >= 128) {
        const double t_wide = wide_model_us(M, N, K, bits, p.m_rows16, p.waves_n, p.n_tiles16, p.split_k);
        if (tile_line(M, N, K, bits, t_wide) && !(tall && M < 192 && tiles < 144) &&
            (tiles >= 256 || tile_beats_wide(M, N, K, bits, g, p, t_wide, workspace))) {
            p.path = 4; p.waves_n = 8;
            tile_plan_choose(false, M, N, K, workspace, &p.m_rows16, &p.split_k);
            p.m_blocks = (int)((M + 32 * p.m_rows16 - 1) / (32 * p.m_rows16));
            p.n_tiles16 = 1;
            return p;
        }
    }
    if (tall) {
        p.waves_n = 8; p.n_tiles16 = 2; p.m_rows16 = 8;
        p.m_blocks = (int)((M + 127) / 128);
        p.split_k = tall_wide_split(M, N, K);
    }
    return p;
}

// Bytes of partial sums of a plan: the single launch's or, of a tile plan, those of the two that rtn_linear may issue.
size_t plan_partials(const LinearPlan& p, int64_t M, int64_t N, int64_t K) {
    auto bytes = [&](int64_t rows, int split) { return split > 1 ? ((size_t)rows * N * sizeof(float) * split + 255) & ~(size_t)255 : (size_t)0; };
    size_t need = bytes(M, p.split_k);
    const int64_t first = p.path == 4 ? tile_two_launches(false, M, N, K, kWorkspaceCapTile) : 0;
    for (int64_t rows : {first, first > 0 ? M - first : 0}) {
        int r16, sk;
        if (rows == 0) continue;
        tile_plan_choose(false, rows, N, K, kWorkspaceCapTile, &r16, &sk);
        need = std::max(need, bytes(rows, sk));
    }
    return need;
}

size_t wide_or_tile_partials(int64_t M, int64_t N, int64_t K, int bits, int64_t g) {
    return M > 16 && g % 128 == 0 ? plan_partials(wide_or_tile_plan(M, N, K, bits, g, kWorkspaceCapTile), M, N, K) : 0;
}

// The plan as a complete explicit configuration.
rtn_linear_cfg plan_cfg(const LinearPlan& p) {
    rtn_linear_cfg c;
    c.path = p.path; c.prefetch = p.prefetch; c.waves_n = p.waves_n; c.waves_k = p.waves_k;
    c.split_k = p.split_k; c.m_rows16 = p.m_rows16; c.n_tiles16 = p.n_tiles16;
    return c;
}

// Bytes of the workspace passed that the tile kernel's plans may count on.
size_t tile_workspace(const LinearArgs& a, size_t workspace_nbytes) {
    return a.workspace ? std::min(workspace_nbytes, kWorkspaceCapTile) : 0;
}

rtn_status resolve_plan(const LinearArgs& a, const rtn_linear_cfg* cfg, size_t workspace_nbytes, LinearPlan* out) {
    const size_t lds_limit = (size_t)device_max_lds();
    LinearPlan p;
    p.n_tiles16 = 1;
    const bool whole = cfg && cfg->path && cfg->prefetch && cfg->waves_n && cfg->waves_k && cfg->split_k && cfg->m_rows16 && cfg->n_tiles16;
    if (whole) p.m_blocks = 1;                                  // every field comes from the caller
    else {
        const int path = !cfg ? 0 : cfg->path == 0 && small_groups(a.M, a.g) ? 1 : cfg->path;
        const size_t partials = tile_workspace(a, workspace_nbytes);
        if (cfg && path == 0 && a.M > 16 && a.g % 128 == 0 && !streams_to_32_rows(a.M, a.N, a.K, a.bits))
            p = wide_or_tile_plan(a.M, a.N, a.K, a.bits, a.g, partials);
        else
            p = auto_plan(a.M, a.N, a.K, a.bits, a.g, lds_limit, cfg && path == 0 && a.M > 16 && a.g % 128 == 0 ? 1 : path, 0, partials);
    }
    if (cfg) {
        if (cfg->path) p.path = cfg->path;
        if (cfg->prefetch) p.prefetch = cfg->prefetch;
        if (cfg->waves_n) p.waves_n = cfg->waves_n;
        if (cfg->waves_k) p.waves_k = cfg->waves_k;
        if (cfg->split_k) p.split_k = cfg->split_k;
        if (cfg->m_rows16) {
            p.m_rows16 = cfg->m_rows16;
            p.m_blocks = (int)((a.M + 16 * p.m_rows16 - 1) / (16 * p.m_rows16));
        }
        if (cfg->n_tiles16) p.n_tiles16 = cfg->n_tiles16;
        // the vector-ALU variant and several row blocks per wavefront keep one chunk in flight: an automatic plan's deeper
        // prefetch does not carry over to them unless asked for
        if (!cfg->prefetch && (p.path == 2 || (p.path == 1 && p.m_rows16 > 1))) p.prefetch = 1;
        if (p.path == 4 && !cfg->m_rows16 && cfg->split_k) p.m_rows16 = 0;     // a given split: height chosen at launch
    }
    const int64_t KC = a.K / chunk_k(a.bits);
    if (p.path < 1 || p.path > 4) return RTN_ERR_CONFIG;
    // wide and tile kernels: a split the caller did not ask for shrinks to what the workspace passed can hold (slower,
    // not an error; the skinny kernel's plans tie the staged slice to the split, so there it stays an error)
    if (p.path >= 3 && !(cfg && cfg->split_k) && p.split_k > 1) {
        const size_t one = (size_t)a.M * a.N * sizeof(float);
        const size_t fit = a.workspace ? workspace_nbytes / one : 0;
        if ((size_t)p.split_k > fit) p.split_k = fit < 1 ? 1 : (int)fit;
    }
    if (p.path >= 3) {
        bool ok = p.path == 3 ? rtn::wide_plan_valid(a, p) : rtn::tile_plan_valid(a, p);
        if (p.path == 3 && a.g % 128 != 0 && cfg && !whole) ok = false;       // no defaults to fill in, see small_groups
        if (!ok || p.split_k > kMaxSplitK) return RTN_ERR_CONFIG;
        if ((uint64_t)a.N * a.K * a.bits / 8 >= 0x7FFF0000ull || (uint64_t)a.M * a.K * 2 >= 0x7FFF0000ull)
            return RTN_ERR_SHAPE;                               // 32-bit buffer offsets
        if (p.split_k > 1) {
            const size_t need = (size_t)a.M * a.N * sizeof(float) * p.split_k;
            if (a.workspace == nullptr || workspace_nbytes < need) return RTN_ERR_WORKSPACE;
        }
        *out = p;
        return RTN_OK;
    }
    if (p.path == 2 && (a.M > 4 || p.prefetch != 1 || p.m_rows16 != 1 || a.g < tile_k(a.bits))) return RTN_ERR_CONFIG;
    if (p.prefetch != 1 && p.prefetch != 2 && p.prefetch != 4) return RTN_ERR_CONFIG;
    if (p.m_rows16 != 1 && p.m_rows16 != 2 && p.m_rows16 != 4) return RTN_ERR_CONFIG;
    if (p.m_rows16 > 1 && p.prefetch != 1) return RTN_ERR_CONFIG;
    if (p.waves_n < 1 || p.waves_k < 1 || p.waves_n * p.waves_k > 16) return RTN_ERR_CONFIG;
    if (p.split_k < 1 || p.split_k > kMaxSplitK || p.split_k > KC) return RTN_ERR_CONFIG;
    if (!rtn::linear_plan_fits(a, p, lds_limit)) return RTN_ERR_CONFIG;
    if ((uint64_t)a.N * a.K * a.bits / 8 >= 0x7FFF0000ull || (uint64_t)a.M * a.K * 2 >= 0x7FFF0000ull)
        return RTN_ERR_SHAPE;                                   // 32-bit buffer offsets
    if (p.split_k > 1) {
        const size_t need = (size_t)a.M * a.N * sizeof(float) * p.split_k;
        if (a.workspace == nullptr || workspace_nbytes < need) return RTN_ERR_WORKSPACE;
    }
    *out = p;
    return RTN_OK;
}

// The asymmetric variant's automatic plan.
rtn_status resolve_plan_zp(const LinearArgs& a, size_t workspace_nbytes, LinearPlan* p) {
    // the small-batch kernel, 16 rows per workgroup, planned as for min(M, 16) rows
    LinearPlan skinny = auto_plan(a.M < 16 ? a.M : 16, a.N, a.K, a.bits, a.g, (size_t)device_max_lds(), 1);
    skinny.prefetch = 1; skinny.m_rows16 = 1; skinny.n_tiles16 = 1;
    skinny.m_blocks = (int)((a.M + 15) / 16);
    if (a.M > 16) skinny.split_k = 1;
    if (a.M > 16 && (a.g % 128 == 0 || small_groups(a.M, a.g))) {
        LinearPlan h;
        bool keep = false;
        if (a.g % 128 != 0) {
            wide_plan(a.M, a.N, a.K, a.bits, a.g, &h);        // the shapes that the small groups' models compare
            h.waves_n = 8; h.n_tiles16 = std::min(h.n_tiles16, 2);
            keep = skinny_on_small_groups(a, skinny, h);
        }
        if (!keep) {
            const size_t cap = a.M >= 64 && a.g % 128 == 0 ? kWorkspaceCapTall : kWorkspaceCap;
            const size_t fit = a.workspace ? std::min(workspace_nbytes, cap) : 0;
            static Remembered<LinearPlan> remembered;
            h = remembered.get({a.M, a.N, a.K, a.g, fit, 0, a.bits, 0}, [&] {
                LinearPlan b;
                block_or_wide_plan(a.M, a.N, a.K, a.bits, a.g, fit, true, &b);
                return b;
            });
            const rtn_linear_cfg cfg = plan_cfg(h);
            if (resolve_plan(a, &cfg, workspace_nbytes, p) == RTN_OK) return RTN_OK;
        }
    }
    const rtn_linear_cfg cfg = plan_cfg(skinny);
    return resolve_plan(a, &cfg, workspace_nbytes, p);
}

// The one or two launches of a call, in order, with their plans.
rtn_status linear_launches(const LinearArgs& a, const rtn_linear_cfg* cfg, size_t workspace_nbytes, LinearArgs part[2],
                           LinearPlan plan[2], int* n) {
    *n = 1;
    part[0] = a;
    rtn_status st = resolve_plan(a, cfg, workspace_nbytes, &plan[0]);
    if (st != RTN_OK || cfg || plan[0].path != 4) return st;
    const int64_t rows_first = tile_two_launches(false, a.M, a.N, a.K, tile_workspace(a, workspace_nbytes));
    if (rows_first == 0) return RTN_OK;
    rtn_linear_cfg tile_cfg = {};
    tile_cfg.path = 4;
    *n = 2;
    for (int i = 0; i < 2 && st == RTN_OK; ++i) {
        const int64_t r0 = i == 0 ? 0 : rows_first;
        part[i] = a;
        part[i].M = i == 0 ? rows_first : a.M - rows_first;
        part[i].A = static_cast<const char*>(a.A) + (size_t)r0 * a.K * 2;
        part[i].C = static_cast<char*>(a.C) + (size_t)r0 * a.N * 2;
        st = resolve_plan(part[i], &tile_cfg, workspace_nbytes, &plan[i]);
    }
    return st;
}

// ---- split-K partial sums for the entry point that allocates nothing ----------------------------------------------
// A fixed device array takes the place of the caller's workspace.  Every GPU the library runs on holds its own copy
// (at its own address) until the process ends.  In host code the array's name is only a handle for the runtime: the
// device address is looked up once per device, with that device current, and kept; kernels and everything else
// only ever see that address.
constexpr size_t kScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices];
std::mutex g_scratch_mutex;

rtn_status scratch_for_current_device(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return RTN_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return RTN_ERR_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return RTN_OK;
}

}  // namespace

extern "C" {

const char* rtn_status_str(rtn_status s) {
    switch (static_cast<int>(s)) {             // callers from C or a foreign-function interface may pass any integer
        case RTN_OK: return "ok";
        case RTN_ERR_NULL: return "null pointer";
        case RTN_ERR_BITS: return "bits must be 4 or 8";
        case RTN_ERR_GROUP: return "unsupported group size";
        case RTN_ERR_SHAPE: return "unsupported shape";
        case RTN_ERR_ALIGN: return "device pointer not 16-byte aligned";
        case RTN_ERR_WORKSPACE: return "workspace too small";
        case RTN_ERR_CONFIG: return "invalid kernel configuration";
        case RTN_ERR_HIP: return "HIP launch error";
    }
    return "unknown status";
}

int rtn_layout_version(void) { return 1; }

size_t rtn_qweight_nbytes(int64_t N, int64_t K, int bits) {
    int64_t g;
    if (check_problem(N, K, bits, 0, &g) != RTN_OK) return 0;
    return (size_t)N * (size_t)K * (size_t)bits / 8;
}

size_t rtn_scales_nbytes(int64_t N, int64_t K, int group_size) {
    if (N <= 0 || K <= 0) return 0;
    int64_t g = group_size <= 0 ? K : group_size;
    if (g > K || K % g != 0) return 0;
    return (size_t)N * (size_t)(K / g) * 2;
}

size_t rtn_workspace_nbytes(int64_t M, int64_t N, int64_t K, int bits, int group_size) {
    int64_t g;
    if (M <= 0 || check_problem(N, K, bits, group_size, &g) != RTN_OK) return 0;
    const LinearPlan p = auto_plan(M, N, K, bits, g, (size_t)device_max_lds());
    return std::max(workspace_bound(M, N), std::max(plan_partials(p, M, N, K), wide_or_tile_partials(M, N, K, bits, g)));
}

rtn_status rtn_quantize(const void* dev_W, int64_t N, int64_t K, int bits, int group_size, int flags,
                        void* dev_qweight, void* dev_scales, void* stream) {
    if (!dev_W || !dev_qweight || !dev_scales) return RTN_ERR_NULL;
    int64_t g;
    rtn_status st = check_problem(N, K, bits, group_size, &g);
    if (st != RTN_OK) return st;
    if (flags != RTN_SCALE_QMAX && flags != RTN_SCALE_EQ2) return RTN_ERR_CONFIG;
    if (!aligned16(dev_W) || !aligned16(dev_qweight) || !aligned16(dev_scales)) return RTN_ERR_ALIGN;
    const float qmax = (float)((1 << (bits - 1)) - 1);
    const float divisor = (flags == RTN_SCALE_EQ2) ? qmax + 0.5f : qmax;
    hipError_t e = rtn::launch_quantize(dev_W, N, K, bits, g, divisor, dev_qweight, dev_scales,
                                        static_cast<hipStream_t>(stream));
    return e == hipSuccess ? RTN_OK : RTN_ERR_HIP;
}

rtn_status rtn_linear_ex(const void* dev_A, int64_t M, const void* dev_qweight, const void* dev_scales,
                         int64_t N, int64_t K, int bits, int group_size, void* dev_C,
                         void* dev_workspace, size_t workspace_nbytes, void* stream,
                         const rtn_linear_cfg* cfg) {
    if (!dev_A || !dev_qweight || !dev_scales || !dev_C) return RTN_ERR_NULL;
    int64_t g;
    rtn_status st = check_problem(N, K, bits, group_size, &g);
    if (st != RTN_OK) return st;
    if (M <= 0 || M > (1 << 20)) return RTN_ERR_SHAPE;
    if (!aligned16(dev_A) || !aligned16(dev_qweight) || !aligned16(dev_scales) || !aligned16(dev_C) ||
        !aligned16(dev_workspace))
        return RTN_ERR_ALIGN;
    LinearArgs a;
    a.A = dev_A; a.qweight = dev_qweight; a.scales = dev_scales; a.C = dev_C;
    a.workspace = static_cast<float*>(dev_workspace);
    a.M = M; a.N = N; a.K = K; a.g = g; a.bits = bits;
    LinearArgs part[2];
    LinearPlan plan[2];
    int n;
    st = linear_launches(a, cfg, workspace_nbytes, part, plan, &n);
    if (st != RTN_OK) return st;
    for (int i = 0; i < n; ++i)
        if (rtn::launch_linear(part[i], plan[i], static_cast<hipStream_t>(stream)) != hipSuccess) return RTN_ERR_HIP;
    return RTN_OK;
}

rtn_status rtn_linear(const void* dev_A, int64_t M, const void* dev_qweight, const void* dev_scales,
                      int64_t N, int64_t K, int bits, int group_size, void* dev_C,
                      void* dev_workspace, size_t workspace_nbytes, void* stream) {
    return rtn_linear_ex(dev_A, M, dev_qweight, dev_scales, N, K, bits, group_size, dev_C, dev_workspace,
                         workspace_nbytes, stream, nullptr);
}

rtn_status rtn_problem_status(int64_t N, int64_t K, int bits, int group_size) {
    int64_t g;
    return check_problem(N, K, bits, group_size, &g);
}

rtn_status rtn_linear_validate(int64_t M, int64_t N, int64_t K, int bits, int group_size, size_t workspace_nbytes,
                               const rtn_linear_cfg* cfg) {
    int64_t g;
    rtn_status st = check_problem(N, K, bits, group_size, &g);
    if (st != RTN_OK) return st;
    if (M <= 0 || M > (1 << 20)) return RTN_ERR_SHAPE;
    LinearArgs a;
    a.A = nullptr; a.qweight = nullptr; a.scales = nullptr; a.C = nullptr;
    // only "is there a workspace" matters to the plan checks; nothing is launched and the address is never used
    static float workspace_stand_in;
    a.workspace = workspace_nbytes > 0 ? &workspace_stand_in : nullptr;
    a.M = M; a.N = N; a.K = K; a.g = g; a.bits = bits;
    LinearPlan p;
    return resolve_plan(a, cfg, workspace_nbytes, &p);
}

rtn_status rtn_linear_noalloc(const void* dev_A, int64_t M, const void* dev_qweight, const void* dev_scales,
                              int64_t N, int64_t K, int bits, int group_size, void* dev_C, void* stream) {
    if (!dev_A || !dev_qweight || !dev_scales || !dev_C) return RTN_ERR_NULL;
    int64_t g;
    rtn_status st = check_problem(N, K, bits, group_size, &g);
    if (st != RTN_OK) return st;
    if (M <= 0 || M > (1 << 20)) return RTN_ERR_SHAPE;
    // from 144 tiles of 128 x 256, which occupy the chip without a split, the call runs with the splits that fit the array
    if (((N + 255) / 256) * ((M + 127) / 128) < 144 && wide_or_tile_partials(M, N, K, bits, g) > kScratchBytes)
        return RTN_ERR_WORKSPACE;
    void* ptr = nullptr;
    st = scratch_for_current_device(&ptr);
    if (st != RTN_OK) return st;
    return rtn_linear_ex(dev_A, M, dev_qweight, dev_scales, N, K, bits, group_size, dev_C, ptr, kScratchBytes, stream,
                         nullptr);
}

rtn_status rtn_linear_query(int64_t M, int64_t N, int64_t K, int bits, int group_size, rtn_linear_cfg* out) {
    if (!out) return RTN_ERR_NULL;
    int64_t g;
    rtn_status st = check_problem(N, K, bits, group_size, &g);
    if (st != RTN_OK) return st;
    if (M <= 0 || M > (1 << 20)) return RTN_ERR_SHAPE;
    if ((uint64_t)N * K * bits / 8 >= 0x7FFF0000ull || (uint64_t)M * K * 2 >= 0x7FFF0000ull)
        return RTN_ERR_SHAPE;                                   // what rtn_linear refuses (32-bit buffer offsets)
    LinearPlan p = auto_plan(M, N, K, bits, g, (size_t)device_max_lds());
    *out = plan_cfg(p);
    return RTN_OK;
}

rtn_status rtn_unpack(const void* dev_qweight, int64_t N, int64_t K, int bits, void* dev_codes_i8, void* stream) {
    if (!dev_qweight || !dev_codes_i8) return RTN_ERR_NULL;
    int64_t g;
    rtn_status st = check_problem(N, K, bits, 0, &g);
    if (st != RTN_OK) return st;
    if (!aligned16(dev_qweight) || !aligned16(dev_codes_i8)) return RTN_ERR_ALIGN;
    hipError_t e = rtn::launch_unpack(dev_qweight, nullptr, N, K, bits, K, false, dev_codes_i8,
                                      static_cast<hipStream_t>(stream));
    return e == hipSuccess ? RTN_OK : RTN_ERR_HIP;
}

rtn_status rtn_dequantize(const void* dev_qweight, const void* dev_scales, int64_t N, int64_t K, int bits,
                          int group_size, void* dev_W_fp16, void* stream) {
    if (!dev_qweight || !dev_scales || !dev_W_fp16) return RTN_ERR_NULL;
    int64_t g;
    rtn_status st = check_problem(N, K, bits, group_size, &g);
    if (st != RTN_OK) return st;
    if (!aligned16(dev_qweight) || !aligned16(dev_scales) || !aligned16(dev_W_fp16)) return RTN_ERR_ALIGN;
    hipError_t e = rtn::launch_unpack(dev_qweight, dev_scales, N, K, bits, g, true, dev_W_fp16,
                                      static_cast<hipStream_t>(stream));
    return e == hipSuccess ? RTN_OK : RTN_ERR_HIP;
}

size_t rtn_quantize_host_staging_nbytes(int64_t K, int64_t rows_per_shard) {
    if (K <= 0 || rows_per_shard <= 0 || rows_per_shard % 16 != 0) return 0;
    return 2 * (size_t)rows_per_shard * (size_t)K * 2;
}

rtn_status rtn_quantize_from_host(const void* host_W, int64_t N, int64_t K, int bits, int group_size, int flags,
                                  void* dev_qweight, void* dev_scales, void* dev_staging, size_t staging_nbytes,
                                  int64_t rows_per_shard, void* stream, void* copy_stream) {
    if (!host_W || !dev_qweight || !dev_scales || !dev_staging) return RTN_ERR_NULL;
    int64_t g;
    rtn_status st = check_problem(N, K, bits, group_size, &g);
    if (st != RTN_OK) return st;
    if (flags != RTN_SCALE_QMAX && flags != RTN_SCALE_EQ2) return RTN_ERR_CONFIG;
    if (rows_per_shard <= 0 || rows_per_shard % 16 != 0) return RTN_ERR_SHAPE;
    if (!aligned16(dev_qweight) || !aligned16(dev_scales) || !aligned16(dev_staging)) return RTN_ERR_ALIGN;
    if (staging_nbytes < rtn_quantize_host_staging_nbytes(K, rows_per_shard)) return RTN_ERR_WORKSPACE;
    if (stream == copy_stream) return RTN_ERR_CONFIG;          // the overlap needs two streams
    hipStream_t qs = static_cast<hipStream_t>(stream), cs = static_cast<hipStream_t>(copy_stream);
    const float qmax = (float)((1 << (bits - 1)) - 1);
    const float divisor = (flags == RTN_SCALE_EQ2) ? qmax + 0.5f : qmax;
    const size_t shard_bytes = (size_t)rows_per_shard * K * 2;
    hipEvent_t ev[5] = {nullptr, nullptr, nullptr, nullptr, nullptr};   // start, copied[0..1], consumed[0..1]
    bool ok = true;
    for (int i = 0; i < 5 && ok; ++i) ok = hipEventCreateWithFlags(&ev[i], hipEventDisableTiming) == hipSuccess;
    if (!ok) {                                                  // destroy what was created before the failure
        for (int i = 0; i < 5; ++i)
            if (ev[i]) (void)hipEventDestroy(ev[i]);
        return RTN_ERR_HIP;
    }
    hipEvent_t start = ev[0], *copied = &ev[1], *consumed = &ev[3];
    // the copy stream starts after whatever the caller queued on `stream` before this call (the staging buffer
    // may still be in use there)
    ok = hipEventRecord(start, qs) == hipSuccess && hipStreamWaitEvent(cs, start, 0) == hipSuccess;
    int64_t shard = 0;
    for (int64_t r0 = 0; r0 < N && ok; r0 += rows_per_shard, ++shard) {
        const int b = (int)(shard & 1);
        const int64_t rows = (N - r0 < rows_per_shard) ? N - r0 : rows_per_shard;
        uint8_t* stage = static_cast<uint8_t*>(dev_staging) + (size_t)b * shard_bytes;
        // copy shard -> staging buffer b, once the quantise pass that last read buffer b is done
        if (shard >= 2) ok = ok && hipStreamWaitEvent(cs, consumed[b], 0) == hipSuccess;
        ok = ok && hipMemcpyAsync(stage, static_cast<const uint8_t*>(host_W) + (size_t)r0 * K * 2, (size_t)rows * K * 2,
                                  hipMemcpyHostToDevice, cs) == hipSuccess;
        ok = ok && hipEventRecord(copied[b], cs) == hipSuccess;
        // quantise it on `stream` into its slice of the packed tensor (tile-rows and scale rows are contiguous)
        ok = ok && hipStreamWaitEvent(qs, copied[b], 0) == hipSuccess;
        if (ok) {
            uint8_t* qdst = static_cast<uint8_t*>(dev_qweight) + (size_t)r0 * K * bits / 8;
            uint8_t* sdst = static_cast<uint8_t*>(dev_scales) + (size_t)r0 * (K / g) * 2;
            ok = rtn::launch_quantize(stage, rows, K, bits, g, divisor, qdst, sdst, qs) == hipSuccess;
        }
        ok = ok && hipEventRecord(consumed[b], qs) == hipSuccess;
    }
    (void)hipEventDestroy(start);
    for (int i = 0; i < 2; ++i) {
        (void)hipEventDestroy(copied[i]);                       // destruction is deferred until the events complete
        (void)hipEventDestroy(consumed[i]);
    }
    return ok ? RTN_OK : RTN_ERR_HIP;
}

rtn_status rtn_gemm_fp16(const void* dev_A, int64_t M, const void* dev_W_fp16, int64_t N, int64_t K, void* dev_C,
                         void* dev_workspace, size_t workspace_nbytes, void* stream) {
    if (!dev_A || !dev_W_fp16 || !dev_C) return RTN_ERR_NULL;
    if (M <= 0 || M > (1 << 20) || N <= 0 || N % 16 != 0 || K <= 0 || K % 128 != 0) return RTN_ERR_SHAPE;
    if ((uint64_t)K * 2 * 128 >= 0x7FFF0000ull) return RTN_ERR_SHAPE;          // one 128-row slab per buffer resource
    if (!aligned16(dev_A) || !aligned16(dev_W_fp16) || !aligned16(dev_C) || !aligned16(dev_workspace)) return RTN_ERR_ALIGN;
    const int64_t rows_first = dev_workspace ? tile_two_launches(true, M, N, K, workspace_nbytes) : 0;
    for (int part = 0; part < (rows_first > 0 ? 2 : 1); ++part) {
        const int64_t r0 = part == 0 ? 0 : rows_first, rows = rows_first == 0 ? M : part == 0 ? rows_first : M - rows_first;
        int r16, split;
        tile_plan_choose(true, rows, N, K, dev_workspace ? workspace_nbytes : 0, &r16, &split);
        if (rtn::launch_gemm_fp16(static_cast<const char*>(dev_A) + (size_t)r0 * K * 2, dev_W_fp16,
                                  static_cast<char*>(dev_C) + (size_t)r0 * N * 2, static_cast<float*>(dev_workspace),
                                  rows, N, K, r16, split, static_cast<hipStream_t>(stream)) != hipSuccess)
            return RTN_ERR_HIP;
    }
    return RTN_OK;
}

size_t rtn_dense_weight_nbytes(int64_t N, int64_t K) {
    if (N <= 0 || K <= 0) return 0;
    return (size_t)N * (size_t)K * 2;
}

rtn_status rtn_linear_dense(const void* dev_A, int64_t M, const void* dev_qweight, const void* dev_scales,
                            int64_t N, int64_t K, int bits, int group_size, void* dev_C, void* dev_W_tmp,
                            size_t w_tmp_nbytes, void* dev_workspace, size_t workspace_nbytes, void* stream) {
    if (!dev_W_tmp) return RTN_ERR_NULL;
    if (w_tmp_nbytes < rtn_dense_weight_nbytes(N, K)) return RTN_ERR_WORKSPACE;
    rtn_status st = rtn_dequantize(dev_qweight, dev_scales, N, K, bits, group_size, dev_W_tmp, stream);
    if (st != RTN_OK) return st;
    return rtn_gemm_fp16(dev_A, M, dev_W_tmp, N, K, dev_C, dev_workspace, workspace_nbytes, stream);
}

// Checks of one module that need no plan, and its kernel arguments.
static rtn_status module_args(const rtn_module& m, void* dev_workspace, LinearArgs* a) {
    if (!m.dev_A || !m.dev_qweight || !m.dev_scales || !m.dev_C) return RTN_ERR_NULL;
    int64_t g;
    rtn_status st = check_problem(m.N, m.K, m.bits, m.group_size, &g);
    if (st != RTN_OK) return st;
    if (m.M <= 0 || m.M > (1 << 20)) return RTN_ERR_SHAPE;
    if (!aligned16(m.dev_A) || !aligned16(m.dev_qweight) || !aligned16(m.dev_scales) || !aligned16(m.dev_C)) return RTN_ERR_ALIGN;
    a->A = m.dev_A; a->qweight = m.dev_qweight; a->scales = m.dev_scales; a->C = m.dev_C;
    a->workspace = static_cast<float*>(dev_workspace);
    a->M = m.M; a->N = m.N; a->K = m.K; a->g = g; a->bits = m.bits;
    return RTN_OK;
}

// Whether running the modules in any order, or at once, gives what running them in order gives: no output overlaps an
// operand or an output of another module.
static bool modules_independent(const LinearArgs* a, int n) {
    struct Range { uintptr_t lo, hi; };
    auto range = [](const void* p, size_t bytes) { const uintptr_t lo = reinterpret_cast<uintptr_t>(p); return Range{lo, lo + bytes}; };
    auto meet = [](const Range& x, const Range& y) { return x.lo < y.hi && y.lo < x.hi; };
    for (int i = 0; i < n; ++i) {
        const Range out = range(a[i].C, (size_t)a[i].M * a[i].N * 2);
        for (int j = 0; j < n; ++j) {
            if (j == i) continue;
            if (meet(out, range(a[j].A, (size_t)a[j].M * a[j].K * 2)) || meet(out, range(a[j].C, (size_t)a[j].M * a[j].N * 2)) ||
                meet(out, range(a[j].qweight, (size_t)a[j].N * a[j].K * a[j].bits / 8)) ||
                meet(out, range(a[j].scales, (size_t)a[j].N * (a[j].K / a[j].g) * 2)))
                return false;
        }
    }
    return true;
}

static int64_t module_blocks(const LinearArgs& a, const LinearPlan& p) { return (a.N / 16 + p.waves_n - 1) / p.waves_n; }

// Whether a merged launch costs more than the launches it saves.  Its workgroups are taken to run one to a compute unit; the
// few of a last round leave the others idle for the time of the longest of them, at the 6.5 TB/s that the launch streams
// at (two modules in 258 workgroups, int4 at four rows: 14.3 us apart, 19.3 merged; 5120 x 17408 beside a small module, int8
// at one to four rows: 22-24 against 24-28).  Drawn from 1048 sets of two to seven modules: all 28 that ran slower merged (up
// to 1.38 x) lie beyond the line, and ten that gained 6-21 %; of 500 further sets merging slowed 22 by 3-30 %, 20 of them
// beyond it.  From five rows a matrix of 40 MB beside a module that hardly matters is also better served by its own plan
// (21 us against 26).
static bool merge_loses(const LinearArgs* a, const LinearPlan* plans, int n, int64_t rows, int64_t steps, double stream_us) {
    constexpr int64_t kCus = 256;
    int64_t blocks = 0, largest = 0, load = 0;
    for (int i = 0; i < n; ++i) {
        blocks += module_blocks(a[i], plans[i]);
        largest = std::max(largest, a[i].N / 16 * (a[i].K / chunk_k(a[i].bits)));
    }
    const int64_t last = blocks > kCus ? blocks % kCus : 0;
    int64_t left = last;
    for (int i = n - 1; i >= 0 && left > 0; --i) {
        load = std::max(load, plans[i].waves_n * (a[i].K / chunk_k(a[i].bits)));
        left -= module_blocks(a[i], plans[i]);
    }
    const double idle_us = last == 0 ? 0.0 : (double)((kCus - last) * load) / (double)steps * stream_us;
    return idle_us > 6.5 * (n - 1) - 2.0 || (n == 2 && rows > 4 && largest > 0.9 * steps && stream_us > 6.0);
}

// Independent modules of one precision and group size in one launch, up to eight rows, 256 MB of weights and 140 KiB of
// activations a module (14336 columns at five rows): a launch costs 4-5 us of start, ramp and drain around its weight
// stream, which one grid over all modules pays once.  Plan of the merged modules: a wavefront takes so many k-chunks that
// there are about 3456 of them in all (6912 from five rows), in workgroups of up to 16 (13) wavefronts, fewer where that
// leaves compute units without one; wavefronts that an even share of the chunks leaves without any are left out (with
// them a 2048-wide layer, int4 at one row, took 11.1 us instead of 10.4, and its slice of 8192 columns at six rows did not
// fit the LDS: 20.2 us instead of 15.2); two chunks in flight, one at 4 bit from five rows.  From sweeps over 4-16
// wavefronts per workgroup and 2-28 chunks per wavefront.  Graph replay over rotating copies, single launches against one:
// 8B layer int4 30.8 -> 22.6 us at one row, 32.9 -> 23.5 at four, 35.4 -> 29.3 at five; int8 44.0 -> 37.5, 47.0 -> 37.9,
// 50.1 -> 41.6; the 2048-wide layer int4 17.3 -> 10.3, 18.9 -> 10.8, 19.9 -> 15.5 at eight; three modules of 4096 columns and
// 4096, 1024, 1024 rows 11.8 -> 5.5 at one row, two of 4096 x 1024 6.3 -> 3.6.
// Beyond the line the modules' own plans are better: from nine rows the staged activations want their shapes (8B int4 at
// 16: 38.5 us against 38.9 at best), 70B and 405B modules lose more by a common shape than they gain (82 -> 86 and
// 268 -> 297 at two rows), and so do slices that do not fit the LDS at once (28672 columns at four rows, int8: 30 -> 36).
static bool merged_layer_plans(const LinearArgs* a, int n, size_t workspace_nbytes, LinearPlan* plans) {
    int64_t rows = 0;
    size_t bytes = 0;
    for (int i = 0; i < n; ++i) {
        rows = std::max(rows, a[i].M);
        bytes += (size_t)a[i].N * a[i].K * a[i].bits / 8;
    }
    if (rows > 8 || bytes >= ((size_t)256 << 20)) return false;
    for (int i = 0; i < n; ++i)
        if ((size_t)a[i].M * a[i].K * 2 > (size_t)140 << 10) return false;
    auto same_class = [](const LinearArgs& x, const LinearArgs& y) {       // one kernel instantiation: bits and groups per chunk
        const int64_t ck = chunk_k(x.bits);
        return x.bits == y.bits && (x.g >= ck ? 1 : ck / x.g) == (y.g >= ck ? 1 : ck / y.g);
    };
    int64_t steps = 0, waves = 0;
    for (int i = 0; i < n; ++i) steps += a[i].N / 16 * (a[i].K / chunk_k(a[i].bits));
    const double chunks = std::max(1.0, (double)steps / (rows <= 4 ? 3456.0 : 6912.0));
    auto waves_k = [&](const LinearArgs& x) {
        return (int)std::max(1.0, std::min(16.0, std::floor((double)(x.K / chunk_k(x.bits)) / chunks + 0.5)));
    };
    for (int i = 0; i < n; ++i) waves += a[i].N / 16 * waves_k(a[i]);
    const int64_t width = rows <= 4 ? std::min<int64_t>(16, std::max<int64_t>(1, waves / 216)) : std::min<int64_t>(13, std::max<int64_t>(1, waves / 256));
    for (int i = 0; i < n; ++i) {
        if (!same_class(a[0], a[i])) return false;
        // the module's own plan: its errors (a workspace too small) are those of the call in order
        if (resolve_plan(a[i], nullptr, workspace_nbytes, &plans[i]) != RTN_OK) return false;
        rtn_linear_cfg cfg;
        cfg.path = 1; cfg.prefetch = chunks >= 2 && (rows <= 4 || a[i].bits == 8) ? 2 : 1;
        cfg.waves_k = waves_k(a[i]);
        cfg.waves_n = (int)std::max<int64_t>(1, std::min<int64_t>(width / cfg.waves_k, a[i].N / 16));
        const int64_t KC = a[i].K / chunk_k(a[i].bits), per = (KC + cfg.waves_k - 1) / cfg.waves_k;
        cfg.waves_k = (int)((KC + per - 1) / per);
        cfg.split_k = 1; cfg.m_rows16 = 1; cfg.n_tiles16 = 1;
        if (resolve_plan(a[i], &cfg, workspace_nbytes, &plans[i]) != RTN_OK) return false;
    }
    return !merge_loses(a, plans, n, rows, steps, (double)bytes / 6.5e6);
}

// Modelled time of a module's own plan.
static double own_plan_us(const LinearArgs& a, const LinearPlan& p, size_t workspace_nbytes) {
    const double packed = (double)a.N * a.K * a.bits / 8.0;
    if (p.path == 1)                                               // the skinny kernel, and the reduce pass of a K split, a launch of its own
        return 4.5 + packed / (a.bits == 8 ? 6.5e6 : a.M <= 16 ? 5.4e6 : 3.9e6) + (p.split_k > 1 ? 2.4 + (double)a.M * a.N * p.split_k * 8.0 / 4.2e6 : 0.0);
    if (p.path == 4) {
        double t;
        tile_two_launches(false, a.M, a.N, a.K, tile_workspace(a, workspace_nbytes), &t);
        return 1.03 * t;
    }
    if (p.n_tiles16 == 1) return wide16_model_us(a.M, a.N, a.K, a.bits, a.g, p.m_rows16, p.split_k);
    return block_model_us(a.M, a.N, a.K, a.bits, a.g, p.m_rows16, p.waves_k, p.split_k);
}

// Independent modules of one precision and number of groups per unit in one launch of the block kernel.  Apart, each fills the
// chip to a half or three quarters and pays the start, the first data and the last store of a launch; together they fill it and
// pay once.  Plan: one height of the tallest row tiles for all (a launch is one kernel), wavefronts along K by module, the longest
// workgroups first, K of the modules with the longest split in up to six.  The time is about the mean of the end of the last workgroup,
// when those of the fullest XCD are dealt in that order to its compute units (32; two of the 32-row ones on each), and the
// average load (the clock is higher while part of the chip is idle); against it the streams.  The fullest XCD is counted as the launch
// deals the tiles, module by module and split by split: 7168-, 5120-, 27648- and 5120-wide modules with K of the last in four are 236
// workgroups, but 33 on one XCD, and took 73 us at 12 rows where their own launches take 64.
struct MergedPlan {
    double us;                          // modelled time, negative: no such plan
    int mb, wk;                         // row blocks of 32 rows (the tile kernel: 16-row blocks per wavefront), least wavefronts along K
    int waves[rtn::kMaxBlockGroup];     // wavefronts along K of each
    int split[rtn::kMaxBlockGroup];
};

// No heap: a C entry point has no way to report that it ran out.
constexpr int64_t kMostSlots = 64;
static double dealt_us(const double* each, const int64_t* count, int n, int64_t slots, double last) {
    struct Load { double end; int64_t slots; };
    Load load[kMostSlots];                                      // by end; each has a slot at least
    int loads = 1, order[2 * rtn::kMaxBlockGroup];
    load[0] = {0.0, slots};
    for (int i = 0; i < n; ++i) {                               // longest first
        int at = i;
        for (; at > 0 && each[order[at - 1]] < each[i]; --at) order[at] = order[at - 1];
        order[at] = i;
    }
    double sum = 0.0;
    for (int k = 0; k < n; ++k) {
        int64_t left = count[order[k]];
        const double d = each[order[k]];
        while (k + 1 < n && each[order[k + 1]] == d && left + count[order[k + 1]] <= 64 * slots) left += count[order[++k]];    // like modules
        sum += d * left;
        if (left > 64 * slots) {                                // many rounds: the load is even to a round
            for (int i = 0; i < loads; ++i) load[i].end += d * (double)(left / slots - 32);
            left -= (left / slots - 32) * slots;
        }
        while (left > 0) {
            const Load first = load[0];
            const int64_t k2 = std::min(first.slots, left);
            if (k2 == first.slots) std::copy(load + 1, load + loads--, load);
            else load[0].slots -= k2;
            int at = 0;
            while (at < loads && load[at].end < first.end + d - 1e-9) ++at;
            if (at < loads && load[at].end < first.end + d + 1e-9) {
                load[at].slots += k2;
            } else {
                std::copy_backward(load + at, load + loads, load + loads + 1);
                load[at] = {first.end + d, k2};
                ++loads;
            }
            left -= k2;
        }
    }
    return last * load[loads - 1].end + (1.0 - last) * sum / (double)slots;
}

// What the time of a launch is made of, fitted for launches of up to 16 rows, of which a workgroup stages no more, and for others.
struct BlockCosts {
    double start, unit[4], group[4], int8;     // a workgroup: its start, a unit of four packed tiles by row blocks, a scale group in it, an 8-bit unit
    double waves[4][3];                        // a unit with 2, 4, 8 wavefronts along K, by row blocks
    double rows, sum;                          // staging 32 rows for a unit, the sum over the wavefronts along K per row block
    double busy, shared, one;                  // slower on a full chip, two on a compute unit, 32-row workgroups
    double stream, norm, reduce, reduce_bw, launch, last;
};
static const BlockCosts kBlockCosts = {0.38, {2.607, 2.141, 2.770, 2.750}, {0.043, 0.168, 0.159, 0.280}, 0.739,
                                       {{1.031, 0.874, 1.120}, {0.956, 0.731, 0.908}, {0.909, 0.861, 1.0}, {0.796, 0.615, 1.0}}, 0.238, 0.226,
                                       0.353, 1.543, 0.955, 0.614, 1.890, 1.558, 6.906e6, 5.003, 0.519};
static const BlockCosts kBlockCosts16 = {0.636, {1.923, 0.0, 0.0, 0.0}, {0.063, 0.0, 0.0, 0.0}, 0.879,
                                         {{0.980, 0.801, 0.495}}, 0.021, 0.624, 0.322, 1.617, 0.967, 0.539, 1.495, 1.621, 6.083e6, 4.197, 0.780};

// Modelled time of m, negative where its partial sums do not fit; the module with the longest workgroups.  The workgroups of a part (row
// tiles of one height) are dealt longest first, as launch_blocks orders them, to the compute units of the fullest XCD.  Fitted to
// 2600 launches: the 8B, 70B and 405B layers in five formats at 5 to 512 rows, two to eight modules of 1024 to 8192 columns at 1 to 16
// rows (4 % rms; the pick is 0.9 % behind the best of 10 to 80 plans measured for each).  From `bound` on a lower bound of the time will do.
// floor: what no plan that shares K among more workgroups gets below (they add to the load and to the reduce pass).
static double merged_blocks_us(const LinearArgs* a, int n, const MergedPlan& m, size_t workspace, int* longest, double bound = INFINITY,
                               double* floor = nullptr) {
    int64_t most = 0;
    for (int i = 0; i < n; ++i) most = std::max(most, a[i].M);
    const BlockCosts& c = most <= 16 && m.mb == 1 ? kBlockCosts16 : kBlockCosts;
    double each[2 * rtn::kMaxBlockGroup], length = 0.0, stream = 0.0, reduce = 0.0;
    int64_t count[2 * rtn::kMaxBlockGroup], wgs = 0, on_xcd = 0;
    size_t partials = 0;
    int parts = 0;
    rtn::BlockTiles tiles[rtn::kMaxBlockGroup];
    for (int i = 0; i < n; ++i) {
        tiles[i] = rtn::block_tiles(a[i].M, a[i].N, m.mb, m.waves[i], m.split[i]);
        wgs += tiles[i].workgroups();
    }
    for (int i = 0; i < n; ++i) {
        const int s = m.split[i], wk = m.waves[i];
        const int64_t unit = chunk_k(a[i].bits);
        const double per = (double)(((a[i].K / unit + s - 1) / s + wk - 1) / wk), groups = a[i].g >= unit ? 1.0 : (double)(unit / a[i].g);
        const double waves = wk == 1 ? 1.0 : c.waves[m.mb - 1][wk == 2 ? 0 : wk == 4 ? 1 : 2];
        const rtn::BlockParts p = rtn::block_parts(tiles[i], m.mb, wgs <= 256);
        for (int h = 0; h < p.n; ++h) {                     // the row tiles of 32 mb rows, those of 32 rows less
            const int mb = p.part[h].tall > 0 ? m.mb : m.mb - 1;
            const double rows = (double)wk * std::min((double)a[i].M, 32.0 * mb) / 32.0;
            each[parts] = c.start + per * (c.unit[mb - 1] * (a[i].bits == 8 ? c.int8 : 1.0) * waves + c.group[mb - 1] * groups +
                                           c.rows * rows * (a[i].bits == 8 ? 0.5 : 1.0)) + (wk > 1 ? c.sum * mb : 0.0);
            count[parts] = p.part[h].on_xcd;
            on_xcd += count[parts];
            if (each[parts] > length) { length = each[parts]; *longest = i; }
            ++parts;
        }
        stream += c.stream * ((double)a[i].N * a[i].K * a[i].bits / 8.0 / 6.83e6 +
                              (double)tiles[i].columns * std::min<int64_t>((int64_t)tiles[i].rows * 32 * m.mb, (a[i].M + 31) / 32 * 32) * a[i].K * 2.0 / 1.71e7);
        if (s > 1) {
            reduce += c.reduce + (double)a[i].M * a[i].N * s * 8.0 / c.reduce_bw;
            partials += (((size_t)a[i].M * a[i].N * sizeof(float) * s) + 255) & ~(size_t)255;
        }
    }
    if (partials > workspace) return -1.0;
    const bool two = m.mb == 1;
    const double slow = (two ? c.one : 1.02) * (1.0 + c.busy * std::min(1.0, (double)wgs / 256.0) * m.mb / 4.0) * (two && on_xcd > 32 ? c.shared : 1.0);
    double load = 0.0;
    for (int i = 0; i < parts; ++i) {
        each[i] *= slow;
        load += each[i] * (double)count[i];
    }
    load /= two ? 64.0 : 32.0;
    const double end = c.last * std::max(load, length * slow) + (1.0 - c.last) * load;
    const double least = c.launch + std::sqrt(end * end + stream * stream) + reduce;       // (c.norm is under 2)
    if (floor) *floor = c.launch + std::sqrt(load * load + stream * stream) + reduce;
    if (least >= bound) return least;                           // no need to deal them out
    const double serial = dealt_us(each, count, parts, two ? 64 : 32, c.last);
    return c.launch + std::pow(std::pow(serial, c.norm) + std::pow(stream, c.norm), 1.0 / c.norm) + reduce;
}

// The plan with the lowest modelled time: row tile height (32 rows up to 96 rows, 128 from 65), wavefronts along K, and then the longest
// workgroups shorter step by step, K shared by more workgroups, before that in further passes by two wavefronts (up to 64 rows only
// where that is modelled 3 % ahead), and up to 8 rows by four: with more rows those are staged too late for the weights that four have in
// flight (8B layer with four for the down projection against one and four splits: 8 rows 26.6 us and 26.9, 16 rows 29.3 and 28.2, 32 rows
// 33.2 and 29.6).
static MergedPlan merged_blocks(const LinearArgs* a, int n, size_t workspace) {
    int64_t rows = 0, shortest = INT64_MAX;
    MergedPlan best;
    best.us = -1.0;
    double best_line = 0.0;
    for (int i = 0; i < n; ++i) {
        if (a[i].N >= (1 << 22)) return best;
        rows = std::max(rows, a[i].M);
        shortest = std::min(shortest, a[i].K / chunk_k(a[i].bits));
    }
    for (int r = 2, last_mb = 0; r <= 8; r *= 2) {
        if ((r == 2 && rows > 96) || (r == 8 && rows <= 64)) continue;
        const int64_t tiles = (rows + 16 * r - 1) / (16 * r);
        const int mb = (int)((rows + 32 * tiles - 1) / (32 * tiles));
        if (mb == last_mb) continue;                            // up to 32 rows: the same tiles
        last_mb = mb;
        for (int wk = 1; wk <= 8 && wk <= shortest; wk *= 2) {
            if (wk == 8 && mb > 2) continue;
            for (int deepen = 1; deepen <= (wk > 1 ? 1 : rows <= 8 ? 4 : 2); deepen *= 2) {
                MergedPlan m;
                m.mb = mb; m.wk = wk;
                for (int i = 0; i < n; ++i) { m.waves[i] = wk; m.split[i] = 1; }
                bool deep = false;
                for (int cuts = 0; cuts < 6; ++cuts) {
                    int longest = 0;
                    double floor;
                    m.us = merged_blocks_us(a, n, m, workspace, &longest, best.us < 0.0 ? INFINITY : best_line, &floor);
                    if (m.us < 0.0) break;
                    const double line = m.us * (deep && mb <= 2 ? 1.03 : 1.0);
                    if (best.us < 0.0 || line < best_line) { best = m; best_line = line; }
                    if (deepen == 1 && floor >= best_line) break;
                    const int s = m.split[longest];
                    const int64_t units = a[longest].K / chunk_k(a[longest].bits);
                    if (m.waves[longest] < deepen && deepen * s <= units) {
                        m.waves[longest] = deepen;
                        deep = deepen == 2;
                        continue;
                    }
                    m.split[longest] = s == 4 ? 6 : s + 1;
                    if (s >= 6 || (int64_t)m.split[longest] * m.waves[longest] > units) break;
                }
            }
        }
    }
    return best;
}

// Independent modules of one precision in one launch of the tile kernel: apart, every one ends in a round that fills the chip in
// part, or pays a second launch or a reduce pass to fill it.  One tile height for all, the longest workgroups first, K of the module
// with the longest split in two, four or eight.  Times of a workgroup as in tile_model_us, dealt to the compute units as above.
static MergedPlan merged_tiles(const LinearArgs* a, int n, size_t workspace) {
    MergedPlan best;
    best.us = -1.0;
    for (int r = 4; r <= 8; r += 4) {
        const double half = r == 8 ? 1.26 : 0.82, full = r == 8 ? 1.58 : 1.00;
        MergedPlan m;
        m.mb = r; m.wk = 0;
        for (int i = 0; i < n; ++i) { m.waves[i] = 0; m.split[i] = 1; }
        for (;;) {
            double each[rtn::kMaxBlockGroup], reduce = 0.0;
            int64_t count[rtn::kMaxBlockGroup], wgs = 0;
            size_t partials = 0;
            int longest = 0;
            for (int i = 0; i < n; ++i) {
                const int64_t s = m.split[i], mn = a[i].M * a[i].N;
                count[i] = (((a[i].N + 255) / 256) * ((a[i].M + 32 * r - 1) / (32 * r)) + 7) / 8 * s;
                wgs += 8 * count[i];
                each[i] = (double)((a[i].K / 64 + s - 1) / s);
                if (each[i] > each[longest]) longest = i;
                if (s > 1) {
                    reduce += 5.3 + (double)mn * (8.0 * s + 2.0) / 8.0e6;
                    partials += ((size_t)mn * sizeof(float) * s + 255) & ~(size_t)255;
                }
            }
            if (partials > workspace) break;
            const double step = half + (full - half) * std::max(0.0, std::min(1.0, (double)wgs / 128.0 - 1.0));
            const int64_t steps = (int64_t)each[longest];
            for (int i = 0; i < n; ++i) each[i] = each[i] * step + 6.0;
            m.us = 1.03 * (dealt_us(each, count, n, 32, 0.78) + reduce);
            if (best.us < 0.0 || m.us < best.us) best = m;
            if (m.split[longest] >= 8 || steps < 16) break;
            m.split[longest] *= 2;
        }
    }
    return best;
}

// The same, remembered (3 to 9 us of host time for four modules, 10 for eight): a table of fixed size, an entry gives way to the next one that falls on it.
static MergedPlan remembered_merge(const LinearArgs* a, int n, size_t workspace, bool tiles = false) {
    struct Key { int64_t v[4 * rtn::kMaxBlockGroup + 3]; };
    struct Entry { Key key; MergedPlan plan; bool used; };
    constexpr size_t kEntries = 512;
    static std::mutex mutex;
    static Entry table[kEntries];
    Key k = {};
    uint64_t h = 0;
    k.v[0] = n; k.v[1] = a[0].bits + (tiles ? 256 : 0); k.v[2] = a[0].workspace ? (int64_t)workspace : 0;
    for (int i = 0; i < n; ++i) { k.v[3 + 4 * i] = a[i].M; k.v[4 + 4 * i] = a[i].N; k.v[5 + 4 * i] = a[i].K; k.v[6 + 4 * i] = a[i].g; }
    for (int64_t v : k.v) h = (h ^ (uint64_t)v) * 0x9E3779B97F4A7C15ull, h ^= h >> 29;
    Entry& e = table[h % kEntries];
    {
        std::lock_guard<std::mutex> lock(mutex);
        if (e.used && memcmp(&e.key, &k, sizeof(k)) == 0) return e.plan;
    }
    const size_t cap = a[0].workspace ? workspace : 0;
    const MergedPlan p = tiles ? merged_tiles(a, n, cap) : merged_blocks(a, n, cap);
    std::lock_guard<std::mutex> lock(mutex);
    e.key = k; e.plan = p; e.used = true;
    return p;
}

static bool one_block_class(const LinearArgs& x, const LinearArgs& y) {
    const int64_t ck = chunk_k(x.bits);
    return x.bits == y.bits && (x.g >= ck ? 1 : ck / x.g) == (y.g >= ck ? 1 : ck / y.g);
}

static hipError_t launch_merged(const LinearArgs* set, int count, const MergedPlan& m, void* stream) {
    LinearPlan plans[rtn::kMaxBlockGroup];
    for (int k = 0; k < count; ++k) {
        LinearPlan& p = plans[k];
        p.path = 3; p.prefetch = 1; p.waves_n = 8; p.waves_k = m.waves[k]; p.split_k = m.split[k];
        p.m_rows16 = 2 * m.mb; p.n_tiles16 = 2;
        p.m_blocks = (int)((set[k].M + 32 * m.mb - 1) / (32 * m.mb));
    }
    return rtn::launch_linear_blocks(set, plans, count, m.mb, static_cast<hipStream_t>(stream));
}

static rtn_status one_module(const rtn_module& m, void* dev_workspace, size_t workspace_nbytes, void* stream) {
    return rtn_linear(m.dev_A, m.M, m.dev_qweight, m.dev_scales, m.N, m.K, m.bits, m.group_size, m.dev_C, dev_workspace,
                      workspace_nbytes, stream);
}

// One launch of a layer or a grouped call: a module alone (count 1), or several on the block or the tile kernel.
struct SharedLaunch {
    int count;
    int member[rtn::kMaxBlockGroup];
    MergedPlan plan;
};
static_assert(rtn::kMaxTileGroup == rtn::kMaxBlockGroup, "");

// The launches of n independent modules, in order of their first module: of those whose state is kOpen, modules of one class
// (precision, groups per unit; the tile kernel: precision) together where that is modelled ahead of their own plans' launches, the others
// one by one.  How far ahead (together_line): up to 16 rows 3 %, two modules 20 % (a plan that rtn_layer_forward has always had; of 36 pairs
// between 0.80 and 0.95 one measured more than 2 % slower together, and 0.94 on the mean); above 16 rows not at all, since the models have launches apart too fast there: of 63 drawn sets and 40 layers that
// they put between 0.97 and 1.066 two ran more than 2 % slower together (7 %), and they take 0.92 of the time on the mean (5120-wide layer
// int8 at 257 rows 243 us apart, 207; 70B layer int4 group 64 at 50 rows 161 and 137); from there to 1.08 every second set did.
// 8B layer int4 group 128, apart -> together: 9 rows 36.5 -> 28.4 us, 32 rows 48.3 -> 31.9, 64 61.6 -> 40.6, 128 85.1 -> 62.8; 70B layer
// 16 rows 98.8 -> 88.5, 32 110 -> 94; three modules of 4096 columns and 4096, 1024, 1024 rows at 32 rows 23.6 -> 9.2.  Tile kernel, 3 %:
// 8B layer int4 at 1536 rows 625 -> 553, 2048 rows 773 -> 726; 5120-wide layer at 2048 rows 996 -> 900; closer to level it measures
// within 1 % either way.
constexpr int64_t kMaxMergedRows = 512;
enum : char { kOpen, kSmall, kAlone, kDone };                   // kSmall: see grouped_blocks
// The line for sets of modules with that many rows at most: time together against time apart.
static double together_line(int count, int64_t rows, bool tiles) { return tiles ? 0.97 : rows > 16 ? 1.066 : count == 2 ? 0.80 : 0.97; }
static int shared_launches(const LinearArgs* args, const double* own_us, char* state, int n, size_t workspace_nbytes, bool tiles,
                           SharedLaunch* out) {
    int launches = 0;
    for (int i = 0; i < n; ++i) {
        if (state[i] == kDone) continue;
        SharedLaunch& l = out[launches++];
        LinearArgs set[rtn::kMaxBlockGroup];
        double apart = 0.0;
        int64_t rows = 0;
        l.count = 0;
        for (int j = i; state[i] == kOpen && j < n && l.count < rtn::kMaxBlockGroup; ++j) {
            if (state[j] != kOpen || !(tiles ? args[i].bits == args[j].bits : one_block_class(args[i], args[j]))) continue;
            apart += own_us[j];
            rows = std::max(rows, args[j].M);
            l.member[l.count] = j;
            set[l.count++] = args[j];
        }
        if (l.count > 1) l.plan = remembered_merge(set, l.count, tiles ? std::min(workspace_nbytes, kWorkspaceCapTile) : workspace_nbytes, tiles);
        const double line = together_line(l.count, rows, tiles);
        if (l.count < 2 || l.plan.us < 0.0 || l.plan.us > line * apart) {
            l.count = 1;
            l.member[0] = i;
        }
        for (int k = 0; k < l.count; ++k) state[l.member[k]] = kDone;
    }
    return launches;
}

// The launches of a layer of independent modules, all of 5 to 512 rows (block kernel) or all above (tile kernel: modules whose
// own plan is on it; other modules, whose weights are not rounded to fp16, keep their kernel).  -1 where the call runs in order: other
// rows, or a module whose own plan does not resolve (the call then stops at that error).
static int layer_launches(const LinearArgs* args, int n, size_t workspace_nbytes, SharedLaunch* out, bool* tiles) {
    constexpr int kMost = 16;
    double own_us[kMost];
    char state[kMost];
    if (n < 2 || n > kMost) return -1;
    *tiles = args[0].M > kMaxMergedRows;
    for (int i = 0; i < n; ++i) {
        LinearPlan own;
        if (args[i].M <= 4 || (args[i].M > kMaxMergedRows) != *tiles || resolve_plan(args[i], nullptr, workspace_nbytes, &own) != RTN_OK) return -1;
        own_us[i] = own_plan_us(args[i], own, workspace_nbytes);
        state[i] = !*tiles || own.path == 4 ? kOpen : kAlone;
    }
    return shared_launches(args, own_us, state, n, workspace_nbytes, *tiles, out);
}

static hipError_t launch_shared(const LinearArgs* args, const SharedLaunch& l, bool tiles, void* stream) {
    LinearArgs set[rtn::kMaxBlockGroup];
    for (int k = 0; k < l.count; ++k) set[k] = args[l.member[k]];
    return tiles ? rtn::launch_linear_tiles(set, l.plan.split, l.count, l.plan.mb, static_cast<hipStream_t>(stream))
                 : launch_merged(set, l.count, l.plan, stream);
}

rtn_status rtn_layer_forward(const rtn_module* mods, int n_mods, void* dev_workspace, size_t workspace_nbytes,
                             void* stream) {
    if (!mods) return RTN_ERR_NULL;
    if (n_mods <= 0) return RTN_ERR_SHAPE;
    constexpr int kMerge = 16;
    if (n_mods > 1 && n_mods <= kMerge && aligned16(dev_workspace)) {
        LinearArgs args[kMerge];
        LinearPlan plans[kMerge];
        bool ok = true;
        for (int i = 0; i < n_mods && ok; ++i) ok = mods[i].M <= 8 && module_args(mods[i], dev_workspace, &args[i]) == RTN_OK;
        if (ok && modules_independent(args, n_mods) && merged_layer_plans(args, n_mods, workspace_nbytes, plans)) {
            hipError_t e = rtn::launch_linear_grouped(args, plans, n_mods, true, static_cast<hipStream_t>(stream));
            return e == hipSuccess ? RTN_OK : RTN_ERR_HIP;
        }
    }
    if (n_mods > 1 && n_mods <= kMerge && aligned16(dev_workspace)) {
        LinearArgs args[kMerge];
        SharedLaunch launches[kMerge];
        bool ok = true, tiles;
        for (int i = 0; i < n_mods && ok; ++i) ok = module_args(mods[i], dev_workspace, &args[i]) == RTN_OK;
        const int n = ok && modules_independent(args, n_mods) ? layer_launches(args, n_mods, workspace_nbytes, launches, &tiles) : -1;
        for (int i = 0; i < n; ++i) {
            const SharedLaunch& l = launches[i];
            const rtn_status st = l.count == 1 ? one_module(mods[l.member[0]], dev_workspace, workspace_nbytes, stream)
                                : launch_shared(args, l, tiles, stream) == hipSuccess ? RTN_OK : RTN_ERR_HIP;
            if (st != RTN_OK) return st;
        }
        if (n >= 0) return RTN_OK;
    }
    for (int i = 0; i < n_mods; ++i) {
        const rtn_module& m = mods[i];
        rtn_status st = one_module(m, dev_workspace, workspace_nbytes, stream);
        if (st != RTN_OK) return st;
    }
    return RTN_OK;
}

rtn_status rtn_quantize_asym(const void* dev_W, int64_t N, int64_t K, int bits, int group_size,
                             void* dev_qweight, void* dev_scales, void* dev_zeros, void* stream) {
    if (!dev_W || !dev_qweight || !dev_scales || !dev_zeros) return RTN_ERR_NULL;
    int64_t g;
    rtn_status st = check_problem(N, K, bits, group_size, &g);
    if (st != RTN_OK) return st;
    if (!aligned16(dev_W) || !aligned16(dev_qweight) || !aligned16(dev_scales) || !aligned16(dev_zeros))
        return RTN_ERR_ALIGN;
    hipError_t e = rtn::launch_quantize_asym(dev_W, N, K, bits, g, dev_qweight, dev_scales, dev_zeros,
                                             static_cast<hipStream_t>(stream));
    return e == hipSuccess ? RTN_OK : RTN_ERR_HIP;
}

rtn_status rtn_dequantize_asym(const void* dev_qweight, const void* dev_scales, const void* dev_zeros,
                               int64_t N, int64_t K, int bits, int group_size, void* dev_W_fp16, void* stream) {
    if (!dev_qweight || !dev_scales || !dev_zeros || !dev_W_fp16) return RTN_ERR_NULL;
    int64_t g;
    rtn_status st = check_problem(N, K, bits, group_size, &g);
    if (st != RTN_OK) return st;
    if (!aligned16(dev_qweight) || !aligned16(dev_scales) || !aligned16(dev_zeros) || !aligned16(dev_W_fp16))
        return RTN_ERR_ALIGN;
    hipError_t e = rtn::launch_unpack(dev_qweight, dev_scales, N, K, bits, g, true, dev_W_fp16,
                                      static_cast<hipStream_t>(stream), dev_zeros);
    return e == hipSuccess ? RTN_OK : RTN_ERR_HIP;
}

rtn_status rtn_linear_asym(const void* dev_A, int64_t M, const void* dev_qweight, const void* dev_scales,
                           const void* dev_zeros, int64_t N, int64_t K, int bits, int group_size,
                           void* dev_C, void* dev_workspace, size_t workspace_nbytes, void* stream) {
    if (!dev_A || !dev_qweight || !dev_scales || !dev_zeros || !dev_C) return RTN_ERR_NULL;
    int64_t g;
    rtn_status st = check_problem(N, K, bits, group_size, &g);
    if (st != RTN_OK) return st;
    if (M <= 0 || M > (1 << 20)) return RTN_ERR_SHAPE;
    if (!aligned16(dev_A) || !aligned16(dev_qweight) || !aligned16(dev_scales) || !aligned16(dev_zeros) ||
        !aligned16(dev_C) || !aligned16(dev_workspace))
        return RTN_ERR_ALIGN;
    LinearArgs a;
    a.A = dev_A; a.qweight = dev_qweight; a.scales = dev_scales; a.C = dev_C; a.zeros = dev_zeros;
    a.workspace = static_cast<float*>(dev_workspace);
    a.M = M; a.N = N; a.K = K; a.g = g; a.bits = bits;
    LinearPlan p;
    st = resolve_plan_zp(a, workspace_nbytes, &p);
    if (st != RTN_OK) return st;
    hipError_t e = rtn::launch_linear(a, p, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? RTN_OK : RTN_ERR_HIP;
}

// One launch of the small-batch kernel for alike modules (N, K, precision and groups; up to sixteen of 1 to 16 rows): one workgroup shape for
// all of them.  A plan of each module's own leaves out that its workgroups share compute units with the others': every one gets the LDS of
// the largest slice, so eight modules of 2048 x 7168 with 1 to 8 rows were 224 workgroups of 4 x 4 wavefronts and, for the one-row module,
// 128 of 1 x 7, one a compute unit: a second round for 96 of them (16.6 us; as 256 of 4 x 3 13.5).  Modelled time: a start, 0.77 us for every
// further round, the weights at 7.2 TB/s (8 bit: 9.2) by what the fullest compute unit streams over the mean, what the wavefronts in
// flight can request, the staged rows at 11.4 TB/s, 0.15 us per thousand wavefronts; modules whose slice takes several stages are a launch
// of their own.  Against 34 thousand launches of 2480 sets (1024 to 6208 columns, K 2048 to 14336, 2 to 16 modules of 1 to 16 rows, groups of
// 64, 128 and a row) it is 2 % slow near the best shape, 8 % rms; the pick is 1.8 % behind the best of fourteen shapes on the mean, more than
// 10 % behind in 5 % of the sets, 31 % at most.  Of 466 drawn sets 9 are more than 10 % slower than with plans of their own (39 % at most), and
// they take 0.87 of that time on the mean.
struct ModuleSetPlan { int wn, wk; double us; };                // wn 0: no shape
struct ModuleSetPlans { ModuleSetPlan chunks[2]; int own; };   // the fastest with one and with two chunks in flight; 1, 2: the modules' own is one
constexpr int kModuleSet = 16, kSetRows = 16;                  // modules of a set at most (those of a launch), rows of one
constexpr int kSetWavesN[] = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16}, kSetWavesK[] = {1, 2, 3, 4, 5, 7, 8};
constexpr double kSetStart = 2.9;                              // us of a launch
constexpr int64_t kSetStage = (int64_t)150 << 10;              // a larger slice goes through its workgroup in stages or fills its LDS
// Chunks that the wavefronts of a workgroup along K take in all; 0 for a shape that leaves more than a quarter of them idle (none of these
// was the fastest by more than 0.1 % on the mean).
static int64_t set_chunks(int64_t KC, int wk) {
    const int64_t all = (KC + wk - 1) / wk * wk;
    return wk <= KC && 3 * all <= 4 * KC ? all : 0;
}
// rows[m]: modules of m rows.  own: the plan that they would all have by themselves, or null: kept where the best is not 6 % ahead.  A shape
// has to run the module of the most rows; those of fewer rows run wherever it does.
static ModuleSetPlans module_set_plans(const LinearArgs& like, const int* rows, const LinearPlan* own, size_t lds_limit) {
    const int64_t NT = like.N / 16, KC = like.K / chunk_k(like.bits);
    const double stream = like.bits == 8 ? 9.2e6 : 7.23e6;
    LinearArgs a = like;
    int most = kSetRows;
    while (most > 1 && rows[most] == 0) --most;
    LinearPlan p = {};
    p.path = 1; p.split_k = p.m_rows16 = p.m_blocks = p.n_tiles16 = 1;
    ModuleSetPlans out = {};
    ModuleSetPlan kept = {};
    for (int wk : kSetWavesK) {
        const int64_t chunks = set_chunks(KC, wk);
        if (chunks == 0) continue;
        p.waves_k = wk;
        double fixed[17] = {}, requests[17] = {};            // us by wn; requests: by the chunks in flight
        for (int nb = 1; nb <= (chunks > wk ? 2 : 1); ++nb) {
            p.prefetch = nb; p.waves_n = 1;
            a.M = 1;
            const size_t row = rtn::linear_stages(a, p).slice;
            const bool stages = row * most > (size_t)kSetStage;      // (they depend on the chunks in flight)
            // modules whose slice is staged at once, and those that take it in stages: a launch each
            int count[2] = {};
            size_t staged[2] = {}, lds[2] = {};
            for (int m = 1; m <= most && (nb == 1 || stages); ++m) {
                if (rows[m] == 0) continue;
                rtn::StagePlan s = {0, 1, row * m, row * m};
                a.M = m;
                if (s.slice > (size_t)kSetStage) s = rtn::linear_stages(a, p);
                const int kind = s.nstage > 1;
                count[kind] += rows[m];
                staged[kind] += s.slice * rows[m];
                lds[kind] = std::max(lds[kind], s.lds);
            }
            a.M = most;
            for (int wn : kSetWavesN) {
                if (wn > NT || wn * wk < 4 || wn * wk > 16) continue;
                p.waves_n = wn;
                if (nb == 1 || stages) fixed[wn] = requests[wn] = 0.0;
                for (int kind = 0; kind < 2 && (nb == 1 || stages); ++kind) {
                    if (count[kind] == 0) continue;
                    const int64_t workgroups = count[kind] * ((NT + wn - 1) / wn);
                    const int64_t by_lds = (int64_t)(rtn::kMaxLdsBytes / std::max(lds[kind], (size_t)(wk - 1) * wn * 1024));
                    const int64_t resident = std::max<int64_t>(1, std::min<int64_t>(32 / (wn * wk), by_lds));
                    const double n = (double)workgroups, bytes = (double)count[kind] * NT * KC * 4096.0;
                    const double fullest = std::max(1.0, (double)((workgroups + 255) / 256 * 256 * wn * KC) * 4096.0 / bytes);
                    fixed[wn] += kSetStart + 0.774 * (double)((workgroups + 256 * resident - 1) / (256 * resident) - 1) + bytes / stream * std::pow(fullest, 0.703) +
                                (double)staged[kind] * (n / count[kind]) / 11.4e6 + 0.152e-3 * n * wn * wk;
                    requests[wn] += bytes * 0.33 / (std::min(n / 256.0, (double)resident) * wn * wk * 4096.0 * 256.0);
                }
                const double shape = 1.0 + 0.033 * (std::log2((double)wn) - 1.5) + 0.034 * (std::log2((double)wk) - 1.0) + 0.057 * (nb - 1.5);
                const double us = (fixed[wn] + requests[wn] / nb) * shape;
                if (own && own->waves_n == wn && own->waves_k == wk && own->prefetch == nb) kept = {wn, wk, us};
                ModuleSetPlan& best = out.chunks[nb - 1];
                if ((best.wn == 0 || us < best.us) && rtn::linear_plan_fits(a, p, lds_limit)) best = {wn, wk, us};
            }
        }
    }
    for (const ModuleSetPlan& best : out.chunks)
        if (best.wn > 0 && best.us <= 0.94 * kept.us) return out;
    if (kept.wn > 0) {
        out.chunks[own->prefetch - 1] = kept;
        out.own = own->prefetch;
    }
    return out;
}

// The rows that a set is planned for.  In a mixture-of-experts model they change with every call, so a plan is made, and remembered, for what
// its time depends on.  Up to `sure` rows a slice is staged at once whatever the shape: these modules stand for one of the most rows and the
// others of the mean, or, beside larger ones, of half as many.  From `never` rows on it goes in stages in every shape: these count as their
// largest.  In between every row counts.  40 thousand lists drawn for eight modules of 1 to 16 rows are planned as 86 with 2048 or
// 4096 columns, 1145 with 6144 and 367 with 7168; the model puts the pick 0.01 % behind that for the rows themselves on the mean of 6000 drawn sets, 3.8 % at most.
static void module_set_rows(const LinearArgs* args, const int* member, int count, int* rows) {
    const LinearArgs& like = args[member[0]];
    const int64_t chunk = chunk_k(like.bits), KC = like.K / chunk;
    int64_t padded = KC;
    for (int wk : kSetWavesK) padded = std::max(padded, set_chunks(KC, wk));
    auto slice = [&](int64_t m, int64_t chunks) { return m * (chunks * chunk + 8) * 2; };
    int sure = 0, never = kSetRows + 1;
    while (sure < kSetRows && slice(sure + 1, padded) <= kSetStage) ++sure;
    while (never > 1 && slice(never - 1, KC) > (int64_t)rtn::kMaxLdsBytes) --never;
    int few = 0, most_few = 0, sum = 0, many = 0, most = 0;
    for (int k = 0; k < count; ++k) {
        const int m = (int)args[member[k]].M;
        if (m <= sure) {
            ++few;
            most_few = std::max(most_few, m);
            sum += m;
        } else if (m < never) {
            ++rows[m];
        } else {
            ++many;
            most = std::max(most, m);
        }
    }
    if (many > 0) rows[most] += many;
    if (few == 0) return;
    const bool all = few == count;
    const int top = all ? most_few : sure, others = all ? (sum - top + (count - 1) / 2) / (count - 1) : (sure + 1) / 2;
    ++rows[top];
    rows[std::max(1, others)] += few - 1;
}

// A module's set (-1: in none) and its part of the set's modelled time.
struct SetShare { int set; double us; };
static rtn_status grouped_plans(const LinearArgs* args, int n, size_t workspace_nbytes, LinearPlan* plans, SetShare* share) {
    const size_t lds_limit = (size_t)device_max_lds();
    int64_t steps_total = 0;                                   // of the modules the skinny kernel will serve
    for (int i = 0; i < n; ++i)
        if (args[i].M <= 16) steps_total += (args[i].N / 16) * (args[i].K / chunk_k(args[i].bits));
    for (int i = 0; i < n; ++i) {
        const LinearArgs& a = args[i];
        rtn_status st = RTN_ERR_CONFIG;
        if (!small_groups(a.M, a.g)) {
            // planned as one slice of a launch that streams all the small-batch modules together
            const LinearPlan h = auto_plan(a.M, a.N, a.K, a.bits, a.g, lds_limit, 0, a.M <= 16 ? steps_total : 0,
                                           tile_workspace(a, workspace_nbytes));
            const rtn_linear_cfg cfg = plan_cfg(h);
            st = resolve_plan(a, &cfg, workspace_nbytes, &plans[i]);
        }
        if (st == RTN_ERR_CONFIG) st = resolve_plan(a, nullptr, workspace_nbytes, &plans[i]);    // the module's own plan
        if (st != RTN_OK) return st;
        share[i] = {-1, 0.0};
    }
    // Sets of alike modules (the errors of a call are those of the plans above)
    struct Set { int first, count; ModuleSetPlans plans; };
    std::vector<Set> sets;
    std::vector<char> tried((size_t)n, 0);                     // in a set, whether or not a shape was found for it
    auto candidate = [&](int i) { return !tried[i] && args[i].M <= 16 && plans[i].path == 1; };
    for (int i = 0; i < n; ++i) {
        if (!candidate(i)) continue;
        int member[kModuleSet], count = 0, rows[kSetRows + 1] = {};
        for (int j = i; j < n && count < kModuleSet; ++j)
            if (candidate(j) && args[j].N == args[i].N && args[j].K == args[i].K && args[j].bits == args[i].bits && args[j].g == args[i].g)
                member[count++] = j;
        for (int k = 0; k < count; ++k) tried[member[k]] = 1;
        // (two modules whose own plans split K go to the block kernel together, as they have: 13.7 us, 12.4 as a set here)
        if (count < 2 || (count == 2 && plans[member[0]].split_k + plans[member[1]].split_k > 2)) continue;
        int64_t key[2] = {};
        const LinearPlan& first = plans[i];
        bool one_shape = first.prefetch <= 2;
        for (int k = 0; k < count; ++k) {
            const LinearPlan& p = plans[member[k]];
            one_shape = one_shape && p.split_k == 1 && p.waves_n == first.waves_n && p.waves_k == first.waves_k && p.prefetch == first.prefetch;
        }
        module_set_rows(args, member, count, rows);
        for (int m = 0; m < kSetRows; ++m) key[m / 12] |= (int64_t)rows[m + 1] << (5 * (m % 12));
        static Remembered<ModuleSetPlans, 4096> remembered;
        const int own = one_shape ? 1 + first.waves_n * 64 + first.waves_k * 4 + first.prefetch : 0;
        const ModuleSetPlans set = remembered.get({key[0], args[i].N, args[i].K, args[i].g, (size_t)key[1], lds_limit, args[i].bits, own},
                                                  [&] { return module_set_plans(args[i], rows, one_shape ? &first : nullptr, lds_limit); });
        if (set.chunks[0].wn == 0 && set.chunks[1].wn == 0) continue;
        for (int k = 0; k < count; ++k) share[member[k]].set = i;
        sets.push_back({i, count, set});
    }
    // Chunks in flight: the same for all that can share a launch (grouped_launches).  5 and 14 rows of 5680 x 4096 beside 8 of 1168 x 4096: 17.2 us
    // as two launches, 11.5 as one; 449 calls of two kinds of modules take 0.96 of the time with plans of their own on the mean, and 15 of them
    // more than 1.1 (64 with each set's fastest shape).
    auto one_launch = [&](int i, int j) {
        const int64_t chunk = chunk_k(args[i].bits);
        return args[i].bits == args[j].bits && std::min(args[i].g, chunk) == std::min(args[j].g, chunk);
    };
    for (const Set& s : sets) {
        double us[2] = {};
        bool others[2] = {};                                   // modules of no set, by their chunks in flight
        int alike = 0;
        for (const Set& t : sets)
            if (one_launch(s.first, t.first)) {
                ++alike;
                for (int c = 0; c < 2; ++c) us[c] += t.plans.chunks[c].wn > 0 ? t.plans.chunks[c].us : 1e6;
            }
        for (int j = 0; j < n; ++j)
            if (share[j].set < 0 && plans[j].path == 1 && plans[j].split_k == 1 && plans[j].prefetch <= 2 && one_launch(s.first, j))
                others[plans[j].prefetch - 1] = true;
        for (int c = 0; c < 2; ++c)
            if (others[1 - c] && !others[c]) us[c] += kSetStart;
        const int c = alike == 1 && !others[0] && !others[1] && s.plans.own ? s.plans.own - 1 : us[1] < us[0] ? 1 : 0;
        const ModuleSetPlan& set = s.plans.chunks[c].wn > 0 ? s.plans.chunks[c] : s.plans.chunks[1 - c];
        for (int j = s.first; j < n; ++j) {
            if (share[j].set != s.first) continue;
            LinearPlan& p = plans[j];
            p.prefetch = s.plans.chunks[c].wn > 0 ? 1 + c : 2 - c; p.waves_n = set.wn; p.waves_k = set.wk;
            p.split_k = p.m_rows16 = p.m_blocks = p.n_tiles16 = 1;
            share[j].us = set.us / s.count;
        }
    }
    return RTN_OK;
}

// Modelled time of a module's share of a grouped launch of the small-batch kernel: its bytes and a part of the start.  A workgroup
// stages all its rows' columns: from 100 KiB one fits a compute unit, from 150 it goes through them in stages.  Medians of 66
// measured launches of two to eight modules, 1024 to 8192 columns of 2048 to 7168, 1 to 16 rows.
static double grouped_share_us(const LinearArgs& a, int n) {
    const double bytes = (double)a.N * a.K * a.bits / 8.0 + (double)a.N * (a.K / a.g) * 2.0 + 2.0 * a.M * (a.K + a.N);
    const int64_t slice = a.M * a.K * 2;
    return (3.0 / n + bytes / (a.bits == 8 ? 6.4e6 : 5.8e6)) * (slice < 50 << 10 ? 1.0 : slice < 100 << 10 ? 1.08 : slice < 150 << 10 ? 1.30 : 2.2);
}

// A set of a grouped call's modules on the block kernel.  In a mixture-of-experts model their rows change with every call, so a plan is
// made, and remembered, for classes of rows, up to 8 or 16 and then by 32, in an order of its own: all lists of up to 16 rows of like modules
// share two plans (all the plans of a call of eight experts with rows drawn anew take 1.2 us of host time, 25 with a plan here for each list).
// With more than 16 rows in the set its time is that of the rows themselves.
static void plan_set(const LinearArgs* args, SharedLaunch* l, size_t workspace) {
    int64_t most = 0;
    for (int k = 0; k < l->count; ++k) most = std::max(most, args[l->member[k]].M);
    auto row_class = [&](int j) { return args[j].M > 16 ? (args[j].M + 31) / 32 * 32 : most <= 8 ? (int64_t)8 : (int64_t)16; };
    auto before = [&](int x, int y) {
        const LinearArgs &a = args[x], &b = args[y];
        if (a.N != b.N) return a.N > b.N;
        if (a.K != b.K) return a.K > b.K;
        if (a.g != b.g) return a.g > b.g;
        return row_class(x) > row_class(y);
    };
    int order[rtn::kMaxBlockGroup];
    for (int k = 0; k < l->count; ++k) {
        int at = k;
        for (; at > 0 && before(l->member[k], l->member[order[at - 1]]); --at) order[at] = order[at - 1];
        order[at] = k;
    }
    LinearArgs set[rtn::kMaxBlockGroup];
    for (int k = 0; k < l->count; ++k) {
        set[k] = args[l->member[order[k]]];
        set[k].M = row_class(l->member[order[k]]);
    }
    const MergedPlan p = remembered_merge(set, l->count, workspace);
    l->plan = p;
    if (p.us < 0.0) return;
    for (int k = 0; k < l->count; ++k) {
        l->plan.waves[order[k]] = p.waves[k];
        l->plan.split[order[k]] = p.split[k];
        set[k].M = args[l->member[order[k]]].M;
    }
    int longest;
    if (most > 16) l->plan.us = merged_blocks_us(set, l->count, p, args[0].workspace ? workspace : 0, &longest);
}

// A grouped call's modules of up to 512 rows: together on the block kernel where that is modelled ahead of the launches that go out
// otherwise.  Modules with a launch of their own (kOpen) make up the sets, in order; the small ones, which the small-batch kernel's
// grouped launches serve, fill the places left where that is modelled level (200, 100 and six times 1 to 6 rows of 4096 x 4096: 0.98,
// measured 30.0 and 34.2 us), and then make sets of their own, those of one shape (module_set_plans) as a whole or not at all, with modules
// of other shapes or by themselves.  Measured against the small-batch kernel, int4 group 128: eight of 2048 x 7168 at 9 to 16 rows 27.7 us and
// 17.4, int8 35.1 and 23.4, 5280 x 6144 39.4 and 32.0; 1024 x 4096 stay there (8.1, 8.4 here), as do few rows (2048 x 7168 at 1 to 8
// 14.9, 15.5 here).  Of 3218 drawn sets the choice is 0.7 % behind the better kernel on the mean, more than 5 % in 155.  The modules alone
// in their launch go on to the small-batch kernel's grouped launches.
static int grouped_blocks(const LinearArgs* args, const LinearPlan* plans, int n, size_t workspace_nbytes, const SetShare* share,
                          SharedLaunch* out) {
    std::vector<double> own_us((size_t)n, 0.0);
    std::vector<char> state((size_t)n, kAlone);
    std::vector<int64_t> most((size_t)n, 0);                   // rows of a module, or of the largest in its set
    std::vector<int> open((size_t)n, 0), decided((size_t)n, -1);   // small modules of a set (or the module itself) still open; see gather_whole
    int small = 0;
    double bytes = 0.0;
    auto grouped = [&](int i) { return plans[i].path == 1 && plans[i].split_k == 1 && plans[i].m_blocks == 1; };
    auto lead = [&](int i) { return share[i].set < 0 ? i : share[i].set; };    // a set goes by its first module
    for (int i = 0; i < n; ++i) {
        if (grouped(i)) { ++small; bytes += (double)args[i].N * args[i].K * args[i].bits / 8.0; }
        most[lead(i)] = std::max(most[lead(i)], args[i].M);
    }
    for (int i = 0; i < n; ++i) {
        if (args[i].M > kMaxMergedRows || (args[i].M <= 4 && !grouped(i))) continue;
        if (grouped(i) && bytes < 24e6 && most[lead(i)] * args[i].K * 2 < 100 << 10) continue;  // none of these was ahead
        state[i] = grouped(i) ? kSmall : kOpen;
        if (grouped(i)) ++open[lead(i)];
        own_us[i] = share[i].set >= 0 ? share[i].us : grouped(i) ? grouped_share_us(args[i], std::min(small, 16)) : own_plan_us(args[i], plans[i], workspace_nbytes);
    }
    int launches = 0;
    // up to eight modules of i's class from i on that are in `wanted`, after those in l; their time apart
    auto gather = [&](SharedLaunch* l, int i, int from, char wanted) {
        double apart = 0.0;
        for (int j = from; j < n && l->count < rtn::kMaxBlockGroup; ++j) {
            if (state[j] != wanted || !one_block_class(args[i], args[j])) continue;
            apart += own_us[j];
            l->member[l->count++] = j;
        }
        return apart;
    };
    // the small modules of i's class from i on, a set's whole or not at all
    auto gather_whole = [&](SharedLaunch* l, int i) {
        double apart = 0.0;
        l->count = 0;
        for (int j = i, places = rtn::kMaxBlockGroup; j < n; ++j) {
            if (state[j] != kSmall || !one_block_class(args[i], args[j])) continue;
            int& v = decided[lead(j)];
            if (v / 2 != i || v < 0) {                         // the first of its set here
                v = 2 * i + (open[lead(j)] <= places ? 1 : 0);
                if (v & 1) places -= open[lead(j)];
            }
            if (!(v & 1)) continue;
            apart += own_us[j];
            l->member[l->count++] = j;
        }
        return apart;
    };
    auto ahead = [&](SharedLaunch* l, double apart, bool more_of_a_launch) {
        if (l->count < 2) return false;
        plan_set(args, l, workspace_nbytes);
        int64_t rows = 0;
        for (int k = 0; k < l->count; ++k) rows = std::max(rows, args[l->member[k]].M);
        const double line = more_of_a_launch ? 1.0 : together_line(l->count, rows, false);
        return l->plan.us >= 0.0 && l->plan.us <= line * apart;
    };
    auto take = [&](const SharedLaunch& l) {
        for (int k = 0; k < l.count; ++k) {
            if (state[l.member[k]] == kSmall) --open[lead(l.member[k])];
            state[l.member[k]] = kDone;
        }
        out[launches++] = l;
    };
    for (char kind : {kOpen, kSmall})
        for (int i = 0; i < n; ++i) {
            if (state[i] != kind) continue;
            SharedLaunch set, filled;
            if (kind == kSmall) {
                if (open[lead(i)] < rtn::kMaxBlockGroup) {
                    const double apart = gather_whole(&set, i);
                    if (set.count > open[lead(i)] && ahead(&set, apart, false)) {
                        take(set);
                        continue;
                    }
                    for (int k = 0; k < set.count; ++k)
                        if (share[set.member[k]].set < 0) state[set.member[k]] = kAlone;
                    if (state[i] == kAlone) continue;
                }
                if (share[i].set < 0) {
                    state[i] = kAlone;
                    continue;
                }
                // a set with a plan of its own: what larger modules left of it here, in launches of like size, or none (14 of 1056 x 7168, up
                // to 12 rows: 23 us on the small-batch kernel, 25 as two launches here, 36 as one of eight and the others there)
                int member[kModuleSet], count = 0;
                for (int j = i; j < n; ++j)
                    if (state[j] == kSmall && share[j].set == share[i].set) member[count++] = j;
                const int parts = (count + rtn::kMaxBlockGroup - 1) / rtn::kMaxBlockGroup;
                SharedLaunch part[kModuleSet / rtn::kMaxBlockGroup];
                bool all = count >= 2;
                double together = 0.0, line = 1.0;
                for (int k = 0, at = 0; k < parts && all; ++k) {
                    part[k].count = (count - at) / (parts - k);
                    std::copy(member + at, member + at + part[k].count, part[k].member);
                    at += part[k].count;
                    plan_set(args, &part[k], workspace_nbytes);
                    all = part[k].plan.us >= 0.0;
                    together += part[k].plan.us;
                    line = std::min(line, together_line(part[k].count, 16, false));
                }
                all = all && together <= line * share[i].us * count;
                for (int k = 0; k < parts && all; ++k) take(part[k]);
                for (int k = 0; k < count && !all; ++k) state[member[k]] = kAlone;
                continue;
            }
            set.count = 0;
            double apart = gather(&set, i, i, kOpen);
            const bool together = ahead(&set, apart, false);
            if (together) apart = set.plan.us;
            filled = set;
            apart += gather(&filled, i, 0, kSmall);
            for (int k = set.count; k < filled.count; ++k) {   // what is left of a set pays its launch's start all the same
                const int first = lead(filled.member[k]);
                int taken = 0;
                for (int x = set.count; x < filled.count; ++x) taken += lead(filled.member[x]) == first;
                if (taken < open[first]) apart -= kSetStart / open[first];
            }
            if (filled.count > set.count && ahead(&filled, apart, true)) {
                take(filled);
                continue;
            }
            if (!together) {
                set.count = 1;
                set.member[0] = i;
            }
            take(set);
        }
    for (int i = 0; i < n; ++i)
        if (state[i] == kAlone) {
            out[launches].count = 1;
            out[launches++].member[0] = i;
        }
    return launches;
}

// What a grouped call issues: launches of the block kernel, then the modules that are left, with their plans, which the small-batch
// kernel's grouped launches serve or which go out by themselves.
struct GroupedCall {
    std::vector<SharedLaunch> blocks;
    std::vector<int> left;
    std::vector<LinearPlan> plans;
};
static rtn_status plan_grouped_call(const LinearArgs* args, int n, size_t workspace_nbytes, GroupedCall* call) {
    std::vector<SetShare> share((size_t)n);
    std::vector<LinearPlan> plans((size_t)n);
    const rtn_status st = grouped_plans(args, n, workspace_nbytes, plans.data(), share.data());
    if (st != RTN_OK) return st;
    call->blocks.resize((size_t)n);
    const int launches = grouped_blocks(args, plans.data(), n, workspace_nbytes, share.data(), call->blocks.data());
    std::vector<char> gone((size_t)n, 0);
    int kept = 0;
    for (int i = 0; i < launches; ++i) {
        const SharedLaunch l = call->blocks[i];
        if (l.count == 1) continue;
        for (int k = 0; k < l.count; ++k) gone[l.member[k]] = 1;
        call->blocks[kept++] = l;
    }
    call->blocks.resize((size_t)kept);
    call->left.reserve((size_t)n);
    for (int i = 0; i < n; ++i) {
        if (gone[i]) continue;
        plans[call->left.size()] = plans[i];                   // (in order)
        call->left.push_back(i);
    }
    call->plans.swap(plans);
    return RTN_OK;
}

rtn_status rtn_grouped_forward(const rtn_module* mods, int n_mods, void* dev_workspace, size_t workspace_nbytes,
                               void* stream) {
    if (!mods) return RTN_ERR_NULL;
    if (n_mods <= 0) return RTN_ERR_SHAPE;
    if (!aligned16(dev_workspace)) return RTN_ERR_ALIGN;
    std::vector<LinearArgs> args((size_t)n_mods);
    for (int i = 0; i < n_mods; ++i) {
        const rtn_status st = module_args(mods[i], dev_workspace, &args[i]);
        if (st != RTN_OK) return st;
    }
    GroupedCall call;
    const rtn_status st = plan_grouped_call(args.data(), n_mods, workspace_nbytes, &call);
    if (st != RTN_OK) return st;
    for (const SharedLaunch& l : call.blocks)
        if (launch_shared(args.data(), l, false, stream) != hipSuccess) return RTN_ERR_HIP;
    const int n = (int)call.left.size();
    for (int k = 0; k < n; ++k) args[k] = args[call.left[k]];  // (in order)
    const hipError_t e = n == 0 ? hipSuccess : rtn::launch_linear_grouped(args.data(), call.plans.data(), n, false, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? RTN_OK : RTN_ERR_HIP;
}

static int layer_selected(int layer, int n_layers, int policy, int X) {
    int start;
    switch (policy) {
        case RTN_POLICY_FIRST: start = 0; break;
        case RTN_POLICY_LAST: start = n_layers - X; break;
        case RTN_POLICY_MIDDLE: start = (n_layers - X) / 2; break;
        default: return -1;
    }
    return (layer >= start && layer < start + X) ? 1 : 0;
}

int rtn_plan_bits(int layer, int n_layers, int module_id, int policy, int X, unsigned module_mask) {
    if (n_layers <= 0 || layer < 0 || layer >= n_layers || X < 0 || X > n_layers) return -1;
    if (module_id < 1 || module_id > 4 || module_mask > 15u) return -1;
    const int sel = layer_selected(layer, n_layers, policy, X);
    if (sel < 0) return -1;
    return (sel && (module_mask >> (module_id - 1) & 1u)) ? 8 : 4;
}

double rtn_plan_effective_bits(int n_layers, const int64_t module_params[4], int policy, int X,
                               unsigned module_mask) {
    if (!module_params || n_layers <= 0) return -1.0;
    long double total = 0, bits = 0;
    for (int l = 0; l < n_layers; ++l)
        for (int m = 1; m <= 4; ++m) {
            const int b = rtn_plan_bits(l, n_layers, m, policy, X, module_mask);
            if (b < 0 || module_params[m - 1] < 0) return -1.0;
            total += (long double)module_params[m - 1];
            bits += (long double)module_params[m - 1] * b;
        }
    return total > 0 ? (double)(bits / total) : -1.0;
}

}  // extern "C"
