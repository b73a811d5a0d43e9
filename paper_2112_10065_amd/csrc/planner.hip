// Kernel choice for one pass of one layer: enumerate the tile variants and reduction splits that
// the shape allows, price each with a small analytic model calibrated on MI355X measurements,
// take the cheapest.  Host code only.  The model:
//
//   blocks       = tiles * splits               concurrent = 256 CUs * blocks_per_CU(variant)
//   t_block      = t0(variant) + steps_per_split * t_step(variant) * share
//                  (share < 1 when fewer blocks than the variant could co-run share a CU)
//   t            = launch + waves(blocks / concurrent) * t_block + t_reduce(splits)
//   t_reduce     = second kernel that sums the fp32 partials: launch + (splits + 1) * out bytes / BW
#include "dp_kernels.h"
#include <algorithm>
#include <cmath>

namespace {

struct Candidate {
    int code;        // override code understood by fast_plan / dma_plan (100.., 200.., 300..)
    int bpc;         // blocks that fit on one CU (LDS / registers)
    float t_step;    // microseconds per reduction step and block on a fully shared CU
    float t0;        // microseconds of prologue + epilogue per block
    int kg = 1;      // reduction groups inside a block: each group walks 1/kg of the block's steps
};

// forward / backward-data candidates
const Candidate kPix[] = {
    {230, 1, 1.30f, 9.0f},   // 256x256x64, 4 waves, 3x3 stride 1 with the pixel strip shared by the three taps of a filter row
    {231, 1, 0.70f, 7.0f},   // the same with 128 pixel rows per tile and three weight stages
    {232, 1, 0.70f, 7.0f},   // the same with 128 output channels per tile (layers with 128 of them)
    {233, 1, 1.15f, 9.0f},   // the same with 224 pixel rows per tile (four waves side by side over the channels)
    {208, 1, 1.55f, 8.0f},   // 256x256x64, 8 waves, direct-to-LDS
    {200, 2, 1.08f, 5.0f},   // 128x128x64 direct-to-LDS
    {204, 3, 0.85f, 4.5f},   // 64x128x64
    {206, 3, 0.85f, 4.5f},   // 128x64x64
    {207, 3, 0.62f, 4.0f},   // 64x64x64
    {201, 4, 1.08f, 4.5f},   // direct-to-LDS with reduction step 32 (channels % 32 only)
    {205, 4, 0.85f, 4.0f},
    {213, 3, 1.30f, 4.5f},
    {210, 1, 1.15f, 6.0f},   // 128x256x64, 8 waves
    {212, 2, 1.30f, 4.5f},   // 64x256x64
    {221, 1, 0.70f, 4.0f},   // reduction step 128 (channels % 128 only): fewer, longer steps for small grids
    {225, 1, 0.70f, 4.0f},
    {222, 1, 1.10f, 4.5f},
    {224, 1, 1.10f, 4.5f},
    {223, 1, 1.90f, 5.0f},
    {226, 1, 0.62f, 5.0f, 4},   // 64x64x64 with 4 / 2 reduction groups per block (no partials in memory)
    {227, 2, 0.62f, 4.5f, 2},
    {228, 1, 0.85f, 5.0f, 2},
    {229, 1, 0.85f, 5.0f, 2},
    {400, 2, 0.75f, 5.5f},   // input patch resident in LDS: 64 x 256 tile (64 reduction channels per tap, stride 1)
    {401, 2, 1.20f, 6.0f},   // same, 128 x 256
    {402, 2, 0.75f, 5.5f},
    {403, 2, 0.72f, 5.5f},
    {404, 2, 0.40f, 0.8f},   // 3x3 only: persistent blocks, weights in registers (180 layers: 8 % in the median)
    {405, 1, 3.66f, 7.9f},   // the same for 128 reduction channels, by rounds of tiles: 4.4 us and 4.1 a round (240 timings, 3 - 8 %) in the currency of the tiles above
    {100, 2, 1.40f, 5.0f},   // register-staged fallbacks (also reduction step 32)
    {101, 3, 1.05f, 4.5f},
    {102, 3, 1.05f, 4.5f},
    {103, 4, 0.75f, 4.0f},
};
// Forward by the flat walk (64x64, with 4 and 2 reduction groups, 64x128, 128x64, 128x128; steps of 64): step and block times fitted to 376
// layers (8 to 448 channels, images 6 to 150, 1 to 32 samples; median error 7 %)
const Candidate kFlatFwd[] = {
    {234, 3, 0.55f, 1.5f}, {235, 1, 0.75f, 2.5f, 4}, {236, 2, 0.70f, 1.5f, 2}, {237, 3, 0.70f, 1.5f}, {238, 3, 0.65f, 1.5f}, {239, 2, 0.75f, 2.5f},
};
// The same for backward-data, 385 layers (median error 5 - 10 %).  A reduction split costs 1.5 us more than price() says.
const Candidate kFlatBwd[] = {
    {234, 3, 0.75f, 3.0f}, {235, 1, 1.00f, 4.0f, 4}, {236, 2, 0.90f, 3.0f, 2}, {237, 3, 0.95f, 3.5f}, {238, 3, 0.95f, 3.5f}, {239, 2, 1.00f, 5.0f},
};
// backward-filter candidates (reduction step 32 unless noted)
const Candidate kWg[] = {
    {300, 4, 1.00f, 4.0f},   // 128x128x32 direct-to-LDS
    {303, 4, 0.70f, 3.5f},   // 64x128x32
    {304, 4, 0.70f, 3.5f},   // 128x64x32
    {305, 5, 0.62f, 3.5f},   // 64x64x32
    {308, 3, 1.45f, 4.0f},   // 64x256x32 (few output channels: widest tap tile)
    {306, 3, 0.93f, 4.0f},   // 64x128x64
    {301, 2, 1.75f, 4.5f},   // 128x128x64
    {307, 2, 1.60f, 5.0f},   // 256x128x32, 8 waves
    {314, 2, 1.65f, 5.0f},   // 128x256x32, 8 waves
    {312, 1, 2.90f, 7.0f},   // 256x256x64, 8 waves
    {316, 1, 1.60f, 9.0f},   // 3x3 stride 1: 256 x (3 taps x 64 channels), x strip shared by the taps, padded pixel slots
    {410, 1, 0.13f, 6.0f},   // input patch in LDS, persistent blocks (64 input channels, stride 1); a step = 16 pixels
    // the same for 3x3 filters with all nine taps in one wave.  With 6.0 it was the cheapest more often, and the window kernel then took its place by 1.35 of its price;
    // at 8.0 split tiles are, and stay (147 of 24000 layers: 0.82 - 1.08 of the window kernel's time, 0.91 in the middle, with flushed caches 0.94)
    {411, 1, 0.10f, 8.0f},
    {100, 3, 1.30f, 4.0f},
    {101, 3, 1.00f, 3.5f},
    {102, 3, 1.00f, 3.5f},
    {103, 4, 0.80f, 3.0f},
};
const int kSplits[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32, 48, 64, 96, 128, 192, 256};

bool family_plan(const ConvGeom &g, int pass, int code, int splits, GemmPlan *pl, int restr = 0)
{
    pl->halo = false;
    pl->wstrip = false;
    pl->wwin = false;
    pl->win = false;
    pl->pw = false;
    if (code >= 400) return halo_plan(g, pass, code, splits, pl);
    if (code >= 200) return dma_plan(g, pass, code, splits, pl, (restr & 1) != 0);
    return fast_plan(g, pass, code, splits, pl);
}

// Window kernel of the filter gradient: fitted to 1140 timings of 3x3 layers (chunks of 256 and of 128 slots; median error 3 %, 8 % for nine
// of ten) and 290 of other filters (6 %, 16 %).  A chunk costs more when all CUs run one: the matrix cores then hold the clock down.
double price_window(const ConvGeom &g, const GemmPlan &pl)
{
    const double blocks = (double)pl.tilesA * pl.tilesB * pl.splits, rounds = std::ceil(blocks / 256.0);
    const double busy = std::min(1.0, std::max(0.0, blocks / 128.0 - 1.0)), out_mb = (double)g.K * g.R * g.S * g.C * 4e-6;
    const double step = !pl.row_taps ? 0.70 : pl.BK == 256 ? 1.52 + 0.21 * busy : 0.86 + 0.09 * busy, t0 = !pl.row_taps ? 7.5 : 3.8;
    return 3.0 + rounds * (t0 + pl.steps_per_split * step) + (pl.splits > 1 ? 3.0 + 0.45 * (pl.splits + 1) * out_mb : 0.45 * out_mb);
}

double price(const ConvGeom &g, int pass, const Candidate &c, const GemmPlan &pl, int restr)
{
    const double blocks = (double)pl.tilesA * pl.tilesB * pl.splits;
    if (c.code == 405) return c.t0 + c.t_step * std::ceil(blocks / 256.0);
    const double conc = 256.0 * c.bpc;
    double share = 1.0, waves;
    if (blocks <= conc) {
        const double r = std::ceil(blocks / 256.0);
        share = 0.45 + 0.55 * r / c.bpc;
        waves = 1.0;
    } else {
        const double w = blocks / conc;
        waves = w >= 4.0 ? w : 0.5 * (w + std::ceil(w));
        // A persistent block's tiles come one after another: 10.2 us for 1.03 tiles per block as for 2, 14 for 2.02 as for 3.  Up to three rounds; beyond, where its price
        // also stands against the 128-wide input-patch tiles (theirs is too low: they take 1.2 - 1.9 times as long), the mean of both as for the others
        if (c.code == 404 && w < 3.0) waves = std::ceil((double)pl.tilesB / std::max(512 / pl.tilesA, 1));
    }
    // a step of reduction length 32 costs about half of a 64 step for the pixel passes
    double t_step = c.t_step;
    if (pass != PASS_WGRAD && pl.BK == 32) t_step *= 0.6;
    // 64x256 tiles in backward-data, short reductions and more than one round: prologue and epilogue weigh more (45 drawn layers against the
    // tiles that replace them: 0.95 - 3.7, 1.25 in the mean).  Not forward: its sums keep their order (forward_flat_plan)
    const bool wide = c.code == 212 && pass == PASS_DGRAD && !(restr & RESTR_BASE) && (g.R * g.S == 1 || blocks > conc);
    const double t_block = (wide ? 8.0 : c.t0) + (pl.steps_per_split + c.kg - 1) / c.kg * t_step * share;
    double t = 3.0 + waves * t_block;
    // The saved input of a masked backward-data tile, read while nothing else runs on the CU and the next tile waits (the strip kernels
    // fetch it ahead, a single round of blocks has no next tile): 3.5 us for the 128 KB of a 256x256 tile at a CU's share of the memory
    // rate.  It decides only by 5 % (10 % for fp32 gradients): nearer, the tiles that replace these are as often slower (64 x 56 x 56 x 256 <- 128,
    // 1x1: 59 us, 52; 60 drawn layers 0.97 - 1.4, 1.13 in the mean).  Not where the input-patch kernels would win by it: they read
    // the mask no better (24 x 65 x 65 x 256 <- 64: 31 us, 46)
    const bool lone_mask = pass == PASS_DGRAD && (restr & 2) && !(restr & RESTR_BASE) && c.bpc == 1 && pl.splits == 1 && blocks > 256.0 &&
                           c.code >= 200 && c.code < 230 && (g.K != 64 || g.sh > 1 || g.sw > 1);
    if (lone_mask) t = std::max(t, ((restr & 1) ? 0.90 : 0.95) * (3.0 + waves * (t_block + 3.5 * pl.TA * pl.TB / 65536.0)));
    if (pl.splits > 1) {
        double out_elems = pass == PASS_FWD ? (double)g.N * g.Ho * g.Wo * g.K
                         : pass == PASS_DGRAD ? (double)g.N * g.H * g.W * g.C
                                              : (double)g.K * g.R * g.S * g.C;
        t += 3.0 + (pl.splits + 1.0) * out_elems * 4.0 / 4.0e6;   // ~4 TB/s for the partial traffic
    }
    return t;
}

}  // namespace

// Eligible fast-path plans of a pass, cheapest first by the model, at most two split counts per tile
// variant; returns how many were written (0: the shape has no fast-path plan).
int auto_plan_list(const ConvGeom &g, int pass, int force_splits, GemmPlan *out, int max_out, int restr, double *times)
{
    struct Priced { double t; GemmPlan pl; int code; };
    Priced all[512];
    int n = 0;
    // dense-layer-like shapes (a handful of pixel rows): the pass streams the weight matrix once and
    // is bound by HBM; the smallest tile with about two blocks per CU does that best
    if (pass != PASS_WGRAD && force_splits <= 0) {
        const long long rowsB = pass == PASS_FWD ? (long long)g.N * g.Ho * g.Wo : (long long)g.N * g.H * g.W;
        if (rowsB <= 64) {
            for (int code : {207, 103}) {
                GemmPlan one;
                if (!family_plan(g, pass, code, 1, &one, restr)) continue;
                const long long tiles = (long long)one.tilesA * one.tilesB;
                int splits = (int)((512 + tiles - 1) / tiles), max_splits = one.steps_total / 8;
                if (max_splits < 1) max_splits = 1;
                if (splits > max_splits) splits = max_splits;
                if (family_plan(g, pass, code, splits, &all[n].pl, restr)) { all[n].t = 0.0; all[n].code = code; ++n; break; }
            }
        }
    }
    const Candidate *cands = pass == PASS_WGRAD ? kWg : kPix;
    const int ncand = pass == PASS_WGRAD ? (int)(sizeof(kWg) / sizeof(kWg[0])) : (int)(sizeof(kPix) / sizeof(kPix[0]));
    for (int ci = 0; ci < ncand; ++ci) {
        if (pass == PASS_FWD && cands[ci].code == 405 && (restr & RESTR_ORDER)) continue;   // two halves of the reduction
        if (pass != PASS_WGRAD && cands[ci].code >= 400 && (restr & 1)) continue;   // the input-patch kernels store bf16 only
        if (pass == PASS_DGRAD && cands[ci].code >= 230 && cands[ci].code <= 233 && (restr & 1)) continue;   // bf16 staged epilogue only
        int last_splits = -1;
        for (int s : kSplits) {
            if (force_splits > 0 && s != kSplits[0]) break;
            // backward-filter blocks of one split share their inputs through one XCD's L2 only if the
            // split count is a multiple of the 8 XCDs
            if (pass == PASS_WGRAD && force_splits <= 0 && s > 8 && (s % 8) != 0) continue;
            GemmPlan cand;
            if (!family_plan(g, pass, cands[ci].code, force_splits > 0 ? force_splits : s, &cand, restr)) break;
            // reduction step 32 only where 64 does not divide the channel count
            if (pass != PASS_WGRAD && cand.BK == 32 && ((pass == PASS_FWD ? g.C : g.K) % 64) == 0) break;
            if (cand.splits == last_splits) continue;   // the request was clamped to the same plan
            // pixel-strip kernels on a grid of few blocks: each block streams its weights alone, which times well on a warm
            // cache (the measured choice) and badly inside a step
            // (restr bit 2: the caller measures with cold caches and can judge these grids itself)
            if (!(restr & 4) && cands[ci].code >= 230 && cands[ci].code <= 233 && (long long)cand.tilesA * cand.tilesB * cand.splits < 160) continue;
            last_splits = cand.splits;
            if (force_splits <= 0 && cand.splits > 1 && cand.steps_per_split < 4) break;
            double t = price(g, pass, cands[ci], cand, restr);
            GemmPlan w;
            // The nine-tap kernel had tiles of 256 pixels, fewer blocks and less scratch in some layers: a buffer that was enough for it then is enough
            if (cands[ci].code == 411 && (restr & RESTR_PATCH) && family_plan(g, pass, 410, cand.splits, &w) && family_plan(g, pass, 411, w.splits, &cand))
                t = price(g, pass, {411, 1, 0.10f, 6.0f}, w, restr);
            if (n < 512) { all[n].t = t; all[n].pl = cand; all[n].code = cands[ci].code; ++n; }
        }
    }
    // selection sort of the few that are wanted; per tile variant only its two cheapest splits
    int written = 0;
    int used_code[64], used_cnt[64], nused = 0;
    double t_first = -1.0;   // the model's best time; plans it puts beyond 1.6x of that are not worth a measurement
    while (written < max_out) {
        int best = -1;
        for (int i = 0; i < n; ++i) {
            if (all[i].t < 0.0) continue;
            if (best < 0 || all[i].t < all[best].t) best = i;
        }
        if (best < 0) break;
        if (all[best].t > 0.0) {
            if (t_first < 0.0) t_first = all[best].t;
            else if (all[best].t > ((restr & 4) ? 2.0 : 1.6) * t_first) break;
        }
        int u = 0;
        while (u < nused && used_code[u] != all[best].code) ++u;
        if (u == nused && nused < 64) { used_code[nused] = all[best].code; used_cnt[nused] = 0; ++nused; }
        if (u < 64 && used_cnt[u] < 2) {
            if (times != nullptr) times[written] = all[best].t;
            out[written++] = all[best].pl;
            ++used_cnt[u];
        }
        all[best].t = -1.0;
    }
    return written;
}

// Forward, channels that 64 does not divide: a flat-walk kernel in the place of `base` (32-wide steps), if one is faster.  It takes the
// reduction apart exactly as `base` does: the same splits, each a whole number of 64-wide steps, either as partials or as the
// reduction groups of a block.  Both walk (tap, channel) in 16-element slices, so the sums run in the same order and y is the same bit
// for bit.  That matters where gradients are taken through [y > 0]: an output whose sum lies at zero changes side with the order of the
// additions (80 -> 192 3x3, 4 x 73 x 73: one of 3.9 M outputs in every twentieth input set), which switches a whole term of dx on or off.
// The window kernel adds in another order; RESTR_ORDER leaves it out of the default choice of layers that mask by their own y.
// Where it is faster (old / new with the same splits, 376 layers):
//   generic kernel: from 3 steps on 1.02 - 1.73; below 0.81 - 1.36, the shortest layers lose
//   64x64 tiles of 32-wide steps, unsplit: 1 step 0.91, 3 steps 0.98, 4 steps 1.01, 6 and more 1.06 - 1.17; split 1.01 - 1.24
//   64x128 / 128x128 pipelined tiles of 32-wide steps: unsplit 0.79 - 1.15, with partials 0.93 - 1.17, neither worth the change; their 2 or
//   4 splits as reduction groups of blocks that all run at once, no reduction kernel: 1.39 - 1.63
bool forward_flat_plan(const ConvGeom &g, const GemmPlan &base, GemmPlan *out, double *time)
{
    if (g.C % 64 == 0 || g.C % 8 != 0 || g.R * g.S > 31 || base.BK != 32 || (base.splits > 1 && base.steps_per_split % 2 != 0)) return false;
    const int steps = (g.R * g.S * g.C + 63) / 64;
    const bool generic = !base.fast, staged = base.fast && !base.dma;
    if (base.splits == 1 && steps < (generic ? 3 : 6)) return false;
    double best = 0.0;
    bool found = false;
    for (const Candidate &c : kFlatFwd) {
        GemmPlan pl;
        if (!family_plan(g, PASS_FWD, c.code, c.kg > 1 ? 1 : base.splits, &pl)) return false;
        if (c.kg == 1) {
            if (!generic && !staged) continue;
            if (generic && base.splits > 1 && base.TA * base.TB == 128 * 128 && c.code != 239) continue;   // partials of many tiles: its tile
            if (pl.splits != base.splits || (base.splits > 1 && pl.steps_per_split * 2 != base.steps_per_split)) continue;
        } else {
            if (base.splits != c.kg || (steps + c.kg - 1) / c.kg * 2 != base.steps_per_split) continue;
            if (!generic && (long long)pl.tilesA * pl.tilesB > 256 * c.bpc) continue;
        }
        const double t = price(g, PASS_FWD, c, pl, 0);
        if (!found || t < best) { best = t; *out = pl; found = true; }
    }
    *time = best;
    return found;
}

// Backward-data, c_out in whole 8s that 64 does not divide: a flat-walk kernel in the place of `base` (32-wide steps; `time` its price) where
// that is faster.  Nothing depends on the order of these sums, so the splits are free.  Measured over 385 layers:
//   generic kernel: 1.01 - 5.9 times as fast; up to 32 input channels and under 3 steps 0.70 - 1.54, left alone.  With a saved output
//     the generic kernel masks dy while it loads and a flat one needs a pass over dy first (2 us and the traffic, 3 - 12 us for a small gradient):
//     under 7 steps 0.33 - 2.2, from there on 1.08 - 3.9, but for small gradients of 1x1 layers and of those that the
//     generic kernel splits (0.74 - 1.2)
//   64x64 register-staged tiles: 0.74 - 0.89 up to 7 steps, 0.93 - 1.15 beyond, left alone; 128x128 pipelined: 0.80 - 1.09, left alone
//   64x128 pipelined, unit stride: unsplit 0.76 - 1.07, left alone; split 0.96 - 1.5, taken where the prices are 8 % apart (then 1.04 - 1.5)
//   64x128 pipelined, stride 2 (by phase): split 1.2 - 1.5; unsplit from 5 steps on and in one block per CU 1.14 - 1.25, else 0.86 - 1.18
bool backward_flat_plan(const ConvGeom &g, const GemmPlan &base, double time, int restr, GemmPlan *out, double *flat_time)
{
    if (g.K % 64 == 0 || g.K % 8 != 0 || g.C % 8 != 0 || g.R * g.S > 31 || base.BK != 32) return false;
    const bool strided = g.sh > 1 || g.sw > 1, generic = !base.fast;
    if (strided && ((restr & 1) || g.sh > 2 || g.sw > 2)) return false;   // fp32 gradients of strided layers go in natural pixel order
    const int steps = (g.R * g.S * g.K + 63) / 64;
    if (generic) {
        if (g.C <= 32 && steps < 3) return false;
        if ((restr & RESTR_SAVED) && (steps < 7 || ((base.splits > 1 || g.R * g.S == 1) && (long long)g.N * g.Ho * g.Wo * g.K < 98304))) return false;
    } else {
        if (!base.dma || base.TA != 64 || base.TB != 128) return false;
        if (base.splits == 1 && (!strided || g.R * g.S == 1 || steps < 5)) return false;
    }
    double best = 0.0;
    bool found = false;
    for (const Candidate &c : kFlatBwd)
        for (int s : kSplits) {
            GemmPlan pl;
            if ((s > 1 && (strided || c.kg > 1)) || !family_plan(g, PASS_DGRAD, c.code, s, &pl, restr)) break;
            if (pl.splits > 1 && pl.steps_per_split < 4) break;
            if (!generic && base.splits == 1 && c.code == 234 && (long long)pl.tilesA * pl.tilesB > 256) return false;
            const double t = price(g, PASS_DGRAD, c, pl, restr) + (pl.splits > 1 ? 1.5 : 0.0);
            if (!found || t < best) { best = t; *out = pl; found = true; }
        }
    *flat_time = best;
    return found && (generic || strided || best < 0.92 * time);
}

// Forward / backward-data by the window kernel (conv_win.hip): us = c0 + rounds of blocks * (c1 + rounds of channels * (c2 + c3 taps + c4 window rows)),
// fitted to 2420 timings (310 layers; median error 2 - 4 %, 5 - 9 % for nine of ten), the tiles of 96 channels to 570 (130 layers; 2 - 3 %, 6 - 9 %)
struct WindowPrice { float c0, c1, c2, c3, c4; };
const WindowPrice kWindowPrice[2][9] = {
    {{-0.6f, 7.5f, 0.13f, 0.280f, 0.0023f}, {1.5f, 4.1f, 0.48f, 0.098f, 0.0007f}, {1.9f, 3.1f, 0.45f, 0.090f, 0.0006f}, {1.4f, 4.0f, 0.44f, 0.188f, 0.0001f},
     {1.2f, 4.4f, 0.29f, 0.196f, 0.0011f}, {1.2f, 5.7f, 0.39f, 0.143f, 0.0014f},
     {1.0f, 4.0f, 0.29f, 0.173f, 0.0008f}, {0.8f, 5.3f, 0.40f, 0.194f, 0.0005f}, {-0.3f, 7.2f, 0.35f, 0.222f, 0.0013f}},
    {{-0.3f, 7.0f, 0.0f, 0.307f, 0.0034f}, {1.5f, 4.9f, 0.39f, 0.103f, 0.0006f}, {1.9f, 3.1f, 0.38f, 0.101f, 0.0006f}, {1.4f, 4.8f, 0.36f, 0.189f, 0.0003f},
     {1.3f, 5.3f, 0.18f, 0.189f, 0.0017f}, {1.0f, 5.5f, 0.34f, 0.160f, 0.0015f},
     {1.3f, 3.6f, 0.18f, 0.200f, 0.0006f}, {1.0f, 5.1f, 0.17f, 0.213f, 0.0013f}, {0.4f, 5.9f, 0.0f, 0.262f, 0.0024f}}};

// What masking dy by the saved output on its way into the window costs: two loads and an LDS store in the place of a copy (median of 31 - 75 layers
// per tile; 1.08 - 1.28 for nine of ten)
const float kMaskedWindow[9] = {1.045f, 1.13f, 1.165f, 1.135f, 1.085f, 1.08f, 1.14f, 1.125f, 1.06f};

bool pixel_window_exists(const ConvGeom &g, int pass)
{
    if (g.sh != 1 || g.sw != 1 || g.R * g.S < 3) return false;   // asked on every call
    GemmPlan pl;
    for (int v = 0; v < 9; ++v)
        if (family_plan(g, pass, 250 + v, 1, &pl)) return true;
    return false;
}

// its two cheapest plans, best first; returns how many there are
int pixel_window_plans(const ConvGeom &g, int pass, GemmPlan out[2], double times[2], bool saved)
{
    int n = 0;
    for (int v = 0; v < 9; ++v) {
        GemmPlan pl;
        int rounds, rows;   // channel rounds of a block, window rows copied per round
        if (!family_plan(g, pass, 250 + v, 1, &pl) || !win_work(g, pass, v, &rounds, &rows)) continue;
        const WindowPrice &c = kWindowPrice[pass == PASS_FWD ? 0 : 1][v];
        const double waves = std::ceil((double)pl.tilesA * pl.tilesB / 256.0);
        double t = c.c0 + waves * (c.c1 + rounds * (c.c2 + c.c3 * g.R * g.S + c.c4 * rows));
        if (saved) t *= kMaskedWindow[v];
        // backward-data with 32 channels to a tile fetches half a line per weight row, which counts where the weights are more than an L2 holds (88 layers,
        // measured / fitted: up to 4 MB 0.86 - 1.03, beyond 0.80 - 1.75, 1.12 in the middle)
        if (v == 2 && pass == PASS_DGRAD && (long long)g.K * g.R * g.S * g.C * 2 > 4 << 20) t *= 1.15;
        if (n == 0 || t < times[0]) {
            if (n > 0) { out[1] = out[0]; times[1] = times[0]; }
            out[0] = pl; times[0] = t;
            n = std::min(n + 1, 2);
        } else if (n == 1 || t < times[1]) {
            out[1] = pl; times[1] = t;
            n = 2;
        }
    }
    return n;
}

// The window kernel in the place of `base` (price `time`), where its own price lies 8 % below what the other's is worth: the prices were made to rank
// the kernels among themselves and are off by a launch's floor and a factor, fitted per family to 510 passes timed both ways (median error 3 - 6 %;
// register-staged and flat kernels by a factor alone).  `mask_us`: what a pass over dy in front of `base` takes, which the window kernel does without.
bool pixel_window_plan(const ConvGeom &g, int pass, const GemmPlan &base, double time, bool saved, double mask_us, GemmPlan *out)
{
    GemmPlan pl[2];
    double t[2];
    if (!base.fast || time <= 0.0 || pixel_window_plans(g, pass, pl, t, saved) == 0) return false;
    const bool fwd = pass == PASS_FWD, split = base.splits > 1;
    if (!fwd && base.BK == 32 && pl[0].variant >= 6 && g.R * g.S < 5) return false;   // 96-channel tiles were fitted from 7 taps on
    double floor_us = 0.0, factor = 0.0;   // not in the place of unsplit register-staged kernels forward, nor of flat ones backward with few taps or short reductions
    // Few enough tiles that the smallest window tile is the cheapest: less to fetch before its first product than nine taps of weights (64 channels; 240 layers of
    // up to 80 tiles: forward 0.90 - 0.95 of the time with flushed caches (8.7 -> 8.1 us) and 0.94 - 1.00 back to back, masked backward-data 0.94 - 1.01 and 0.95 - 1.01)
    if (base.halo && base.variant == 4 && pl[0].variant == 2) { *out = pl[0]; return true; }
    if (base.halo && base.variant == 4) factor = 1.0;
    else if (base.halo && base.variant == 5) { floor_us = -4.5; factor = 1.12; }
    else if (base.halo) { floor_us = fwd ? 0.3 : -1.6; factor = fwd ? 1.13 : 1.34; }
    else if (dma_plan_is_strip(base)) { floor_us = -4.4; factor = fwd ? 1.11 : 1.16; }
    else if (dma_plan_is_flat(base)) factor = fwd || (g.R * g.S > 8 && g.R * g.S * g.K >= 512) ? 1.0 : 0.0;   // backward-data: 1.17 - 1.78 times as fast
    else if (!base.dma) { floor_us = fwd ? 0.0 : -3.6; factor = !fwd ? 1.03 : split ? 0.76 : 0.0; }
    else if (fwd) { floor_us = split ? -7.0 : -4.6; factor = split ? 1.3 : 1.08; }
    else { floor_us = split ? -6.0 : -4.4; factor = split ? 1.3 : 1.25; }
    double worth = floor_us + factor * time;
    if (fwd && base.dma && base.BK == 32) worth = std::max(worth, 1.5 * time - 14.0);   // 32-wide steps: 1.3 - 1.6 of the price for long layers, 0.75 for short ones
    if (base.dma && base.BK != 32 && !base.halo && !dma_plan_is_strip(base)) worth = std::min(worth, (fwd ? 1.0 : 1.05) * time);   // long: 0.8 - 1.0, 0.95 - 1.15
    // more than one round of blocks: the last one is priced as full, the others' is not; three or four taps: little is saved on the window, and
    // the shortest layers lie at the floor of a launch
    const long long tiles = (long long)pl[0].tilesA * pl[0].tilesB;
    const double margin = g.R * g.S < 5 ? 0.75 : tiles > 512 ? 0.78 : tiles > 256 ? 0.85 : 0.92;
    if (t[0] >= margin * (worth + mask_us)) return false;
    *out = pl[0];
    return true;
}

// 1x1 layers by the kernel with stationary weights (conv_pw.hip), us with cold caches, fitted to 768 timings of 560 passes (64 - 512 reduction channels,
// 16 - 2048 others, 7 - 100 pixels, 1 - 64 samples; median error 5 %, 13 % for nine of ten): a launch, the weights, then the longer of what a block does for
// its buffers of pixels and what memory takes.  The cheapest tile by it is 1 % slower than the fastest in the mean, 5 % for nineteen of twenty.
double price_pointwise(const ConvGeom &g, int pass, const GemmPlan &pl, bool masked)
{
    const bool fwd = pass == PASS_FWD;
    const double rows = fwd ? (double)g.N * g.Ho * g.Wo : (double)g.N * g.H * g.W, red = fwd ? g.C : g.K, outs = fwd ? g.K : g.C;
    const int tc = pl.steps_total, aw = pl.variant == 2 ? 2 : 1, groups = pl.TB / 32, frags = pl.variant == 0 ? groups / 2 : groups, blocks = pw_blocks(pl);
    const double waves = std::max(1.0, (double)blocks * pl.tilesA / 512.0), buffers = std::ceil((double)pl.tilesB / blocks);
    const int per_cu = std::min(2, (blocks * pl.tilesA + 255) / 256);
    const double work = buffers * waves * (0.38 + frags * aw * (0.097 * tc * per_cu + 0.20 + (masked ? 0.21 : 0.0)) + (pl.pw_gather ? 0.35 * groups : 0.0));
    const double memory = (0.27 * rows * (red + outs * (masked ? 2 : 1)) + 0.022 * rows * red * (pl.tilesA - 1)) * 2e-6;
    return 5.8 + 0.31 * tc * aw * waves + std::sqrt(std::sqrt(std::pow(work, 4) + std::pow(memory, 4)));
}

// its two cheapest plans, best first; returns how many there are
int pointwise_plans(const ConvGeom &g, int pass, bool masked, GemmPlan out[2], double times[2])
{
    int n = 0;
    for (int v = 0; v < 3; ++v) {
        GemmPlan pl;
        if (!family_plan(g, pass, 260 + v, 0, &pl)) continue;
        const double t = price_pointwise(g, pass, pl, masked);
        if (n == 0 || t < times[0]) {
            if (n > 0) { out[1] = out[0]; times[1] = times[0]; }
            out[0] = pl; times[0] = t;
            n = std::min(n + 1, 2);
        } else if (n == 1 || t < times[1]) {
            out[1] = pl; times[1] = t;
            n = 2;
        }
    }
    return n;
}

// The stationary-weight kernel in the place of `base`, 560 passes timed both ways (other / this, back to back):
//   backward-data: 0.96 - 3.2, 1.33 in the middle, whatever the size (with flushed caches 0.93 - 2.0, 1.14)
//   forward, from 8 MB of pixels on: 0.95 - 2.5, 1.21 in the middle; below, both lie at the floor of a launch or the tiles are faster (0.74 - 1.1).
//   Up to 32 output channels half a tile and more is idle: 0.91 - 0.96.  Strided, from 16 MB on 0.97 - 1.6; below, the places of its pixels cost 0.77 - 1.0.
// Forward keeps the order of its sums (forward_flat_plan), which is that of the tiles that take the reduction in one piece.
bool pointwise_plan(const ConvGeom &g, int pass, const GemmPlan &base, bool masked, GemmPlan *out)
{
    GemmPlan pl[2];
    double t[2];
    if (pass == PASS_FWD) {
        const double mb = (double)g.N * g.Ho * g.Wo * (g.C + g.K) * 2e-6;
        if (g.K < 48 || mb < (g.sh > 1 || g.sw > 1 ? 16.0 : 8.0)) return false;
        if (base.splits > 1 || dma_plan_groups(base) > 1) return false;
    } else if ((long long)g.N * g.H * g.W < 256) return false;   // not timed
    if (pointwise_plans(g, pass, masked, pl, t) == 0) return false;
    *out = pl[0];
    return true;
}

// The filter gradient's window kernel: its two cheapest plans, best first; returns how many there are.  Chunks of 256 slots where the window fits (never slower
// than 128 in the timings behind price_window), up to eight splits or what fills the chip once or twice.
int wgrad_window_plans(const ConvGeom &g, GemmPlan out[2], double times[2])
{
    GemmPlan pl;
    const int code = family_plan(g, PASS_WGRAD, 318, 1, &pl) ? 318 : 317;
    if (!family_plan(g, PASS_WGRAD, code, 1, &pl)) return 0;
    const int tiles = pl.tilesA * pl.tilesB, wanted[] = {1, 2, 3, 4, 5, 6, 8, 256 / tiles, 512 / tiles};
    int n = 0;
    for (int s : wanted) {
        if (s < 1 || !family_plan(g, PASS_WGRAD, code, s, &pl) || (pl.splits > 1 && pl.steps_per_split < 2)) continue;
        const double t = price_window(g, pl);
        if ((n > 0 && out[0].splits == pl.splits) || (n > 1 && out[1].splits == pl.splits)) continue;
        if (n == 0 || t < times[0]) {
            if (n > 0) { out[1] = out[0]; times[1] = times[0]; }
            out[0] = pl; times[0] = t;
            n = std::min(n + 1, 2);
        } else if (n == 1 || t < times[1]) {
            out[1] = pl; times[1] = t;
            n = 2;
        }
    }
    return n;
}

// The nine-tap filter gradient of 64-channel layers (conv_halo.hip) by its own price, whole passes in us: fitted to 125 timings (median error 6 %, 11 % for nine
// of ten).  False: another layer.
bool nine_tap_plan(const ConvGeom &g, GemmPlan *out, double *time)
{
    bool found = false;
    for (int blocks : {256, 192, 128}) {
        GemmPlan pl;
        const int per_tile = std::max(blocks / ((g.K + 63) / 64), 2);
        if (!family_plan(g, PASS_WGRAD, 411, per_tile, &pl)) return found;
        const double t = 10.1 + 0.173 * pl.steps_per_split + 1.26e-6 * (pl.splits + 1) * g.K * g.R * g.S * g.C;
        if (!found || t < *time) { *out = pl; *time = t; found = true; }
    }
    return found;
}

// The window kernel's plan of a layer that the nine-tap kernel may take instead: what a call with less scratch than that asks for falls back to
bool wgrad_window_form(const ConvGeom &g, GemmPlan *out)
{
    GemmPlan pl[2];
    double t[2];
    if (!family_plan(g, PASS_WGRAD, 411, 0, &pl[0]) || wgrad_window_plans(g, pl, t) == 0) return false;
    *out = pl[0];
    return true;
}

// Filter gradient: the window kernel in the place of `base` (price `time`) where its price lies that far below.  The factors are what the
// other kernels' prices are worth on 230 layers timed both ways: pipelined tiles take 0.7 - 1.1 of their price split and down to 0.6 unsplit,
// register-staged ones 1.1 - 1.6, the input-patch kernel with a wave per tap 1.4 - 2.2.  Taken on 48 of 175 layers that both run: 0.98 - 2.0 times as fast.
bool wgrad_window_plan(const ConvGeom &g, const GemmPlan &base, double time, GemmPlan *out)
{
    GemmPlan pl[2];
    double t[2];
    if (!base.fast || wgrad_window_plans(g, pl, t) == 0) return false;
    const double worth = !pl[0].row_taps ? 0.8 : base.halo ? 1.35 : !base.dma ? 1.0 : base.splits == 1 ? 0.75 : 0.92;
    const bool nine = base.halo && base.variant == 11;
    if (!nine && t[0] >= worth * time) return false;
    // Both by prices of their own, where the window kernel has won against `base` or that is the nine-tap kernel.  With flushed caches the window kernel loses
    // 10 - 50 % more (40 layers nearer than that to each other back to back; 60 layers that went to the nine-tap kernel: 1.04 of its time warm in the middle, 0.92 cold)
    GemmPlan nine_pl;
    double nine_time;
    if (nine_tap_plan(g, &nine_pl, &nine_time) && t[0] >= 0.96 * nine_time) { *out = nine_pl; return true; }
    *out = pl[0];
    return true;
}

// Fills *pl with the cheapest eligible fast-path plan; false if the shape has none.
bool auto_plan(const ConvGeom &g, int pass, int force_splits, GemmPlan *pl, int restr, double *time)
{
    return auto_plan_list(g, pass, force_splits, pl, 1, restr, time) == 1;
}
