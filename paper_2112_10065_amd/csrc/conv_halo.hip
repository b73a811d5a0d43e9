// Forward / backward-data kernels for stride-1 layers whose reduction has exactly 64 channels per
// tap (VGG conv1_2, conv2_1): the tiled kernels re-fetch every input pixel once per filter tap, and
// with only R*S reduction steps per tile that traffic through the per-CU global->LDS path is what
// bounds them.  Here a block owns a TH x TW patch of output pixels of one image (TH*TW = 256) and
// copies the input patch with its halo ((TH+R-1) x (TW+S-1) pixels x 64 channels, zero outside the
// image) into LDS ONCE; the R*S taps then read their pixel rows from that patch at shifted positions.
// Only the weight tile of each tap still streams through the NS-stage pipeline.
//
// Patch layout: pixel pp = pr*(TW+S-1) + pc occupies 128 bytes; its 16-byte channel chunk c sits at
// chunk position c ^ ((pp >> 1) & 7) (two 128-byte rows span the 64 banks), which makes the fragment reads of 32 consecutive pixels conflict-free.
// A direct-to-LDS instruction fills 8 consecutive patch pixels.
#include "dma_common.h"
#include <utility>
#include <cstdio>

namespace {

constexpr int HALO_TB = 256;        // output pixels per tile
constexpr int HALO_PP = 352;        // patch pixels the LDS slot holds (44 KiB): 10x34 and 18x18 fit

// PASS_FWD : A = weights [c_out][tap][64 c_in] (rows K-major in LDS), patch from x.
// PASS_DGRAD: A = weights [64 c_out][tap][c_in] kept reduction-major in LDS and read with the LDS
//             transpose read, patch from dy; tap (r, s) of the filter meets patch offset (R-1-r, S-1-s).
template <int PASS, int TA, int WA, int WB, int NS>
__global__ __launch_bounds__(64 * WA * WB) void k_halo(const KArgs p, int tws, int tiles_x, int tiles_y)
{
    constexpr int NT = 64 * WA * WB, NW = WA * WB, TB = HALO_TB;
    constexpr int KS = 4;                                     // 16-wide slices per 64-channel step
    constexpr int FA = TA / WA / 32, FB = TB / WB / 32;
    constexpr int A_BYTES = TA * 128;                         // one tap's weight tile (either orientation)
    constexpr int IA = A_BYTES / 1024 / NW;                   // weight copies per wave and step
    constexpr int IP = (HALO_PP * 128 / 1024 + NW - 1) / NW;  // patch copies per wave
    constexpr int PATCH_BYTES = IP * NW * 1024;
    static_assert(IA * NW * 1024 == A_BYTES, "weight tile must divide over the waves");
    constexpr int STAGES_END = PATCH_BYTES + NS * A_BYTES, EPI = TB * (TA + 8) * 2;
    constexpr int TILE_BYTES = STAGES_END > EPI ? STAGES_END : EPI;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    float *bias_lds = reinterpret_cast<float *>(smem + TILE_BYTES);   // [TA]

    const ConvGeom &g = p.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int R = g.R, S = g.S, TW = 1 << tws, TH = TB >> tws, PW = TW + S - 1, PP = (TH + R - 1) * PW;
    const int tile = logical_block(blockIdx.x, gridDim.x);
    const int a0 = (tile % p.tilesA) * TA, bt = tile / p.tilesA;
    const int n = bt / (tiles_x * tiles_y), trem = bt - n * (tiles_x * tiles_y), ty = trem / tiles_x, tx = trem - ty * tiles_x;
    const int p0 = ty * TH, q0 = tx * TW;
    // image the patch is cut from, its extent, and the patch origin
    const int IH = PASS == PASS_FWD ? g.H : g.Ho, IW = PASS == PASS_FWD ? g.W : g.Wo;
    const int h0 = PASS == PASS_FWD ? p0 - g.ph : p0 + g.ph - (R - 1), w0 = PASS == PASS_FWD ? q0 - g.pw : q0 + g.pw - (S - 1);
    const int OH = PASS == PASS_FWD ? g.Ho : g.H, OW = PASS == PASS_FWD ? g.Wo : g.W;   // output image
    const int RSC = R * S * g.C;
    __amdgpu_buffer_rsrc_t rw = make_rsrc(p.w, (size_t)g.K * RSC * 2);
    __amdgpu_buffer_rsrc_t rsrc_in = PASS == PASS_FWD ? make_rsrc(p.x, (size_t)g.N * g.H * g.W * g.C * 2)
                                                      : make_rsrc(p.dy, (size_t)g.N * g.Ho * g.Wo * g.K * 2);
    const unsigned smem_base = lds_offset(smem);

    if ((p.flags & KF_BIAS) && PASS == PASS_FWD)
        for (int i = tid; i < TA; i += NT) bias_lds[i] = a0 + i < p.rowsA ? p.bias[a0 + i] : 0.f;

    // ---- patch: all copies issued up front -------------------------------------------------
#pragma unroll
    for (int q = 0; q < IP; ++q) {
        const int id = (wave * IP + q) * 64 + lane, pp = id >> 3, c = (id & 7) ^ ((pp >> 1) & 7);
        const int pr = pp / PW, pc = pp - pr * PW, ih = h0 + pr, iw = w0 + pc;
        const bool ok = pp < PP && (unsigned)ih < (unsigned)IH && (unsigned)iw < (unsigned)IW;
        const unsigned voff = ok ? (unsigned)(((n * IH + ih) * IW + iw) * 64 + c * 8) * 2u : OOR;
        dma16(rsrc_in, smem_base + (wave * IP + q) * 1024, voff);
    }

    // ---- weight tile of one tap ----------------------------------------------------------------
    unsigned voffA[IA];
#pragma unroll
    for (int q = 0; q < IA; ++q) {
        if (PASS == PASS_FWD) {   // row = c_out, 8 rows per copy, chunk swizzle by row pair
            const int row = (wave * IA + q) * 8 + lane / 8;
            const int c = (lane % 8) ^ ((row / 2) % 8);
            voffA[q] = ((unsigned)(a0 + row) * RSC + c * 8) * 2u;
        } else {                  // row = c_out (reduction), TA c_in per row, 512/TA rows per copy, segment swizzle
            const int t = (wave * IA + q) * (512 / TA) + lane / (TA / 8);
            const int c = (lane % (TA / 8)) ^ (seg_swz<TA>(t) << 2);
            voffA[q] = ((unsigned)t * RSC + a0 + c * 8) * 2u;
        }
    }
    const unsigned ldsA_w = smem_base + PATCH_BYTES + wave * IA * 1024;
    auto issueA = [&](int stage, int step) {   // filter tap of reduction step `step`
        const int tap = PASS == PASS_FWD ? step : (R * S - 1 - step);
        const unsigned ua = (unsigned)tap * g.C * 2u;
#pragma unroll
        for (int q = 0; q < IA; ++q) dma16(rw, ldsA_w + stage * A_BYTES + q * 1024, voffA[q] + ua);
    };

    f32x16 acc[FA][FB];
#pragma unroll
    for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int j = 0; j < FB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    const int arow = (wave % WA) * FA * 32, brow = (wave / WA) * FB * 32;

    // fragment addresses of the weight tile
    unsigned fa[KS][PASS == PASS_FWD ? 1 : FA];
    if (PASS == PASS_FWD) {
        const int rA = arow + (lane & 31);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            fa[ks][0] = smem_base + PATCH_BYTES + rA * 128 + (((2 * ks + (lane >> 5)) ^ ((rA / 2) % 8)) << 4);
    } else {
        const int i16 = lane & 15, tl = (lane >> 5) * 8 + (i16 >> 2), cl = ((lane >> 4) & 1) * 16 + (i16 & 3) * 4;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int t = ks * 16 + tl;
#pragma unroll
            for (int i = 0; i < (PASS == PASS_FWD ? 1 : FA); ++i) {
                const int col = arow + i * 32 + cl;
                fa[ks][i] = smem_base + PATCH_BYTES + t * (TA * 2) + ((((col >> 5) ^ seg_swz<TA>(t)) << 6) | ((col & 31) << 1));
            }
        }
    }
    // patch pixel of this lane's row in each of its B fragments, at patch offset (0, 0)
    int pp0[FB];
#pragma unroll
    for (int j = 0; j < FB; ++j) {
        const int jj = brow + j * 32 + (lane & 31);
        pp0[j] = (jj >> tws) * PW + (jj & (TW - 1));
    }
    const unsigned hsel = lane >> 5;

    const int nsteps = R * S;
    constexpr int LPS = IA;
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (s < nsteps) issueA(s, s);

    u32x4 fr_a[2][FA], fr_b[2][FB];
    u32x2 tr_lo[2][FA], tr_hi[2][FA];
    unsigned brow_addr[FB], bsw[FB];
    auto set_tap = [&](int step) {   // patch rows of reduction step `step` (patch offset r*PW + s)
        const int r = step / S, s = step - r * S;
        const int off = r * PW + s;
#pragma unroll
        for (int j = 0; j < FB; ++j) {
            const int pp = pp0[j] + off;
            brow_addr[j] = smem_base + pp * 128;
            bsw[j] = (pp >> 1) & 7;
        }
    };
    auto read_slice = [&](int ks, int buf, unsigned sb) {
        if constexpr (PASS == PASS_FWD) {
            if constexpr (FA >= 1) fr_a[buf][0] = lds_read16<0>(fa[ks][0] + sb);
            if constexpr (FA >= 2) fr_a[buf][1] = lds_read16<32 * 128>(fa[ks][0] + sb);
            if constexpr (FA >= 3) fr_a[buf][2] = lds_read16<64 * 128>(fa[ks][0] + sb);
            if constexpr (FA >= 4) fr_a[buf][3] = lds_read16<96 * 128>(fa[ks][0] + sb);
        } else {
#pragma unroll
            for (int i = 0; i < FA; ++i) {
                tr_lo[buf][i] = lds_read_tr<0>(fa[ks][i] + sb);
                tr_hi[buf][i] = lds_read_tr<4 * TA * 2>(fa[ks][i] + sb);
            }
        }
#pragma unroll
        for (int j = 0; j < FB; ++j) fr_b[buf][j] = lds_read16<0>(brow_addr[j] + (((2 * ks + hsel) ^ bsw[j]) << 4));
    };
    constexpr int RPS_ = (PASS == PASS_FWD ? FA : 2 * FA) + FB;   // LDS reads per slice
    static_assert(RPS_ < 16, "lgkmcnt is a 4-bit counter");
    auto wait_slice = [&](int buf, bool newer_in_flight) {
        if (newer_in_flight) asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(RPS_));
        else asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
        for (int i = 0; i < FA; ++i) {
            if constexpr (PASS == PASS_FWD) asm volatile("" : "+v"(fr_a[buf][i]));
            else { asm volatile("" : "+v"(tr_lo[buf][i])); asm volatile("" : "+v"(tr_hi[buf][i])); }
        }
#pragma unroll
        for (int j = 0; j < FB; ++j) asm volatile("" : "+v"(fr_b[buf][j]));
    };

    // patch and the first weight tile have landed; later weight tiles may be in flight
    {
        const int younger = min(NS - 1, nsteps - 1);
        if (NS >= 2 && younger == NS - 1) wait_vmcnt<(NS - 1) * LPS>();
        else if (NS >= 3 && younger == NS - 2) wait_vmcnt<(NS >= 3 ? NS - 2 : 0) * LPS>();
        else if (NS >= 4 && younger == NS - 3) wait_vmcnt<(NS >= 4 ? NS - 3 : 0) * LPS>();
        else wait_vmcnt<0>();
    }
    __syncthreads();   // also publishes bias_lds
    set_tap(0);
    read_slice(0, 0, 0);
    for (int i = 0; i < nsteps; ++i) {
        const unsigned sb = (i % NS) * A_BYTES;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int cur = ks & 1;
            if (ks < KS - 1) {
                read_slice(ks + 1 < KS ? ks + 1 : 0, cur ^ 1, sb);
                wait_slice(cur, true);
            } else {
                wait_slice(cur, false);   // this wave has read all it needs of the weight stage
                if (i + 1 < nsteps) {
                    const int younger = min(i + NS - 1, nsteps - 1) - (i + 1);
                    if (NS >= 3 && younger == NS - 2) wait_vmcnt<(NS - 2) * LPS>();
                    else if (NS >= 4 && younger == NS - 3) wait_vmcnt<(NS >= 4 ? NS - 3 : 0) * LPS>();
                    else wait_vmcnt<0>();
                    __builtin_amdgcn_s_barrier();
                    if (i + NS < nsteps) issueA(i % NS, i + NS);
                    set_tap(i + 1);
                    read_slice(0, 0, ((i + 1) % NS) * A_BYTES);
                }
            }
#pragma unroll
            for (int ii = 0; ii < FA; ++ii)
#pragma unroll
                for (int jj = 0; jj < FB; ++jj) {
                    u32x4 av;
                    if constexpr (PASS == PASS_FWD) av = fr_a[cur][ii];
                    else av = u32x4{tr_lo[cur][ii].x, tr_lo[cur][ii].y, tr_hi[cur][ii].x, tr_hi[cur][ii].y};
                    acc[ii][jj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av),
                                                                         __builtin_bit_cast(bf16x8, fr_b[cur][jj]), acc[ii][jj], 0, 0, 0);
                }
        }
    }
    __syncthreads();   // every wave is done reading patch and stages before they are reused for staging

    // ---- epilogue: bias / ReLU / bf16 through LDS, 16-byte rows to the NHWC output ------------
    constexpr int LSO = TA + 8;
    bf16_t *stage = reinterpret_cast<bf16_t *>(smem);
#pragma unroll
    for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq) {
            const int ch = arow + i * 32 + 8 * gq + 4 * (lane >> 5);
            f32x4 bv = {0.f, 0.f, 0.f, 0.f};
            if ((p.flags & KF_BIAS) && PASS == PASS_FWD) bv = *reinterpret_cast<const f32x4 *>(bias_lds + ch);
#pragma unroll
            for (int j = 0; j < FB; ++j) {
                float v0 = acc[i][j][4 * gq] + bv.x, v1 = acc[i][j][4 * gq + 1] + bv.y;
                float v2 = acc[i][j][4 * gq + 2] + bv.z, v3 = acc[i][j][4 * gq + 3] + bv.w;
                if ((p.flags & KF_RELU) && PASS == PASS_FWD) { v0 = fmaxf(v0, 0.f); v1 = fmaxf(v1, 0.f); v2 = fmaxf(v2, 0.f); v3 = fmaxf(v3, 0.f); }
                const int pix = brow + j * 32 + (lane & 31);
                *reinterpret_cast<u32x2 *>(stage + pix * LSO + ch) = u32x2{pack_bf16(v0, v1), pack_bf16(v2, v3)};
            }
        }
    constexpr int CPR = TA / 8;
    bf16_t *out = reinterpret_cast<bf16_t *>(p.out);
    if (PASS == PASS_DGRAD && (p.flags & KF_MASK_IN)) {
        // fused backward of the input ReLU: all saved-input vectors of this thread are requested before the
        // staging barrier, so that their latency overlaps
        constexpr int ITERS = TB * CPR / NT;
        static_assert(TB * CPR % NT == 0 && ITERS <= 16, "copy-out iterations");
        u32x4 xm[ITERS];
#pragma unroll
        for (int u = 0; u < ITERS; ++u) {
            const int id = tid + u * NT, pix = id / CPR, cc = id % CPR;
            const int pr = p0 + (pix >> tws), qc = q0 + (pix & (TW - 1)), gc = a0 + cc * 8;
            xm[u] = (pr < OH && qc < OW && gc < p.rowsA) ? ldg16(p.x + ((size_t)(n * OH + pr) * OW + qc) * p.rowsA + gc) : u32x4{0, 0, 0, 0};
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < ITERS; ++u) {
            const int id = tid + u * NT, pix = id / CPR, cc = id % CPR;
            const int pr = p0 + (pix >> tws), qc = q0 + (pix & (TW - 1)), gc = a0 + cc * 8;
            if (pr < OH && qc < OW && gc < p.rowsA)
                *reinterpret_cast<u32x4 *>(out + ((size_t)(n * OH + pr) * OW + qc) * p.rowsA + gc) =
                    apply_mask(*reinterpret_cast<const u32x4 *>(stage + pix * LSO + cc * 8), xm[u]);
        }
        return;
    }
    __syncthreads();
#pragma unroll
    for (int id = tid; id < TB * CPR; id += NT) {
        const int pix = id / CPR, cc = id % CPR;
        const int pr = p0 + (pix >> tws), qc = q0 + (pix & (TW - 1)), gc = a0 + cc * 8;
        if (pr < OH && qc < OW && gc < p.rowsA)
            *reinterpret_cast<u32x4 *>(out + ((size_t)(n * OH + pr) * OW + qc) * p.rowsA + gc) =
                *reinterpret_cast<const u32x4 *>(stage + pix * LSO + cc * 8);
    }
}

// Filter gradient, what a product over whole tiles does not give: a tile that reaches past the last row or column holds zeros of dy there, and they meet the
// pixels of x that lie in the patch beside them (or padding's zeros meet a dy).  Zero times infinity is NaN, so a sum with a NaN is made again from the pairs
// that the tap has: dW[row .. row + 3][tap][col] over this block's tiles of th x tw pixels.  Line by line, so that the sums stay as short as the
// product's; a sum that is all NaN stays so.  The check costs up to 0.3 us (2 x 56 x 56, 64 -> 64: 15.3 -> 15.6), such a sum what a plain loop costs
// (8 x 153 x 149, 64 -> 128 with one infinite pixel in the last column: 40 us -> 2.2 ms).
DEVFN f32x4 sum_of_pairs(const KArgs &p, int tiles_x, int tiles_y, int tiles, int th, int tw, int row, int tap, int col)
{
    const ConvGeom &g = p.g;
    const TileWalk walk = tile_walk(tiles);
    const int r = tap / g.S - g.ph, s = tap % g.S - g.pw;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int t = walk.first; t < walk.end; t += walk.stride) {
        const int n = t / (tiles_x * tiles_y), rem = t - n * (tiles_x * tiles_y), ty = rem / tiles_x, q0 = (rem - ty * tiles_x) * tw;
        const int h0 = max(ty * th, -r), h1 = min(min(ty * th + th, g.Ho), g.H - r), w0 = max(q0, -s), w1 = min(min(q0 + tw, g.Wo), g.W - s);
        for (int h = h0; h < h1; ++h) {
            const bf16_t *dy = p.dy + ((size_t)(n * g.Ho + h) * g.Wo) * g.K + row, *x = p.x + ((ptrdiff_t)(n * g.H + h + r) * g.W + s) * 64 + col;
            f32x4 line = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
            for (int w = w0; w < w1; ++w) {
                const u32x2 d = *reinterpret_cast<const u32x2 *>(dy + (size_t)w * g.K);
                const float v = __uint_as_float((unsigned)*reinterpret_cast<const unsigned short *>(x + (ptrdiff_t)w * 64) << 16);
                line.x = fmaf(__uint_as_float(d.x << 16), v, line.x); line.y = fmaf(__uint_as_float(d.x & 0xffff0000u), v, line.y);
                line.z = fmaf(__uint_as_float(d.y << 16), v, line.z); line.w = fmaf(__uint_as_float(d.y & 0xffff0000u), v, line.w);
            }
            sum += line;
        }
        if (sum.x != sum.x && sum.y != sum.y && sum.z != sum.z && sum.w != sum.w) break;
    }
    return sum;
}

// ---------------------------------------------------------------------------------------
// Backward-filter with the input patch in LDS (stride 1, 64 input channels, up to 16 taps).
// The tiled kernel copies, for every 64 pixels of reduction, the x rows of each tap again; here a
// block copies the x patch of a 256-pixel tile once, next to the tile's 256 x 64 slice of dy, and
// wave t accumulates tap t: dW[k][t][c] += sum over the tile's pixels of dy[pixel][k] * x[pixel + tap t][c]
// (64 c_out x 64 c_in per wave = 4 matrix tiles).  Both operands are pixel-major in LDS (rows of 128
// bytes, 64-byte segment swizzle by (row/2)&1) and read with the LDS transpose read.  Blocks are
// persistent: they walk tiles blockIdx.x, +gridDim.x, ... with the next tile's copies in flight
// (two LDS buffers), keep their sums in registers, and write ONE fp32 partial per block, which the
// split-reduce kernel adds in block order.  grid = (blocks, 64-row tiles of c_out).
// ---------------------------------------------------------------------------------------
constexpr int WH_BUF = HALO_PP * 128 + HALO_TB * 128;   // patch + dy slice of one tile: 76 KiB

__global__ __launch_bounds__(1024) void k_wgrad_halo(const KArgs p, int tws, int tiles_x, int tiles_y, int tiles)
{
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const ConvGeom &g = p.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwaves = blockDim.x >> 6;   // wave = tap
    const int R = g.R, S = g.S, TW = 1 << tws, TH = HALO_TB >> tws, PW = TW + S - 1, PP = (TH + R - 1) * PW;
    const int a0 = blockIdx.y * 64;
    const unsigned smem_base = lds_offset(smem);
    __amdgpu_buffer_rsrc_t rdy = make_rsrc(p.dy, (size_t)g.N * g.Ho * g.Wo * g.K * 2);
    __amdgpu_buffer_rsrc_t rx = make_rsrc(p.x, (size_t)g.N * g.H * g.W * g.C * 2);
    constexpr int NPI = HALO_PP / 8, NDI = HALO_TB / 8;   // copies (8 rows each) of the patch / of the dy slice

    auto issue_tile = [&](int tile, int buf) {
        const int n = tile / (tiles_x * tiles_y), trem = tile - n * (tiles_x * tiles_y), ty = trem / tiles_x, tx = trem - ty * tiles_x;
        const int p0 = ty * TH, q0 = tx * TW;
        const unsigned base = smem_base + buf * WH_BUF;
        for (int ii = wave; ii < NPI + NDI; ii += nwaves) {
            unsigned voff = OOR;
            if (ii < NPI) {   // patch rows 8*ii .. +7
                const int pp = ii * 8 + (lane >> 3), c = (lane & 7) ^ (seg_swz<64>(pp) << 2);
                const int pr = pp / PW, pc = pp - pr * PW, ih = p0 - g.ph + pr, iw = q0 - g.pw + pc;
                if (pp < PP && (unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W)
                    voff = (unsigned)(((n * g.H + ih) * g.W + iw) * 64 + c * 8) * 2u;
                dma16(rx, base + ii * 1024, voff);
            } else {          // dy rows (tile pixels) 8*d .. +7, c_out a0 .. a0+63
                const int d = ii - NPI, j = d * 8 + (lane >> 3), c = (lane & 7) ^ (seg_swz<64>(j) << 2);
                const int pr = p0 + (j >> tws), qc = q0 + (j & (TW - 1));
                if (pr < g.Ho && qc < g.Wo && a0 + c * 8 + 8 <= g.K)
                    voff = (unsigned)(((n * g.Ho + pr) * g.Wo + qc) * g.K + a0 + c * 8) * 2u;
                dma16(rdy, base + HALO_PP * 128 + d * 1024, voff);
            }
        }
    };

    f32x16 acc[2][2];   // [c_out half][c_in half]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // transpose-read lane roles: reduction row tl (+4 for the second read), operand columns cl .. cl+3
    const int i16 = lane & 15, tl = (lane >> 5) * 8 + (i16 >> 2), cl = ((lane >> 4) & 1) * 16 + (i16 & 3) * 4;
    // A block launched with one wave more than taps sums the bias gradient in that wave: it multiplies the dy^T fragments with
    // an all-ones operand (column 0 of the product = sum over the tile's pixels) and reads no x.  The waves sit 3-3-2-2 on the
    // four SIMDs instead of 3-2-2-2, and this wave issues half the matrix instructions of a tap wave: the block is no slower.
    const bool dbw = wave == R * S;
    const int tr = dbw ? 0 : wave / S, ts = dbw ? 0 : wave - tr * S;        // this wave's tap
    const int tapoff = tr * PW + ts;
    unsigned a_lane[2];   // dy: row tl of slice 0, column half i; later slices add 16 rows = 2048 bytes
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int col = i * 32 + cl;
        a_lane[i] = HALO_PP * 128 + tl * 128 + ((((col >> 5) ^ seg_swz<64>(tl)) << 6) | ((col & 31) << 1));
    }

    const TileWalk tw = tile_walk(tiles);
    int tile = tw.first;
    if (tile < tw.end) issue_tile(tile, 0);
    for (int it = 0; tile < tw.end; tile += tw.stride, ++it) {
        wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();   // tile `it` has landed everywhere; the other buffer is no longer read
        if (tile + tw.stride < tw.end) issue_tile(tile + tw.stride, (it + 1) & 1);
        const unsigned base = smem_base + (it & 1) * WH_BUF;
        // fragments are double-buffered in registers: the transpose reads of slice sl+1 are issued before the
        // matrix instructions of slice sl
        u32x2 alo[2][2], ahi[2][2], blo[2][2], bhi[2][2];
        auto read_slice = [&](int sl, int buf) {
            const int j = sl * 16 + tl;
            const int pp = (j >> tws) * PW + (j & (TW - 1)) + tapoff;
            const unsigned brow = base + pp * 128, bsw = seg_swz<64>(pp);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                alo[buf][i] = lds_read_tr<0>(base + a_lane[i] + sl * 2048);
                ahi[buf][i] = lds_read_tr<4 * 128>(base + a_lane[i] + sl * 2048);
            }
            if (dbw) return;   // wave-uniform
#pragma unroll
            for (int jf = 0; jf < 2; ++jf) {
                const int col = jf * 32 + cl;
                const unsigned addr = brow + ((((col >> 5) ^ bsw) << 6) | ((col & 31) << 1));
                blo[buf][jf] = lds_read_tr<0>(addr);
                bhi[buf][jf] = lds_read_tr<4 * 128>(addr);
            }
        };
        auto multiply = [&](int buf, bool newer_in_flight) {
            // reads of the next slice issued after this slice's: 8 for a tap wave, 4 for the bias-gradient wave
            if (!newer_in_flight) asm volatile("s_waitcnt lgkmcnt(0)");
            else if (dbw) asm volatile("s_waitcnt lgkmcnt(4)");
            else asm volatile("s_waitcnt lgkmcnt(8)");
            if (dbw) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    asm volatile("" : "+v"(alo[buf][i])); asm volatile("" : "+v"(ahi[buf][i]));
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const u32x4 av = {alo[buf][i].x, alo[buf][i].y, ahi[buf][i].x, ahi[buf][i].y};
                    acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), ones_bf16(), acc[i][0], 0, 0, 0);
                }
                return;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                asm volatile("" : "+v"(alo[buf][i])); asm volatile("" : "+v"(ahi[buf][i]));
                asm volatile("" : "+v"(blo[buf][i])); asm volatile("" : "+v"(bhi[buf][i]));
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int jf = 0; jf < 2; ++jf) {
                    const u32x4 av = {alo[buf][i].x, alo[buf][i].y, ahi[buf][i].x, ahi[buf][i].y};
                    const u32x4 bv = {blo[buf][jf].x, blo[buf][jf].y, bhi[buf][jf].x, bhi[buf][jf].y};
                    acc[i][jf] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv), acc[i][jf], 0, 0, 0);
                }
        };
        read_slice(0, 0);
        for (int sl = 0; sl < HALO_TB / 16; sl += 2) {
            read_slice(sl + 1, 1);
            multiply(0, true);
            if (sl + 2 < HALO_TB / 16) read_slice(sl + 2, 0);
            multiply(1, sl + 2 < HALO_TB / 16);
        }
    }
    if (dbw) {   // column 0 of the ones-product: this block's bias-gradient sums, one row of [blocks][c_out]
        if (p.dbp != nullptr)
#pragma unroll
            for (int i = 0; i < 2; ++i) store_db_fragment(acc[i][0], p.dbp + (size_t)blockIdx.x * p.rowsA, a0 + i * 32, p.rowsA, lane);
        return;
    }
    // partial[block][c_out][tap][c_in]; accumulator element v of lane l: row 8*(v/4) + 4*(l/32) + v%4, column l%32
    float *out = p.partial + (size_t)blockIdx.x * p.rowsA * p.rowsB;
    bool nan = false;   // among this lane's sums
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int jf = 0; jf < 2; ++jf)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int k = a0 + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                if (k < p.rowsA) out[(size_t)k * p.rowsB + wave * 64 + jf * 32 + (lane & 31)] = acc[i][jf][v];
                nan |= acc[i][jf][v] != acc[i][jf][v];
            }
    if (__builtin_expect(!nan, 1)) return;
    for (int j = 0; j < 16; ++j) {   // four rows of c_out each, in whole 8s
        const int row = a0 + (j >> 1) * 8 + 4 * (lane >> 5), col = (j & 1) * 32 + (lane & 31);
        float *o = out + (size_t)row * p.rowsB + wave * 64 + col;
        if (row >= p.rowsA || !(__builtin_isunordered(o[0], o[p.rowsB]) || __builtin_isunordered(o[2 * p.rowsB], o[3 * p.rowsB]))) continue;
        const f32x4 sum = sum_of_pairs(p, tiles_x, tiles_y, tiles, TH, TW, row, wave, col);
        o[0] = sum.x; o[p.rowsB] = sum.y; o[2 * p.rowsB] = sum.z; o[3 * p.rowsB] = sum.w;
    }
}

// ---------------------------------------------------------------------------------------
// The 3x3 form of the kernel above with all nine taps in ONE wave.  A block has eight waves, two per SIMD: wave (pg, kh, ch) takes rows
// 4 pg .. 4 pg + 3 of an 8 x 16 pixel tile, half kh of the 64 output channels and half ch of the input channels, for all nine taps
// (nine accumulator tiles, 144 registers).  A row of the tile is one 16-pixel slice, so the fragment of patch row y shifted by s
// serves the taps (r, s) of the rows y - r: 18 x fragments and four dy fragments for 36 matrix instructions, and every address is a
// base of three (one per s) and an immediate.  The reads of fragment i + 4 are issued before the matrix instructions of fragment i.
// Tiles come through four LDS buffers, three of them on their way; one barrier per tile.  The two row halves' sums meet in LDS once, at the
// end of the kernel.  The bias gradient (one small matrix instruction per row) rides in the ch = 0 waves.
// Patch layout: the pixel in column pc has its 64-byte segment sg at sg ^ ((pc >> 1) & 1).
// What bounds it: memory, 4.6 - 4.9 TB/s of tiles with their halo, and for few tiles the partials (38 MB for 64 x 64 channels).  With one wave per SIMD, two
// buffers of 16 x 16 pixels and a fragment read per tap it was the one tile in flight and the address arithmetic.  16 x 224 x 224, 64 -> 64 with its reduction, us
// back to back / with flushed caches: 84 / 96 -> 62 / 88; 28 x 206 x 209, 64 -> 256: 375 / 364 -> 312 / 305; 32 x 112 x 112, 64 -> 128: 75 / 81 -> 57 / 72.
// ---------------------------------------------------------------------------------------
constexpr int W9_TH = 8, W9_TW = 16, W9_PW = W9_TW + 2, W9_PP = (W9_TH + 2) * W9_PW, W9_SLOTS = 192;   // patch pixels, and those its copies fill
constexpr int W9_DY = W9_SLOTS * 128, W9_BUF = W9_DY + W9_TH * W9_TW * 128, W9_NB = 4, W9_CPW = W9_BUF / 1024 / 8;
static_assert(W9_PP <= W9_SLOTS && W9_CPW * 8 * 1024 == W9_BUF && W9_NB * W9_BUF <= 160 * 1024, "the copies divide evenly over the eight waves");
constexpr int W9_XCH = 4 * 9 * 4096;   // exchange: nine tiles of each of the four (kh, ch) pairs, then the bias gradient's
static_assert(W9_XCH + 2 * 64 * 16 <= W9_NB * W9_BUF, "the exchange fits the buffers");

template <int OFF> DEVFN void lds_write_f32x4(unsigned addr, f32x4 v) { asm volatile("ds_write_b128 %0, %1 offset:%2" ::"v"(addr), "v"(v), "n"(OFF) : "memory"); }

struct Halo9Arguments { KArgs p; int tiles_x, tiles_y, tiles; };   // the kernel's arguments as they lie in memory

template <bool DB>
__global__ __launch_bounds__(512, 2) void k_wgrad_halo9(const KArgs p, int tiles_x, int tiles_y, int tiles)
{
#if __HIP_DEVICE_COMPILE__   // the host pass only needs the launch stub
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const ConvGeom &g = p.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pg = wave >> 2, kh = (wave >> 1) & 1, ch = wave & 1;
    const int a0 = blockIdx.y * 64;
    const unsigned smem_base = lds_offset(smem);
    const __amdgpu_buffer_rsrc_t rdy = make_rsrc(p.dy, (size_t)g.N * g.Ho * g.Wo * g.K * 2), rx = make_rsrc(p.x, (size_t)g.N * g.H * g.W * 128);

    // Copies of a tile, eight pixels each: 24 of the patch (three per wave), 16 of the dy slice (two per wave).  What does not depend on the tile is
    // computed once: the byte offset relative to the tile's first pixel, and the pixel's row and column (past the patch, past the channels: row 0xffff).
    constexpr int NX = W9_SLOTS / 64;
    unsigned rel[W9_CPW], rc[W9_CPW];
#pragma unroll
    for (int c = 0; c < W9_CPW; ++c) {
        const int px = ((c < NX ? c : c - NX) * 8 + wave) * 8 + (lane >> 3);
        if (c < NX) {
            const int pr = px / W9_PW, pc = px - pr * W9_PW;
            rel[c] = (unsigned)(pr * g.W + pc) * 128u + ((unsigned)((lane & 7) ^ (((pc >> 1) & 1) << 2)) << 4);
            rc[c] = px < W9_PP ? (unsigned)(pr << 16 | pc) : 0xffff0000u;
        } else {
            const int pr = px / W9_TW, pc = px % W9_TW, k = a0 + ((lane & 7) ^ (((pc >> 1) & 1) << 2)) * 8;
            rel[c] = ((unsigned)(pr * g.Wo + pc) * (unsigned)g.K + k) * 2u;
            rc[c] = k + 8 <= g.K ? (unsigned)(pr << 16 | pc) : 0xffff0000u;
        }
    }
    // the patch origin may lie outside the image: the offset wraps, and wraps back for every pixel that passes the range checks
    struct Tile { int p0, q0; unsigned x, d; };
    auto place = [&](int t) {
        const int n = t / (tiles_x * tiles_y), rem = t - n * (tiles_x * tiles_y), ty = rem / tiles_x, p0 = ty * W9_TH, q0 = (rem - ty * tiles_x) * W9_TW;
        return Tile{p0, q0, (unsigned)((n * g.H + p0 - g.ph) * g.W + q0 - g.pw) * 128u, (unsigned)((n * g.Ho + p0) * g.Wo + q0) * (unsigned)g.K * 2u};
    };
    auto copy_one = [&](const Tile &t, int c, unsigned buf, bool on) {   // a tile past the last fetches nothing
        if (c < NX) {
            const int ih = t.p0 - g.ph + (int)(rc[c] >> 16), iw = t.q0 - g.pw + (int)(rc[c] & 0xffffu);
            const bool row = (unsigned)ih < (unsigned)(on ? g.H : 0), column = (unsigned)iw < (unsigned)g.W;
            dma16(rx, buf + (c * 8 + wave) * 1024, row & column ? t.x + rel[c] : OOR);
        } else {
            const bool row = t.p0 + (int)(rc[c] >> 16) < (on ? g.Ho : 0), column = t.q0 + (int)(rc[c] & 0xffffu) < g.Wo;
            dma16(rdy, buf + W9_DY + ((c - NX) * 8 + wave) * 1024, row & column ? t.d + rel[c] : OOR);
        }
    };

    const TileWalk tw = tile_walk(tiles);
    int tile = tw.first;
    for (int j = 0; j < W9_NB - 1; ++j) {
        const Tile t = place(tile + j * tw.stride);
#pragma unroll
        for (int c = 0; c < W9_CPW; ++c) copy_one(t, c, smem_base + j * W9_BUF, tile + j * tw.stride < tw.end);
    }

    f32x16 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
    f32x4 accdb = {0.f, 0.f, 0.f, 0.f};
    const bool do_db = DB && ch == 0;   // wave-uniform
    const bf16x8 selector = colsum_selector(lane);

    // transpose-read lane roles: reduction row tl (+4 for the second read), operand columns cl .. cl+3
    const int i16 = lane & 15, tl = (lane >> 5) * 8 + (i16 >> 2), cl = ((lane >> 4) & 1) * 16 + (i16 & 3) * 4;
    const unsigned dcol = smem_base + W9_DY + (pg * 4 * W9_TW + tl) * 128 + ((kh ^ ((tl >> 1) & 1)) << 6) + cl * 2;
    unsigned xcol[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) xcol[s] = smem_base + (pg * 4 * W9_PW + tl + s) * 128 + ((ch ^ (((tl + s) >> 1) & 1)) << 6) + cl * 2;

    for (int it = 0; tile < tw.end; tile += tw.stride, ++it) {
        wait_vmcnt<(W9_NB - 2) * W9_CPW>();
        __builtin_amdgcn_s_barrier();   // tile `it` has landed everywhere; the buffer of the tile before is no longer read
        const Tile ahead = place(tile + (W9_NB - 1) * tw.stride);
        const bool more = tile + (W9_NB - 1) * tw.stride < tw.end;
        const unsigned buf = it % W9_NB * W9_BUF, abuf = smem_base + (it + W9_NB - 1) % W9_NB * W9_BUF;
        unsigned xb[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) xb[s] = xcol[s] + buf;
        const unsigned db = dcol + buf;
        constexpr int DEPTH = 4;
        u32x2 xlo[DEPTH + 1], xhi[DEPTH + 1], dlo[4], dhi[4];
        // item i: the x fragment of patch row i / 3 (of this wave's six) shifted by i % 3; the dy fragment of row y comes with item 3 y
        auto read_item = [&](auto I) {
            constexpr int i = I, y = i / 3, s = i % 3;
            if constexpr (s == 0 && y < 4) { dlo[y] = lds_read_tr<y * W9_TW * 128>(db); dhi[y] = lds_read_tr<y * W9_TW * 128 + 512>(db); }
            xlo[i % (DEPTH + 1)] = lds_read_tr<y * W9_PW * 128>(xb[s]);
            xhi[i % (DEPTH + 1)] = lds_read_tr<y * W9_PW * 128 + 512>(xb[s]);
        };
        for_constant<DEPTH>([&](auto I) { read_item(I); });
        for_constant<18>([&](auto I) {
            constexpr int i = I, y = i / 3, s = i % 3, sl = i % (DEPTH + 1), last = i + DEPTH < 17 ? i + DEPTH : 17;
            // reads issued after item i's own: two per later item, two more where a row of dy begins
            constexpr int rows = (last < 9 ? last / 3 : 3) - (i < 9 ? i / 3 : 3);
            if constexpr (i + DEPTH < 18) read_item(std::integral_constant<int, i + DEPTH>{});
            asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(2 * (last - i) + 2 * rows));
            asm volatile("" : "+v"(xlo[sl])); asm volatile("" : "+v"(xhi[sl]));
            if constexpr (s == 0 && y < 4) { asm volatile("" : "+v"(dlo[y])); asm volatile("" : "+v"(dhi[y])); }
            const bf16x8 bv = __builtin_bit_cast(bf16x8, u32x4{xlo[sl].x, xlo[sl].y, xhi[sl].x, xhi[sl].y});
            for_constant<3>([&](auto R) {
                constexpr int r = R, q = y - r;
                if constexpr (q >= 0 && q < 4) {
                    const bf16x8 av = __builtin_bit_cast(bf16x8, u32x4{dlo[q].x, dlo[q].y, dhi[q].x, dhi[q].y});
                    acc[r * 3 + s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc[r * 3 + s], 0, 0, 0);
                    if constexpr (DB && r == 0 && s == 0)
                        if (do_db) accdb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, selector, accdb, 0, 0, 0);
                }
            });
            if constexpr (i % 3 == 1 && i / 3 < W9_CPW) copy_one(ahead, i / 3, abuf, more);
        });
    }
    // Wave pg = 0 finishes taps 0 - 4 and its partner pg = 1 taps 5 - 8; each leaves the other's tiles in LDS, sixteen values of a lane as four
    // vectors.  Accumulator element v of lane l: row 8*(v/4) + 4*(l/32) + v%4, column l%32.
    wait_vmcnt<0>();
    // The last matrix instructions have written their results before the stores below, which the compiler does not know, read them (at most 18 wait
    // states).  The sums are operands: no matrix instruction moves past this
    asm volatile("s_nop 15\n\ts_nop 15"
                 : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]), "+v"(acc[5]), "+v"(acc[6]), "+v"(acc[7]), "+v"(acc[8]), "+v"(accdb)::"memory");
    __syncthreads();
    const int pair = kh * 2 + ch;
    const unsigned xch = smem_base + pair * (9 * 4096) + lane * 16;
    const unsigned dxch = smem_base + W9_XCH + (kh * 64 + lane) * 16;
    for_constant<9>([&](auto T) {
        constexpr int t = T;
        if ((t < 5) != (pg == 0))
            for_constant<4>([&](auto V) {
                constexpr int v = V;
                lds_write_f32x4<t * 4096 + v * 1024>(xch, f32x4{acc[t][4 * v], acc[t][4 * v + 1], acc[t][4 * v + 2], acc[t][4 * v + 3]});
            });
    });
    if (do_db && pg == 1) lds_write_f32x4<0>(dxch, accdb);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();
    float *out = p.partial + ((size_t)blockIdx.x * p.rowsA + a0 + kh * 32) * 576 + ch * 32 + (lane & 31);
    bool nan = false;   // among this lane's sums
    auto finish = [&](auto T) {
        constexpr int t = T;
        u32x4 o[4];
        for_constant<4>([&](auto V) { o[V] = lds_read16<t * 4096 + V * 1024>(xch); });
        asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            asm volatile("" : "+v"(o[v]));
            const f32x4 of = __builtin_bit_cast(f32x4, o[v]);
            const float sums[4] = {acc[t][4 * v] + of.x, acc[t][4 * v + 1] + of.y, acc[t][4 * v + 2] + of.z, acc[t][4 * v + 3] + of.w};
            nan |= __builtin_isunordered(sums[0], sums[1]) | __builtin_isunordered(sums[2], sums[3]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = 8 * v + 4 * (lane >> 5) + e;
                if (a0 + kh * 32 + row < p.rowsA) out[(size_t)row * 576 + t * 64] = sums[e];
            }
        }
    };
    if (pg == 0) for_constant<5>([&](auto T) { finish(T); });
    else for_constant<4>([&](auto T) { finish(std::integral_constant<int, T + 5>{}); });
    if (do_db && pg == 0 && p.dbp != nullptr) {
        const f32x4 o = __builtin_bit_cast(f32x4, lds_read16<0>(dxch));
        asm volatile("s_waitcnt lgkmcnt(0)");
        u32x4 ov = __builtin_bit_cast(u32x4, o);
        asm volatile("" : "+v"(ov));
        store_colsum_fragment(accdb + __builtin_bit_cast(f32x4, ov), p.dbp + (size_t)blockIdx.x * p.rowsA, a0 + kh * 32, p.rowsA, lane);
    }
    if (__builtin_expect(!nan, 1)) return;
    // The arguments are read once more, and the sums from where they have been stored: kept for this, they would cost the loop registers
    const Halo9Arguments *args = (const Halo9Arguments *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const KArgs &pa = args->p;
    const int c = ch * 32 + (lane & 31);
    for (int t = pg == 0 ? 0 : 5; t < (pg == 0 ? 5 : 9); ++t)
        for (int row = blockIdx.y * 64 + kh * 32 + 4 * (lane >> 5), i = 0; i < 4 && row < pa.rowsA; ++i, row += 8) {   // c_out in whole 8s
            float *o = pa.partial + ((size_t)blockIdx.x * pa.rowsA + row) * 576 + t * 64 + c;
            if (!(__builtin_isunordered(o[0], o[576]) || __builtin_isunordered(o[2 * 576], o[3 * 576]))) continue;
            const f32x4 sum = sum_of_pairs(pa, args->tiles_x, args->tiles_y, args->tiles, W9_TH, W9_TW, row, t, c);
            o[0] = sum.x; o[576] = sum.y; o[2 * 576] = sum.z; o[3 * 576] = sum.w;
        }
#endif
}

// ---------------------------------------------------------------------------------------
// 3x3 (nine-tap) forward / backward-data with 64 reduction channels per tap, weights stationary in
// REGISTERS.  A block has four waves and a CU two blocks, so that two waves of different blocks share a
// SIMD and one multiplies while the other waits, converts or stores.  A wave keeps the fragments of 32
// output channels for all nine taps (36 fragments, 144 registers) and multiplies them with 64 of the
// tile's 128 pixels (8 x 16); nothing but the input patch goes through LDS and no barrier separates the
// taps.  Blocks are persistent (two per CU over all 64-channel tiles) and keep three patch buffers: while tile i
// is multiplied, the patches of tiles i+1 and i+2 are on their way.  A wave's results are reordered in its own
// share of the patch buffer that the tile has just left, and go out 64 bytes per pixel.  One barrier per tile.
// Patch layout: the pixel in column pc has its chunk c at position c ^ ((pc >> 1) & 7): sixteen pixels of a row are
// conflict-free, and a tap's row is an immediate offset.
// What bounds it: with one wave per SIMD holding all 64 channels (288 registers) every wait, conversion and store of the wave was the
// SIMD's; the LDS reads per matrix instruction have doubled and are still half of what LDS gives.  16 x 224 x 224, 64 -> 64 (us, back to back /
// with flushed caches): forward 76 / 84 -> 56 / 68, masked backward-data 89 / 112 -> 64 / 102 (without its loads and stores 46 and 42: the matrix
// instructions and LDS reads alone).  180 layers of 32 - 450 channels, 7 - 224 pixels: 0.95 - 1.4 times as fast as the best other.  Not where a block has little more
// than one or two tiles (price()), nor below 80 tiles, where the smallest window tile is (pixel_window_plan).  The 128-wide input-patch tiles take 1.2 - 1.9 times
// as long, but their price is too low and still keeps some layers of many tiles with them (15 x 221 x 214, 64 -> 128 forward).
// ---------------------------------------------------------------------------------------
// 128 reduction channels (RH = 2), us back to back / with flushed caches, the best other kernel -> this one: 32 x 112 x 112, 128 -> 128 forward 145 / 156 ->
// 107 / 115 (1.1 PFLOP/s), masked backward-data 159 / 170 -> 114 / 132; 64 <- 128 93 / 128 -> 59 / 75, at 8 samples 41 / 53 -> 23 / 30, at 2 12.7 / 16.7 -> 8.4 / 12.8.
// 240 passes: 1.06 - 1.27 times the best other in the middle from half a round of tiles on, 0.8 below a fifth (the weights are its fixed cost).
constexpr int WS_TH = 8, WS_TW = 16, WS_TB = WS_TH * WS_TW, WS_PW = WS_TW + 2, WS_PP = (WS_TH + 2) * WS_PW;
constexpr int WS_CPW = (WS_PP / 8 + 4) / 4;   // patch copies per wave, eight pixels each
constexpr int WS_PATCH = 4 * WS_CPW * 1024;   // 24 KiB per patch buffer
constexpr int WS_LDS = 3 * WS_PATCH + 64 * 4, WS_LDS2 = 6 * WS_PATCH + 64 * 4;   // one and two blocks of reduction channels
static_assert(WS_PP <= 4 * WS_CPW * 8 && 2 * WS_LDS <= 160 * 1024 && WS_LDS2 <= 160 * 1024 && 4096 + 2048 <= WS_CPW * 1024, "a patch fits its copies, two blocks a CU");
static_assert(3 * 8192 <= WS_PATCH && 64 * 64 <= WS_CPW * 1024, "three taps of weights, and a wave's results, fit a patch buffer");

// MASK (backward-data): fused backward of the ReLU in front of the layer.  RH: blocks of 64 reduction channels.  With two of them a block has eight waves and a
// CU one block: waves 4 - 7 hold the weights of the second 64 channels and multiply the same pixels; each wave hands the sums of one of its two pixel
// fragments to its partner through LDS (in the share of the patch buffer that the partner refills itself) and finishes the other.
#if __HIP_DEVICE_COMPILE__   // the host pass only needs the launch stubs
template <int PASS, bool MASK, int RH>
DEVFN void halo_ws(const KArgs &p, int tiles_x, int tiles_y, int tiles_all)
{
    constexpr int WS_DEPTH = MASK || RH > 1 ? 2 : 3;   // fragment reads run this many 16-channel slices ahead of the matrix cores
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const ConvGeom &g = p.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hc = wave & 1, pg = (wave >> 1) & 1, rh = RH > 1 ? wave >> 2 : 0, share = wave & 3;   // channel half, pixel group, reduction block
    constexpr int PATCH = RH * WS_PATCH, PB = RH * 128, NF = RH > 1 ? 1 : 2;   // bytes of a patch buffer and of a pixel; pixel fragments that a wave finishes
    const int a0 = blockIdx.y * 64;
    const int IH = PASS == PASS_FWD ? g.H : g.Ho, IW = PASS == PASS_FWD ? g.W : g.Wo;
    const int OH = PASS == PASS_FWD ? g.Ho : g.H, OW = PASS == PASS_FWD ? g.Wo : g.W;
    const int RSC = 9 * g.C;
    const unsigned smem_base = lds_offset(smem);
    float *bias_lds = reinterpret_cast<float *>(smem + 3 * PATCH);
    const __amdgpu_buffer_rsrc_t rin = PASS == PASS_FWD ? make_rsrc(p.x, (size_t)g.N * g.H * g.W * g.C * 2)
                                                        : make_rsrc(p.dy, (size_t)g.N * g.Ho * g.Wo * g.K * 2);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(p.w, (size_t)g.K * RSC * 2);
    const size_t out_bytes = (size_t)g.N * OH * OW * p.rowsA * 2;
    const __amdgpu_buffer_rsrc_t rout = make_rsrc(p.out, out_bytes), rx = make_rsrc(MASK ? (const void *)p.x : p.out, out_bytes);

    // weights, three taps at a time, on their way to registers.  Forward: step st is [64 c_out][64 c_in], chunk swizzle by row
    // pair; backward-data: step st (filter tap 8 - st) is [64 c_out][64 c_in] with c_out the reduction, read transposed
    auto issue_weights = [&](int part, int buf) {
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const int id = share * 6 + q, st = part * 3 + (id >> 3), row = (id & 7) * 8 + (lane >> 3);
            unsigned voff;
            if (PASS == PASS_FWD) {
                const int c = (lane & 7) ^ ((row >> 1) & 7);
                voff = a0 + row < p.rowsA ? ((unsigned)(a0 + row) * RSC + (st * RH + rh) * 64 + c * 8) * 2u : OOR;
            } else {
                const int c = (lane & 7) ^ (seg_swz<64>(row) << 2);
                voff = a0 + c * 8 < p.rowsA ? ((unsigned)(rh * 64 + row) * RSC + (8 - st) * g.C + a0 + c * 8) * 2u : OOR;
            }
            dma16(rw, smem_base + buf * PATCH + rh * WS_PATCH + id * 1024, voff);
        }
    };
    // patch copies: copy q of a wave fills patch pixels (wave * WS_CPW + q) * 8 .. + 7; the lane's pixel and chunk are fixed, the tile's origin
    // changes.  Past the patch the slots take its first pixels again.
    unsigned pk[WS_CPW];
#pragma unroll
    for (int q = 0; q < WS_CPW; ++q) {
        const int id = (share * WS_CPW + q) * 8 + (lane >> 3), pp = id < WS_PP ? id : lane >> 3, pr = pp / WS_PW, pc = pp - pr * WS_PW;
        pk[q] = (unsigned)pr | ((unsigned)pc << 8) | ((unsigned)((lane & 7) ^ ((pc >> 1) & 7)) << 20);
    }
    struct Tile { int n, h, w; };
    auto place = [&](int t) {
        const int n = t / (tiles_x * tiles_y), rem = t - n * (tiles_x * tiles_y), ty = rem / tiles_x;
        return Tile{n, ty * WS_TH, (rem - ty * tiles_x) * WS_TW};
    };
    auto copy_one = [&](const Tile &t, int q, unsigned dst, bool on) {   // a tile past the last fetches nothing
        const int h0 = PASS == PASS_FWD ? t.h - g.ph : t.h + g.ph - 2, w0 = PASS == PASS_FWD ? t.w - g.pw : t.w + g.pw - 2;
        unsigned v = pk[q];
        asm volatile("" : "+v"(v));   // stays packed in the loop
        const int pr = (int)(v & 255u), pc = (int)((v >> 8) & 255u);
        const bool row = (unsigned)(h0 + pr) < (unsigned)(on ? IH : 0), column = (unsigned)(w0 + pc) < (unsigned)IW;
        const unsigned at = (unsigned)((t.n * IH + h0) * IW + w0) * (unsigned)PB + (unsigned)(pr * IW + pc) * (unsigned)PB + rh * 128 + (v >> 16);
        dma16(rin, dst + rh * WS_PATCH + (share * WS_CPW + q) * 1024, row & column ? at : OOR);
    };

    const TileWalk tw = tile_walk(tiles_all);
    int tile = tw.first;
    const int stride = tw.stride, tiles = tw.end;   // this block's tiles: tile, tile + stride, ... below `tiles`
    Tile now = place(tile), next = place(tile + stride);
    issue_weights(0, 1);
    issue_weights(1, 2);
#pragma unroll
    for (int q = 0; q < WS_CPW; ++q) copy_one(now, q, smem_base, tile < tiles);
    if (tid < 64) bias_lds[tid] = (PASS == PASS_FWD && (p.flags & KF_BIAS) && a0 + tid < p.rowsA) ? p.bias[a0 + tid] : 0.f;

    u32x4 afr[9][4];   // [step][16-channel slice]
    unsigned wad[4];   // this lane's weights of slice k of a step
    if (PASS == PASS_FWD) {
        const int row = hc * 32 + (lane & 31);
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) wad[ks] = smem_base + PATCH + rh * WS_PATCH + row * 128 + (((2 * ks + (lane >> 5)) ^ ((row >> 1) & 7)) << 4);
    } else {
        const int i16 = lane & 15, t = (lane >> 5) * 8 + (i16 >> 2), cl = ((lane >> 4) & 1) * 16 + (i16 & 3) * 4;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) wad[ks] = smem_base + PATCH + rh * WS_PATCH + (ks * 16 + t) * 128 + ((hc ^ seg_swz<64>(t)) << 6) + cl * 2;
    }
    for_constant<3>([&](auto PART) {
        constexpr int part = PART;
        constexpr unsigned buf = part == 1 ? PATCH : 0;
        if (part == 2) wait_vmcnt<0>();
        else wait_vmcnt<6 + WS_CPW>();   // younger: the next part and the first patch
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        for_constant<3>([&](auto J) {
            constexpr int st = part * 3 + J, off = J * 8192;
            u32x2 lo[4], hi[4];
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                if constexpr (PASS == PASS_FWD) afr[st][ks] = lds_read16<off>(wad[ks] + buf);
                else { lo[ks] = lds_read_tr<off>(wad[ks] + buf); hi[ks] = lds_read_tr<off + 512>(wad[ks] + buf); }
            }
            asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                if constexpr (PASS == PASS_FWD) asm volatile("" : "+v"(afr[st][ks]));
                else {
                    asm volatile("" : "+v"(lo[ks]));
                    asm volatile("" : "+v"(hi[ks]));
                    afr[st][ks] = u32x4{lo[ks].x, lo[ks].y, hi[ks].x, hi[ks].y};
                }
            }
        });
        if (part != 1) __builtin_amdgcn_s_barrier();   // everyone has read the buffer that is filled next
        if (part == 0) issue_weights(2, 1);
    });
#pragma unroll
    for (int q = 0; q < WS_CPW; ++q) copy_one(next, q, smem_base + PATCH, tile + stride < tiles);

    // this lane's pixel of fragment 0 in column tap s, slice 0; slices differ in two bits, rows and fragments by immediates
    unsigned col[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        const int pc = (lane & 15) + s, pr = pg * 4 + 2 * rh + ((lane >> 4) & 1);   // with two reduction blocks fragment 0 is the one this wave finishes
        col[s] = smem_base + rh * WS_PATCH + (pr * WS_PW + pc) * 128 + (((lane >> 5) ^ ((pc >> 1) & 7)) << 4);
    }
    // results: written by pixel fragment, read back four lanes to a pixel
    const unsigned own = smem_base + rh * WS_PATCH + share * WS_CPW * 1024, stg = own + (RH > 1 ? 4096 : 0);
    const unsigned give = smem_base + (1 - rh) * WS_PATCH + share * WS_CPW * 1024;               // the partner's share
    const unsigned other = rh == 0 ? 2 * WS_PW * 128 : 0u - 2 * WS_PW * 128;                    // bytes from fragment 0 to fragment 1
    const int wpx = lane & 31, rpx = lane >> 2;
    const unsigned stw = stg + wpx * 64 + ((((lane >> 5)) ^ ((wpx >> 2) & 3)) << 4), str = stg + rpx * 64 + (((lane & 3) ^ ((rpx >> 2) & 3)) << 4);
    const int och = a0 + hc * 32 + (lane & 3) * 8;
    const unsigned bad = lds_offset(bias_lds) + (hc * 32 + 4 * (lane >> 5)) * 4;

    for (int it = 0; tile < tiles; tile += stride, ++it) {
        const unsigned base = (it % 3) * PATCH, nbuf = smem_base + ((it + 2) % 3) * PATCH;   // which tile it - 1 left before the last barrier
        const Tile after = place(tile + 2 * stride);
        const bool more = tile + 2 * stride < tiles;
        // this lane's output vectors: row pg * 4 + i of the tile, pixel lane / 4
        const int orow = now.h + pg * 4 + 2 * rh;
        unsigned voff = now.w + rpx < OW && och < p.rowsA ? ((unsigned)((now.n * OH + orow) * OW + now.w + rpx) * (unsigned)p.rowsA + och) * 2u : OOR;
        auto at = [&](int i) { return orow + i < OH && voff != OOR ? voff + (unsigned)(i * OW) * (unsigned)p.rowsA * 2u : OOR; };
        constexpr int NV = 2 * NF;   // output vectors
        u32x4 mk[NV];
        if constexpr (MASK) {
#pragma unroll
            for (int i = 0; i < NV; ++i) mk[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, at(i), 0, 0);
            asm volatile("" : "+v"(voff));   // the four offsets are made again for the stores
        }
        unsigned cb[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) cb[s] = col[s] + base;
        f32x16 acc[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
        u32x4 fb[WS_DEPTH + 1][2];   // [buffer][pixel fragment]
        auto read_b = [&](auto SL) {
            constexpr int st = SL / 4, ks = SL % 4, off = st / 3 * WS_PW * 128;
            const unsigned ad = cb[st % 3] ^ (unsigned)(ks << 5);
            fb[SL % (WS_DEPTH + 1)][0] = lds_read16<off>(ad);
            if constexpr (RH > 1) fb[SL % (WS_DEPTH + 1)][1] = lds_read16<off>((cb[st % 3] + other) ^ (unsigned)(ks << 5));
            else fb[SL % (WS_DEPTH + 1)][1] = lds_read16<off + 2 * WS_PW * 128>(ad);
        };
        for_constant<WS_DEPTH>([&](auto SL) { read_b(SL); });
        for_constant<36>([&](auto SL) {
            constexpr int sl = SL, cur = sl % (WS_DEPTH + 1), newer = 2 * (35 - sl < WS_DEPTH ? 35 - sl : WS_DEPTH);   // reads issued after this slice's
            if constexpr (sl + WS_DEPTH < 36) read_b(std::integral_constant<int, sl + WS_DEPTH>{});
            asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(newer));
            asm volatile("" : "+v"(fb[cur][0]));
            asm volatile("" : "+v"(fb[cur][1]));
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, afr[sl / 4][sl % 4]), __builtin_bit_cast(bf16x8, fb[cur][j]), acc[j], 0, 0, 0);
            if constexpr (sl % 4 == 1 && sl / 4 < WS_CPW) copy_one(after, sl / 4, nbuf, more);
        });
        // of the loads after this wave's share of the next patch only the copies above may be outstanding
        wait_vmcnt<WS_CPW>();
        __builtin_amdgcn_s_barrier();   // all shares of the next patch have landed; this tile's buffer has been read
        if constexpr (RH > 1) {
            unsigned l16 = lane * 16;
            asm volatile("" : "+v"(l16));   // made here, not kept
            // the last matrix instruction has written its result before the stores below, which the compiler does not know, read it (at most 18 wait states)
            asm volatile("s_nop 15\n\ts_nop 15" : "+v"(acc[1]));
            const unsigned to = give + base + l16;
            for_constant<4>([&](auto V) {
                constexpr int v = V;
                lds_write16(to + v * 1024, __builtin_bit_cast(u32x4, f32x4{acc[1][4 * v], acc[1][4 * v + 1], acc[1][4 * v + 2], acc[1][4 * v + 3]}));
            });
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            u32x4 got[4];
            for_constant<4>([&](auto V) { got[V] = lds_read16<V * 1024>(own + base + l16); });
            asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                asm volatile("" : "+v"(got[v]));
                const f32x4 o = __builtin_bit_cast(f32x4, got[v]);
                acc[0][4 * v] += o.x; acc[0][4 * v + 1] += o.y; acc[0][4 * v + 2] += o.z; acc[0][4 * v + 3] += o.w;
            }
        }
        f32x4 bv[4];
        if constexpr (PASS == PASS_FWD) {
            bv[0] = __builtin_bit_cast(f32x4, lds_read16<0>(bad)); bv[1] = __builtin_bit_cast(f32x4, lds_read16<32>(bad));
            bv[2] = __builtin_bit_cast(f32x4, lds_read16<64>(bad)); bv[3] = __builtin_bit_cast(f32x4, lds_read16<96>(bad));
            asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
            for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(bv[k]));
        }
        // accumulator element v of lane l is channel 8*(v/4) + 4*(l/32) + v%4 of pixel l%32 of fragment j; the lanes l and
        // l+32 swap halves of two channel groups, after which each holds 8 consecutive channels of one group
#pragma unroll
        for (int j = 0; j < NF; ++j)
#pragma unroll
            for (int gp = 0; gp < 2; ++gp) {
                unsigned pkd[2][2];   // [group 2gp, 2gp+1][channel pair]
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int gq = 2 * gp + e;
                    float v0 = acc[j][4 * gq], v1 = acc[j][4 * gq + 1], v2 = acc[j][4 * gq + 2], v3 = acc[j][4 * gq + 3];
                    if constexpr (PASS == PASS_FWD) {
                        v0 += bv[gq].x; v1 += bv[gq].y; v2 += bv[gq].z; v3 += bv[gq].w;
                        if (p.flags & KF_RELU) { v0 = fmaxf(v0, 0.f); v1 = fmaxf(v1, 0.f); v2 = fmaxf(v2, 0.f); v3 = fmaxf(v3, 0.f); }
                    }
                    pkd[e][0] = pack_bf16(v0, v1);
                    pkd[e][1] = pack_bf16(v2, v3);
                }
                const auto s0 = __builtin_amdgcn_permlane32_swap(pkd[0][0], pkd[1][0], false, false);
                const auto s1 = __builtin_amdgcn_permlane32_swap(pkd[0][1], pkd[1][1], false, false);
                // chunk 2 gp + lane / 32 of pixel j * 32 + lane % 32; (pixel >> 2) & 3 is the same for both fragments
                lds_write16((stw ^ (unsigned)(gp << 5)) + base + j * 2048, u32x4{s0[0], s1[0], s0[1], s1[1]});
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        u32x4 o[NV];
        for_constant<NV>([&](auto I) { o[I] = lds_read16<I * 1024>(str + base); });
        asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            asm volatile("" : "+v"(o[i]));
            if constexpr (MASK) o[i] = apply_mask(o[i], mk[i]);
            __builtin_amdgcn_raw_buffer_store_b128(o[i], rout, at(i), 0, 0);
        }
        now = next;
        next = after;
    }
}
#endif
template <int PASS, bool MASK = false>
__global__ __launch_bounds__(256, 2) void k_halo_ws(const KArgs p, int tiles_x, int tiles_y, int tiles_all)
{
#if __HIP_DEVICE_COMPILE__
    halo_ws<PASS, MASK, 1>(p, tiles_x, tiles_y, tiles_all);
#endif
}
template <int PASS, bool MASK, int RH>
__global__ __launch_bounds__(256 * RH, 2) void k_halo_ws(const KArgs p, int tiles_x, int tiles_y, int tiles_all)
{
#if __HIP_DEVICE_COMPILE__
    halo_ws<PASS, MASK, RH>(p, tiles_x, tiles_y, tiles_all);
#endif
}

struct HaloVariant { int TA, WA, WB, NS; };
const HaloVariant kHalo[] = {{64, 1, 4, 2}, {128, 2, 2, 2}, {64, 1, 4, 3}, {64, 1, 4, 4}};
constexpr int kNumHalo = 4;
typedef void (*HaloFn)(const KArgs, int, int, int);
HaloFn pick_halo(int pass, int v)
{
    if (pass == PASS_FWD) {
        switch (v) {
        case 1: return k_halo<PASS_FWD, 128, 2, 2, 2>;
        case 2: return k_halo<PASS_FWD, 64, 1, 4, 3>;
        case 3: return k_halo<PASS_FWD, 64, 1, 4, 4>;
        default: return k_halo<PASS_FWD, 64, 1, 4, 2>;
        }
    }
    switch (v) {
    case 1: return k_halo<PASS_DGRAD, 128, 2, 2, 2>;
    case 2: return k_halo<PASS_DGRAD, 64, 1, 4, 3>;
    case 3: return k_halo<PASS_DGRAD, 64, 1, 4, 4>;
    default: return k_halo<PASS_DGRAD, 64, 1, 4, 2>;
    }
}
size_t halo_lds_bytes(const HaloVariant &h)
{
    const int nw = h.WA * h.WB;
    const size_t ip = (HALO_PP * 128 / 1024 + nw - 1) / nw;
    const size_t stages = ip * nw * 1024 + (size_t)h.NS * h.TA * 128, epi = (size_t)HALO_TB * (h.TA + 8) * 2;
    return (stages > epi ? stages : epi) + (size_t)h.TA * 4;
}
// tile shape with the least padded area: 8 x 32 (tws 5) or 16 x 16 (tws 4) output pixels
int halo_tws(int oh, int ow)
{
    const long long a5 = (long long)((oh + 7) / 8 * 8) * ((ow + 31) / 32 * 32), a4 = (long long)((oh + 15) / 16 * 16) * ((ow + 15) / 16 * 16);
    return a4 < a5 ? 4 : 5;
}

}  // namespace

hipError_t halo_init()
{
    {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_wgrad_halo), hipFuncAttributeMaxDynamicSharedMemorySize, 2 * WH_BUF);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_wgrad_halo9<true>), hipFuncAttributeMaxDynamicSharedMemorySize, W9_NB * W9_BUF);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_wgrad_halo9<false>), hipFuncAttributeMaxDynamicSharedMemorySize, W9_NB * W9_BUF);
        if (e != hipSuccess) return e;
    }
    {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_halo_ws<PASS_FWD>), hipFuncAttributeMaxDynamicSharedMemorySize, WS_LDS);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(k_halo_ws<PASS_DGRAD>), hipFuncAttributeMaxDynamicSharedMemorySize, WS_LDS);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_halo_ws<PASS_DGRAD, true>), hipFuncAttributeMaxDynamicSharedMemorySize, WS_LDS);
        for (const void *f : {reinterpret_cast<const void *>(&k_halo_ws<PASS_FWD, false, 2>), reinterpret_cast<const void *>(&k_halo_ws<PASS_DGRAD, false, 2>),
                              reinterpret_cast<const void *>(&k_halo_ws<PASS_DGRAD, true, 2>)})
            if (e == hipSuccess) e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, WS_LDS2);
        if (e != hipSuccess) return e;
    }
    for (int pass = 0; pass < 2; ++pass)
        for (int v = 0; v < kNumHalo; ++v) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(pick_halo(pass, v)), hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)halo_lds_bytes(kHalo[v]));
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

// variant override 400 + v; forward needs c_in == 64, backward-data c_out == 64 (405: 128); stride 1; no reduction split
bool halo_plan(const ConvGeom &g, int pass, int force_variant, int force_splits, GemmPlan *pl)
{
    if (pass == PASS_WGRAD) {   // 410: input-patch filter gradient, a wave per tap; 411: 3x3, all taps per wave; force_splits = number of persistent blocks
        if ((force_variant != 410 && force_variant != 411) || g.sh != 1 || g.sw != 1 || g.C != 64 || (g.K % 8) != 0 || g.R * g.S > 16) return false;
        if (force_variant == 411 && (g.R != 3 || g.S != 3)) return false;
        const bool nine = force_variant == 411;
        const int tws = halo_tws(g.Ho, g.Wo), tw = nine ? W9_TW : 1 << tws, th = nine ? W9_TH : HALO_TB >> tws, tb = tw * th;
        if (!nine && (th + g.R - 1) * (tw + g.S - 1) > HALO_PP) return false;
        const long long tiles = (long long)g.N * ((g.Ho + th - 1) / th) * ((g.Wo + tw - 1) / tw);
        const int ktiles = (g.K + 63) / 64;
        int blocks = force_splits > 1 ? force_splits : 256 / ktiles;   // default: one persistent block per CU
        if (blocks > tiles) blocks = (int)tiles;
        if (blocks < 2) return false;   // the split-reduce kernel writes the result
        pl->variant = force_variant - 400;
        pl->db_wave = nine || g.R * g.S <= 15;   // 16 waves per block at most; the nine-tap kernel sums it in its own waves
        pl->fast = true; pl->dma = true; pl->halo = true;
        pl->TA = 64; pl->TB = 64 * g.R * g.S; pl->BK = 16; pl->vecA = pl->vecB = true;
        pl->tilesA = ktiles; pl->tilesB = 1;
        pl->steps_total = (int)tiles * (tb / 16);
        pl->steps_per_split = (int)((tiles + blocks - 1) / blocks) * (tb / 16);
        pl->splits = blocks;
        return true;
    }
    if (pass != PASS_FWD && pass != PASS_DGRAD) return false;
    pl->blocks = 0;
    if (force_variant == 404 || force_variant == 405) {   // weights in registers, persistent blocks; force_splits = blocks per 64-row tile; 405: 128 reduction channels
        const int red_c = pass == PASS_FWD ? g.C : g.K, rowsA = pass == PASS_FWD ? g.K : g.C;
        if (g.sh != 1 || g.sw != 1 || g.R != 3 || g.S != 3 || red_c != (force_variant == 404 ? 64 : 128) || (rowsA % 8) != 0) return false;
        if (pass == PASS_DGRAD && (g.ph > 2 || g.pw > 2)) return false;
        const int oh = pass == PASS_FWD ? g.Ho : g.H, ow = pass == PASS_FWD ? g.Wo : g.W;
        const long long tiles = (long long)g.N * ((oh + WS_TH - 1) / WS_TH) * ((ow + WS_TW - 1) / WS_TW);
        if (tiles > 0x7fffff) return false;
        pl->variant = force_variant - 400;
        pl->fast = true; pl->dma = true; pl->halo = true;
        pl->TA = 64; pl->TB = WS_TB; pl->BK = 64; pl->vecA = pl->vecB = true;
        pl->tilesA = (rowsA + 63) / 64;
        pl->tilesB = (int)tiles;
        pl->steps_total = pl->steps_per_split = red_c / 64 * 9;
        pl->splits = 1;
        pl->blocks = force_splits > 1 ? force_splits : 0;
        return true;
    }
    if (force_variant < 400 || force_variant >= 400 + kNumHalo || force_splits > 1) return false;
    if (g.sh != 1 || g.sw != 1 || g.R * g.S > 32) return false;
    const int red_c = pass == PASS_FWD ? g.C : g.K, rowsA = pass == PASS_FWD ? g.K : g.C;
    if (red_c != 64 || (rowsA % 8) != 0) return false;
    if (pass == PASS_DGRAD && (g.ph > g.R - 1 || g.pw > g.S - 1)) return false;
    const int oh = pass == PASS_FWD ? g.Ho : g.H, ow = pass == PASS_FWD ? g.Wo : g.W;
    const int tws = halo_tws(oh, ow), tw = 1 << tws, th = HALO_TB >> tws;
    if ((th + g.R - 1) * (tw + g.S - 1) > HALO_PP) return false;
    const HaloVariant &h = kHalo[force_variant - 400];
    pl->variant = force_variant - 400;
    pl->fast = true; pl->dma = true; pl->halo = true;
    pl->TA = h.TA; pl->TB = HALO_TB; pl->BK = 64; pl->vecA = pl->vecB = true;
    pl->tilesA = (rowsA + h.TA - 1) / h.TA;
    pl->tilesB = g.N * ((oh + th - 1) / th) * ((ow + tw - 1) / tw);
    pl->steps_total = pl->steps_per_split = g.R * g.S;
    pl->splits = 1;
    return true;
}

void halo_kernel_name(int pass, const GemmPlan &pl, bool masked, char *name, size_t name_bytes)
{
    if (pass == PASS_WGRAD) { snprintf(name, name_bytes, pl.variant == 11 ? "k_wgrad_halo9<true>" : "k_wgrad_halo"); return; }
    if (pl.variant == 4 || pl.variant == 5) {
        snprintf(name, name_bytes, pl.variant == 4 ? "k_halo_ws<%d, %s>" : "k_halo_ws<%d, %s, 2>", pass, pass == PASS_DGRAD && masked ? "true" : "false");
        return;
    }
    const HaloVariant &h = kHalo[pl.variant];
    snprintf(name, name_bytes, "k_halo<%d, %d, %d, %d, %d>", pass, h.TA, h.WA, h.WB, h.NS);
}

hipError_t halo_launch(const ConvArgs &a, hipStream_t st)
{
    KArgs p;
    p.g = a.g;
    if (a.pass == PASS_WGRAD) {
        const ConvGeom &g = a.g;
        p.rowsA = g.K; p.rowsB = g.R * g.S * g.C; p.red = g.N * g.Ho * g.Wo;
        p.tilesA = a.plan.tilesA; p.tilesB = 1; p.steps_total = a.plan.steps_total; p.steps_per_split = a.plan.steps_per_split;
        p.splits = a.plan.splits; p.flags = a.flags;
        p.x = a.x; p.w = nullptr; p.dy = a.dy; p.ymask = nullptr; p.bias = nullptr; p.out = a.out; p.partial = a.partial;
        // the bias gradient, when asked for, is summed by one extra wave per block; its [blocks][c_out] rows are added up by the split-reduce
        const bool db = (a.flags & KF_DB) && a.plan.db_wave && a.db_partial != nullptr && a.db_out != nullptr;
        p.dbp = db ? a.db_partial : nullptr;
        if (!db) p.flags &= ~KF_DB;
        const int tws = halo_tws(g.Ho, g.Wo), tw = 1 << tws, th = HALO_TB >> tws;
        const int tiles_x = (g.Wo + tw - 1) / tw, tiles_y = (g.Ho + th - 1) / th;
        if (a.plan.variant == 11) {
            void (*kern)(const KArgs, int, int, int) = k_wgrad_halo9<false>;
            if (db) kern = k_wgrad_halo9<true>;
            const int nx = (g.Wo + W9_TW - 1) / W9_TW, ny = (g.Ho + W9_TH - 1) / W9_TH;
            hipLaunchKernelGGL(kern, dim3((unsigned)a.plan.splits, (unsigned)a.plan.tilesA), dim3(512), W9_NB * W9_BUF, st, p, nx, ny, g.N * nx * ny);
        } else
            hipLaunchKernelGGL(k_wgrad_halo, dim3((unsigned)a.plan.splits, (unsigned)a.plan.tilesA), dim3(64 * (g.R * g.S + (db ? 1 : 0))), 2 * WH_BUF, st, p, tws,
                               tiles_x, tiles_y, g.N * tiles_x * tiles_y);
        dp_trace_main_kernel_done(st);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_split_reduce(a, p.rowsA, p.rowsB, st, db);
    }
    const bool fwd = a.pass == PASS_FWD;
    p.rowsA = fwd ? a.g.K : a.g.C;
    p.rowsB = fwd ? a.g.N * a.g.Ho * a.g.Wo : a.g.N * a.g.H * a.g.W;
    p.red = a.g.R * a.g.S * (fwd ? a.g.C : a.g.K);
    p.tilesA = a.plan.tilesA; p.tilesB = a.plan.tilesB;
    p.steps_total = a.plan.steps_total; p.steps_per_split = a.plan.steps_per_split; p.splits = 1;
    p.flags = a.flags;
    p.x = a.x; p.w = a.w; p.dy = a.dy; p.ymask = nullptr; p.bias = a.bias; p.out = a.out; p.partial = a.partial;
    const int oh = fwd ? a.g.Ho : a.g.H, ow = fwd ? a.g.Wo : a.g.W;
    if (a.plan.variant == 4 || a.plan.variant == 5) {
        const bool two = a.plan.variant == 5;
        int blocks = a.plan.blocks > 0 ? a.plan.blocks : (two ? 256 : 512) / p.tilesA;   // default: two persistent blocks per CU, one of eight waves
        if (blocks < 1) blocks = 1;
        if (blocks > p.tilesB) blocks = p.tilesB;
        void (*kern)(const KArgs, int, int, int) = k_halo_ws<PASS_FWD>;
        if (two) kern = k_halo_ws<PASS_FWD, false, 2>;
        if (!fwd) {
            const bool masked = (p.flags & KF_MASK_IN) != 0;
            if (two) { kern = k_halo_ws<PASS_DGRAD, false, 2>; if (masked) kern = k_halo_ws<PASS_DGRAD, true, 2>; }
            else { kern = k_halo_ws<PASS_DGRAD>; if (masked) kern = k_halo_ws<PASS_DGRAD, true>; }
        }
        hipLaunchKernelGGL(kern, dim3((unsigned)blocks, (unsigned)p.tilesA), dim3(two ? 512 : 256), two ? WS_LDS2 : WS_LDS, st, p,
                           (ow + WS_TW - 1) / WS_TW, (oh + WS_TH - 1) / WS_TH, p.tilesB);
        dp_trace_main_kernel_done(st);
        return hipGetLastError();
    }
    const int tws = halo_tws(oh, ow), tw = 1 << tws, th = HALO_TB >> tws;
    const int tiles_x = (ow + tw - 1) / tw, tiles_y = (oh + th - 1) / th;
    const HaloVariant &h = kHalo[a.plan.variant];
    dim3 grid((unsigned)(p.tilesA * p.tilesB), 1, 1), block(64 * h.WA * h.WB, 1, 1);
    hipLaunchKernelGGL(pick_halo(a.pass, a.plan.variant), grid, block, halo_lds_bytes(h), st, p, tws, tiles_x, tiles_y);
    dp_trace_main_kernel_done(st);
    return hipGetLastError();
}
