// fp32 convolutions, the reference-precision path: every product and sum in fp32, on the fp32 matrix instruction
// v_mfma_f32_16x16x4_f32 (exact fp32 operands, fp32 accumulation).
//
// The layers that run here are small (tens of channels, a few thousand pixels): what bounds them is latency, one chain of
// dependent loads and sums per output, and the number of launches.  So nothing is staged: a wave owns a 16 x 16 (or 16 x 64)
// output tile, loads its operands from the caches straight into registers, several reduction steps ahead, and the waves of a
// block share the tile's reduction; their sums meet in LDS in wave order.  A lane of the matrix instruction supplies one
// reduction element per operand (row l % 16, element l / 16); which element of the tensors that is does not matter as long as both
// operands agree, so a step takes 16 consecutive reduction channels and lane group g the channels 4g .. 4g+3 of them: one 16-byte
// load per lane and operand feeds four instructions.
// Measured against one thread per output (forward, backward-data) and one wave per filter element, 3x3 layers, forward + backward-data
// + both gradients back to back, in a graph: 2 x 16 x 16 x 16 -> 16: 63.5 -> 14.6 us (5.0 / 5.6 / 7.2 alone);
// 3 x 38 x 38 x 15 -> 34: 180 -> 52 us (9.2 / 12.4 / 33.4); 4 x 40 x 40 x 64 -> 64: 2603 -> 93 us (21 / 28 / 46).
#include "tile_common.h"
#include <algorithm>
#include <cstdio>
#include <type_traits>

namespace {

// n / d for 0 <= n < 2^31 by one multiplication (d >= 1 fixed per launch): the reciprocal rounded up (Granlund and Montgomery,
// "Division by invariant integers using multiplication", 1994)
struct FastDiv {
    unsigned mul, shift, d;
    __host__ __device__ static FastDiv of(int dv)
    {
        FastDiv f{0u, 0u, (unsigned)dv};
        if (dv > 1) {
            unsigned lg = 0;
            while ((1ull << lg) < (unsigned long long)dv) ++lg;   // 2^lg >= d > 2^(lg-1)
            f.shift = lg - 1;
            f.mul = (unsigned)(((1ull << (31 + lg)) + (unsigned)dv - 1) / (unsigned)dv);
        }
        return f;
    }
    __device__ __forceinline__ int div(int n) const { return d == 1 ? n : (int)(__umulhi((unsigned)n, mul) >> shift); }
};

struct F32Args {
    ConvGeom g;
    FastDiv plane, row, sh, sw, tap, cblk;   // pixels per image and per row of the pass's pixel grid, strides, filter columns, 16-channel blocks
    int rowsA, rowsB, red;             // output channels of the pass, pixels, reduction channels
    int tile0;                         // first tile of this launch
    unsigned flags;
    const float *w, *b, *mask;         // weights, pixel operand (x or dy), saved output that masks dy
    const float *bias, *xin;
    float *out;
};

// four consecutive floats of which `valid` exist; a load that does not exist reads `safe` (any valid address)
template <bool V4> DEVFN f32x4 load4(const float *p, const float *safe, int valid)
{
    f32x4 v;
    if constexpr (V4) {   // the tensors' channel counts are multiples of 4: all or nothing, 16-byte aligned
        v = *reinterpret_cast<const f32x4 *>(valid > 0 ? p : safe);
        if (valid <= 0) v = f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) { const float t = *(valid > e ? p + e : safe); v[e] = valid > e ? t : 0.f; }
    }
    return v;
}

// One output from the taps that reach it, one after the other: what a tile's product does not give when a weight is infinite or NaN.  A tap
// outside the image (or off the stride grid) supplies a zero to the matrix instruction, and zero times infinity is NaN.  Costs what a
// plain loop costs, and only where the product is NaN.
template <bool DG, bool MASK> DEVFN float sum_of_reached_taps(const F32Args &p, int pix, int ch)
{
    const ConvGeom &g = p.g;
    const int n = p.plane.div(pix), rem = pix - n * (int)p.plane.d, pr = p.row.div(rem), pc = rem - pr * (int)p.row.d;
    const int Hl = DG ? g.Ho : g.H, Wl = DG ? g.Wo : g.W;
    float s = 0.f;
    for (int r = 0; r < g.R; ++r)
        for (int t = 0; t < g.S; ++t) {
            int hh = DG ? pr + g.ph - r : pr * g.sh - g.ph + r, ww = DG ? pc + g.pw - t : pc * g.sw - g.pw + t;
            if constexpr (DG) {
                if (hh < 0 || ww < 0) continue;
                const int hq = p.sh.div(hh), wq = p.sw.div(ww);
                if (hq * g.sh != hh || wq * g.sw != ww) continue;
                hh = hq; ww = wq;
            }
            if ((unsigned)hh >= (unsigned)Hl || (unsigned)ww >= (unsigned)Wl) continue;
            const size_t o = (((size_t)n * Hl + hh) * Wl + ww) * p.red;
            const int tap = r * g.S + t;
            for (int c = 0; c < p.red; ++c) {
                float b = p.b[o + c];
                if constexpr (MASK) b = p.mask[o + c] > 0.f ? b : 0.f;
                s = fmaf(b, p.w[DG ? ((size_t)c * g.R * g.S + tap) * g.C + ch : ((size_t)ch * g.R * g.S + tap) * g.C + c], s);
            }
        }
    return s;
}

// Forward and backward-data: D[channel][pixel] = sum over (tap, reduction channel).  DG: backward-data (pixel operand dy, filter
// taps addressed through the stride); MASK: dy counts where the saved output is > 0.  Everything that decides which loads
// happen is a template parameter or an address select: a branch in the loop body would make every load wait for the one before.  J: pixel fragments of 16 per wave: 1 while the grid is small, 4 where there are enough tiles
// to fill the chip without it (the weights are then loaded once per 64 pixels).
constexpr int kPixWaves = 4;
template <bool DG, int J, bool V4, bool MASK>
__global__ __launch_bounds__(64 * kPixWaves) void k_f32_pix(const F32Args p)
{
    constexpr int U = J == 1 ? 4 : 2;   // reduction steps whose loads are issued together
    const ConvGeom &g = p.g;
    __shared__ f32x4 part[kPixWaves - 1][J][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const int ta = (p.rowsA + 15) >> 4, tile = p.tile0 + blockIdx.x;
    const int a0 = (tile % ta) * 16, b0 = (tile / ta) * 16 * J;
    const int cblocks = (p.red + 15) >> 4, steps = g.R * g.S * cblocks;

    int ih0[J], iw0[J], img[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int m = (int)((unsigned)b0 + j * 16 + lr);   // pixels past the last may be past 2^31: compared unsigned
        const int n = p.plane.div(m), rem = m - n * (int)p.plane.d, r = p.row.div(rem), c = rem - r * (int)p.row.d;
        img[j] = (unsigned)m < (unsigned)p.rowsB ? n : -1;
        ih0[j] = DG ? r + g.ph : r * g.sh - g.ph;
        iw0[j] = DG ? c + g.pw : c * g.sw - g.pw;
    }
    f32x4 acc[J];
#pragma unroll
    for (int j = 0; j < J; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int s0 = wave; s0 < steps; s0 += kPixWaves * U) {
        f32x4 a[U], b[U][J];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int st = s0 + u * kPixWaves;
            const bool on = st < steps;
            const int tap = p.cblk.div(st), c = (st - tap * cblocks) * 16 + lg * 4;
            const int tr = p.tap.div(tap), ts = tap - tr * g.S;
            const int left = on ? p.red - c : 0;
            if constexpr (DG) {
                // weights [k][tap][c]: four reduction rows k = c .. c+3, channel a0 + lr
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool ok = left > e && a0 + lr < p.rowsA;
                    const float t = *(ok ? p.w + ((size_t)(c + e) * g.R * g.S + tap) * g.C + a0 + lr : p.w);
                    a[u][e] = ok ? t : 0.f;
                }
            } else {
                a[u] = load4<V4>(p.w + ((size_t)(a0 + lr) * g.R * g.S + tap) * g.C + c, p.w, a0 + lr < p.rowsA ? left : 0);
            }
#pragma unroll
            for (int j = 0; j < J; ++j) {
                bool ok = img[j] >= 0;
                int hh = DG ? ih0[j] - tr : ih0[j] + tr, ww = DG ? iw0[j] - ts : iw0[j] + ts;
                const int Hl = DG ? g.Ho : g.H, Wl = DG ? g.Wo : g.W;
                if constexpr (DG) {
                    ok = ok && hh >= 0 && ww >= 0;
                    const int hq = p.sh.div(ok ? hh : 0), wq = p.sw.div(ok ? ww : 0);   // a tap counts where it meets the stride grid
                    ok = ok && hq * g.sh == hh && wq * g.sw == ww;
                    hh = hq; ww = wq;
                }
                ok = ok && (unsigned)hh < (unsigned)Hl && (unsigned)ww < (unsigned)Wl;
                const size_t o = ok ? (((size_t)img[j] * Hl + hh) * Wl + ww) * p.red + c : 0;
                b[u][j] = load4<V4>(p.b + o, p.b, ok ? left : 0);
                if constexpr (MASK) {
                    const f32x4 y = load4<V4>(p.mask + o, p.mask, ok ? left : 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) b[u][j][e] = y[e] > 0.f ? b[u][j][e] : 0.f;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][e], b[u][j][e], acc[j], 0, 0, 0);
    }
    if (wave > 0)
#pragma unroll
        for (int j = 0; j < J; ++j) part[wave - 1][j][lane] = acc[j];
    __syncthreads();
    if (wave > 0) return;
    // register v of lane l: channel 4 * (l / 16) + v, pixel l % 16
    const int ch = a0 + 4 * lg;
    auto store = [&](const F32Args &q, float r, int pix, int c) {
        const size_t o = (size_t)pix * q.rowsA + c;
        if (q.flags & KF_BIAS) r += q.bias[c];
        if ((q.flags & KF_RELU) && !(r > 0.f)) r = 0.f;
        if (q.xin != nullptr && !(q.xin[o] > 0.f)) r = 0.f;   // backward of the ReLU that produced the layer's input
        q.out[o] = r;
    };
    unsigned nan = 0;   // products that are NaN: bit 4 * j + v
#pragma unroll
    for (int j = 0; j < J; ++j) {
        for (int q = 0; q < kPixWaves - 1; ++q) acc[j] += part[q][j][lane];
        const int pix = (int)((unsigned)b0 + j * 16 + lr);
        if ((unsigned)pix >= (unsigned)p.rowsB) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (ch + v >= p.rowsA) continue;
            nan |= acc[j][v] != acc[j][v] ? 1u << (4 * j + v) : 0u;
            store(p, acc[j][v], pix, ch + v);
        }
    }
    if (nan == 0) return;
    // rare, and at no cost in registers to the rest: a loop of its own, the arguments read afresh
    auto args = (const __attribute__((address_space(4))) F32Args *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const F32Args &q = *(const F32Args *)args;
    for (; nan != 0; nan &= nan - 1) {
        const int e = __ffs(nan) - 1, pix = b0 + (e >> 2) * 16 + lr, c = ch + (e & 3);
        store(q, sum_of_reached_taps<DG, MASK>(q, pix, c), pix, c);
    }
}

// Filter gradient: D[k][c] of one tap = sum over output pixels dy[m][k] * x[m at tap][c]; the reduction runs over pixels, 16 per
// step, dealt over the block's waves.  A block owns 16 k x 16 c of one tap; one more block per 16 k (the one behind the last tap)
// multiplies dy with ones instead of x: the bias gradient, without a launch of its own.  There are few tiles (30 for 15 -> 34
// channels), so a block has 16 waves; bound by the address unit (4-byte loads, 16 channels of 4 pixels each).
constexpr int kWgWaves = 16;
// U: steps per wave whose loads are issued together.  A layer with few pixels has one or two steps for each of the waves and
// takes no more (the waves of a tile share one CU, whose load rate bounds them: 2 x 16 x 16 pixels with four, two of them empty, 8.7 us, with
// two 6.2 us).
// PAD: a tap can lie outside the image.
template <bool MASK, int U, bool PAD>
__global__ __launch_bounds__(64 * kWgWaves, U == 4 ? 4 : 8) void k_f32_wgrad(const F32Args p, float *dbias)
{
    const ConvGeom &g = p.g;
    __shared__ f32x4 part[kWgWaves - 1][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 15, lg = lane >> 4;
    const int ktiles = (g.K + 15) >> 4, ctiles = (g.C + 15) >> 4, bt = blockIdx.x / ktiles, k0 = (blockIdx.x - bt * ktiles) * 16, k = k0 + lr;
    const int tap = bt / ctiles, c = (bt - tap * ctiles) * 16 + lr;
    const bool ones = tap >= g.R * g.S;
    if (ones && dbias == nullptr) return;   // block-uniform
    const int tr = tap / g.S, ts = tap - tr * g.S, steps = (p.rowsB + 15) >> 4;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = wave; s0 < steps; s0 += kWgWaves * U) {
        float a[U][4], b[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int m0 = (s0 + u * kWgWaves) * 16 + lg * 4;   // four pixels in a row: one division, then carries
            int n = p.plane.div(m0), rem = m0 - n * (int)p.plane.d, pp = p.row.div(rem), q = rem - pp * (int)p.row.d;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // both operands are zero where the tap is outside the image (an infinite dy times zero is NaN)
                const int ih = pp * g.sh - g.ph + tr, iw = q * g.sw - g.pw + ts;
                const bool in = (unsigned)m0 + e < (unsigned)p.rowsB && (!PAD || ones || ((unsigned)ih < (unsigned)g.H && (unsigned)iw < (unsigned)g.W)), ok = in && k < g.K;
                const size_t oa = ok ? (size_t)(m0 + e) * g.K + k : 0;
                float t = p.b[oa];
                if constexpr (MASK) t = p.mask[oa] > 0.f ? t : 0.f;
                a[u][e] = ok ? t : 0.f;
                const bool okx = in && !ones && c < g.C;
                const float x = p.w[okx ? (((size_t)n * g.H + ih) * g.W + iw) * g.C + c : 0];
                b[u][e] = okx ? x : ones ? 1.f : 0.f;
                const bool wrap = ++q == g.Wo;
                q = wrap ? 0 : q;
                pp += wrap ? 1 : 0;
                const bool next = pp == g.Ho;
                pp = next ? 0 : pp;
                n += next ? 1 : 0;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][e], b[u][e], acc, 0, 0, 0);
    }
    if (wave > 0) part[wave - 1][lane] = acc;
    __syncthreads();
    if (wave > 0) return;
    for (int q = 0; q < kWgWaves - 1; ++q) acc += part[q][lane];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int kk = k0 + 4 * lg + v;
        if (kk >= g.K) continue;
        if (ones) { if (lr == 0) dbias[kk] = acc[v]; }
        else if (c < g.C) p.out[((size_t)kk * g.R * g.S + tap) * g.C + c] = acc[v];
    }
}

bool wgrad_padded(const ConvGeom &g) { return g.ph > 0 || g.pw > 0; }
int wgrad_unroll(int pixels) { return pixels <= 16 * kWgWaves ? 1 : pixels <= 2 * 16 * kWgWaves ? 2 : 4; }

bool wide_tiles(long long rowsA, long long rowsB) { return (rowsA + 15) / 16 * ((rowsB + 63) / 64) >= 1024; }   // enough 16 x 64 tiles for four blocks per CU

hipError_t launch_pix(bool dg, const F32Args &a, hipStream_t st)
{
    const long long ta = (a.rowsA + 15) / 16;
    const bool wide = wide_tiles(a.rowsA, a.rowsB);
    const long long tiles = ta * (wide ? ((long long)a.rowsB + 63) / 64 : ((long long)a.rowsB + 15) / 16);
    const bool v4 = a.red % 4 == 0;
    // a grid holds fewer than 2^32 threads: a layer of few channels and more than 2^30 pixels takes several launches
    constexpr long long kMaxTiles = (1ll << 32) / (64 * kPixWaves) - 1;
    auto run = [&](auto kernel) {
        F32Args part = a;
        for (long long t0 = 0; t0 < tiles; t0 += kMaxTiles) {
            part.tile0 = (int)t0;
            hipLaunchKernelGGL(kernel, dim3((unsigned)std::min(kMaxTiles, tiles - t0)), dim3(64 * kPixWaves), 0, st, part);
        }
    };
    auto pick = [&](auto dgc, auto maskc) {
        constexpr bool DG = decltype(dgc)::value, MASK = decltype(maskc)::value;
        if (wide && v4) run(k_f32_pix<DG, 4, true, MASK>);
        else if (wide) run(k_f32_pix<DG, 4, false, MASK>);
        else if (v4) run(k_f32_pix<DG, 1, true, MASK>);
        else run(k_f32_pix<DG, 1, false, MASK>);
    };
    if (!dg) pick(std::false_type(), std::false_type());
    else if (a.mask != nullptr) pick(std::true_type(), std::true_type());
    else pick(std::true_type(), std::false_type());
    return hipGetLastError();
}

}  // namespace

void f32_kernel_name(const ConvGeom &g, int pass, bool masked, char *name, size_t name_bytes)
{
    if (pass == PASS_WGRAD) { snprintf(name, name_bytes, "k_f32_wgrad<%s, %d, %s>", masked ? "true" : "false", wgrad_unroll(g.N * g.Ho * g.Wo), wgrad_padded(g) ? "true" : "false"); return; }
    const bool dg = pass == PASS_DGRAD, v4 = (dg ? g.K : g.C) % 4 == 0;
    const bool wide = dg ? wide_tiles(g.C, (long long)g.N * g.H * g.W) : wide_tiles(g.K, (long long)g.N * g.Ho * g.Wo);
    snprintf(name, name_bytes, "k_f32_pix<%s, %d, %s, %s>", dg ? "true" : "false", wide ? 4 : 1, v4 ? "true" : "false", dg && masked ? "true" : "false");
}

hipError_t f32_conv_fwd(const ConvGeom &g, unsigned flags, const float *x, const float *w, const float *bias,
                        float *y, hipStream_t st)
{
    F32Args a{};
    a.g = g; a.plane = FastDiv::of(g.Ho * g.Wo); a.row = FastDiv::of(g.Wo); a.sh = FastDiv::of(g.sh); a.sw = FastDiv::of(g.sw); a.tap = FastDiv::of(g.S);
    a.cblk = FastDiv::of((g.C + 15) / 16);
    a.rowsA = g.K; a.rowsB = g.N * g.Ho * g.Wo; a.red = g.C; a.flags = flags;
    a.w = w; a.b = x; a.bias = bias; a.out = y;
    return launch_pix(false, a, st);
}

hipError_t f32_conv_dgrad(const ConvGeom &g, const float *dy, const float *ymask, const float *w, const float *xin, float *dx, hipStream_t st)
{
    F32Args a{};
    a.g = g; a.plane = FastDiv::of(g.H * g.W); a.row = FastDiv::of(g.W); a.sh = FastDiv::of(g.sh); a.sw = FastDiv::of(g.sw); a.tap = FastDiv::of(g.S);
    a.cblk = FastDiv::of((g.K + 15) / 16);
    a.rowsA = g.C; a.rowsB = g.N * g.H * g.W; a.red = g.K;
    a.w = w; a.b = dy; a.mask = ymask; a.xin = xin; a.out = dx;
    return launch_pix(true, a, st);
}

// dw and, if asked for, the bias gradient in one launch
hipError_t f32_conv_wgrad(const ConvGeom &g, const float *x, const float *dy, const float *ymask, float *dw, float *dbias, hipStream_t st)
{
    F32Args a{};
    a.g = g; a.plane = FastDiv::of(g.Ho * g.Wo); a.row = FastDiv::of(g.Wo);
    a.rowsB = g.N * g.Ho * g.Wo;
    a.w = x; a.b = dy; a.mask = ymask; a.out = dw;
    const long long tiles = (long long)g.R * g.S * ((g.C + 15) / 16);
    const dim3 grid((unsigned)((g.K + 15) / 16 * (tiles + (dbias != nullptr ? 1 : 0)))), block(64 * kWgWaves);
    auto pick = [&](auto maskc, auto padc) {
        constexpr bool MASK = decltype(maskc)::value, PAD = decltype(padc)::value;
        const int u = wgrad_unroll(a.rowsB);
        hipLaunchKernelGGL((u == 1 ? k_f32_wgrad<MASK, 1, PAD> : u == 2 ? k_f32_wgrad<MASK, 2, PAD> : k_f32_wgrad<MASK, 4, PAD>), grid, block, 0, st, a, dbias);
    };
    const bool pad = wgrad_padded(g);
    if (ymask != nullptr && pad) pick(std::true_type(), std::true_type());
    else if (ymask != nullptr) pick(std::true_type(), std::false_type());
    else if (pad) pick(std::false_type(), std::true_type());
    else pick(std::false_type(), std::false_type());
    return hipGetLastError();
}
