// 1x1 forward (any stride and padding) and unit-stride backward-data with the weights stationary in registers.
//
// These layers stream: 64 x 56 x 56, 256 -> 128 channels moves 154 MB for 13 GFLOP.  A tiled kernel spends a block on each tile,
// with weights, a pipeline to fill and an epilogue of its own for 2 - 8 reduction steps, and reads the pixels once per channel tile.
// Here blocks are persistent (two per CU over all channel tiles, so that one multiplies or stores while the other waits): a wave keeps
// the weights of its 32 or 64 output channels for the whole reduction (up to 512 channels) and the pixels go by through a ring of
// LDS buffers, NB - 1 of them on their way at any time.  One barrier per buffer; results are reordered in the wave's own staging area and
// go out 64 or 128 bytes per pixel; the saved input of a masked tile is asked for a whole buffer ahead.
// Bound by memory (us back to back / with flushed caches, before -> now; 5.2 TB/s is what a large copy reaches):
//   64 x 56 x 56, 256 -> 128 forward 34 / 57 -> 27 / 50, masked backward-data (257 MB) 57 / 87 -> 38 / 79; 64 -> 256 forward 53 / 61 -> 21 / 32;
//   64 x 28 x 28, 128 -> 512 forward 24 / 29 -> 16 / 22; 64 x 56 x 56, 256 -> 512 stride 2 29 / 38 -> 21 / 34; 64 x 28 x 28, 512 -> 512 42 / 51 -> 30 / 43.
// Weights straight from memory into registers (32 rows an instruction) took 1 - 4 us longer than through the ring.  More than 512 reduction channels do not fit
// the registers of two blocks a CU; those layers are long enough for the tiles.
#include "dma_common.h"
#include <algorithm>
#include <cstdio>

namespace {

// TC: 64-channel blocks of the reduction; AW: 32-channel groups of a wave; WC: waves side by side over the channels (the other 4 / WC
// groups of waves take every second pixel fragment)
template <int TC, int AW, int WC> struct Pw {
    static constexpr int WP = 4 / WC, TA = 32 * AW * WC;
    static constexpr int PIX = TC == 1 ? 128 : TC == 2 || WP == 2 ? 64 : 32;     // pixels per buffer
    static constexpr int BUF = PIX * TC * 128, STAGE = 4 * AW * 2048, LDS_MAX = 80 * 1024;
    static constexpr int NB_FIT = (LDS_MAX - STAGE - TA * 4) / BUF, NB = NB_FIT < 4 ? NB_FIT : 4;
    static constexpr int LDS = NB * BUF + STAGE + TA * 4;
    static constexpr int F = PIX / 32 / WP;          // pixel fragments per wave and buffer
    static constexpr int PG = PIX / 32, CP = PG * TC;   // groups of 8 pixels, and copies, per wave and buffer
    static constexpr int M = F * AW * 2;             // 16-byte stores per lane and buffer
    static_assert(NB >= 2 && F >= 1, "a ring of buffers");
};

// out of range of any tensor, and so is what is added to it: tensors are smaller than 2 GiB
constexpr unsigned FAR = 0x80000000u;

// OPT: forward: the input is strided or padded; backward-data: fused backward of the ReLU in front of the layer
template <int PASS, int TC, int AW, int WC, bool OPT>
__global__ __launch_bounds__(256, 2) void k_pointwise(const KArgs p, int tiles)
{
#if __HIP_DEVICE_COMPILE__   // the host pass only needs the launch stub
    typedef Pw<TC, AW, WC> D;
    constexpr bool FWD = PASS == PASS_FWD, MASK = !FWD && OPT, GATHER = FWD && OPT;
    constexpr int T = TC * 64, NB = D::NB, DEPTH = 3;   // fragment reads run DEPTH 16-channel slices ahead
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const ConvGeom &g = p.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wc = wave % WC, wp = wave / WC;
    const int a0 = blockIdx.y * D::TA, aw0 = a0 + wc * (AW * 32);
    const unsigned smem_base = lds_offset(smem);
    float *bias_lds = reinterpret_cast<float *>(smem + NB * D::BUF + D::STAGE);
    const __amdgpu_buffer_rsrc_t rin = FWD ? make_rsrc(p.x, (size_t)g.N * g.H * g.W * T * 2) : make_rsrc(p.dy, (size_t)g.N * g.Ho * g.Wo * T * 2);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(p.w, (size_t)p.rowsA * T * 2);
    const size_t out_bytes = (size_t)p.rowsB * p.rowsA * 2;
    const __amdgpu_buffer_rsrc_t rout = make_rsrc(p.out, out_bytes), rx = make_rsrc(MASK ? (const void *)p.x : p.out, out_bytes);

    if constexpr (FWD)
        if (tid < D::TA) bias_lds[tid] = (p.flags & KF_BIAS) && a0 + tid < p.rowsA ? p.bias[a0 + tid] : 0.f;

    // Pixel copies: instruction (pixel group j, 64-channel block tc) of a wave fills 8 pixels x 128 bytes; chunk c of pixel px lies at c ^ ((px >> 1) & 7)
    auto copy_tile = [&](int tile, unsigned buf, bool on) {   // a tile past the last fetches nothing
#pragma unroll
        for (int j = 0; j < D::PG; ++j) {
            const int pl = (wave * D::PG + j) * 8 + (lane >> 3), pix = tile * D::PIX + pl;
            const unsigned chunk = (unsigned)(lane & 7) ^ ((unsigned)(pl >> 1) & 7u);
            unsigned at;
            if constexpr (GATHER) {
                const unsigned row = (unsigned)pix / (unsigned)g.Wo, n = row / (unsigned)g.Ho;
                const int h = (int)(row - n * g.Ho) * g.sh - g.ph, w = (int)((unsigned)pix - row * g.Wo) * g.sw - g.pw;
                const bool in = on && pix < p.rowsB && (unsigned)h < (unsigned)g.H && (unsigned)w < (unsigned)g.W;
                at = in ? (unsigned)(((int)n * g.H + h) * g.W + w) * (unsigned)(T * 2) + (chunk << 4) : FAR;
            } else at = on && pix < p.rowsB ? (unsigned)pix * (unsigned)(T * 2) + (chunk << 4) : FAR;
#pragma unroll
            for (int tc = 0; tc < TC; ++tc)
                dma16(rin, buf + tc * (D::PIX * 128) + (wave * D::PG + j) * 1024, at + tc * 128);
        }
    };

    // This wave's weights, fragment (aw, 16-channel slice), through its share of the ring in units of a few KB: forward: 32 output channels x 64 reduction
    // channels, chunk c of a row at c ^ ((row >> 1) & 7); backward-data, [reduction][channel] in memory: 32 reduction rows, read transposed
    u32x4 wf[AW][TC * 4];
    constexpr int RB = FWD ? 128 : AW * 64, UNIT = 32 * RB, UNITS = FWD ? AW * TC : TC * 2;   // bytes per row and unit
    constexpr int SHARE = NB * D::BUF / 4, FIT = SHARE / UNIT, SLOTS = FIT < UNITS ? FIT : UNITS;
    static_assert(FIT >= 2, "units in flight");
    const unsigned share = smem_base + wave * SHARE;
    auto copy_unit = [&](int u) {
#pragma unroll
        for (int q = 0; q < UNIT / 1024; ++q) {
            const int row = q * (1024 / RB) + lane / (RB / 16), c = lane % (RB / 16);
            unsigned at;
            if constexpr (FWD) {
                const int ch = aw0 + u / TC * 32 + row;
                at = ch < p.rowsA ? (unsigned)ch * (T * 2u) + u % TC * 128 + ((c ^ ((row >> 1) & 7)) << 4) : FAR;
            } else {
                const int ch = aw0 + (AW == 2 ? c ^ (seg_swz<64>(row) << 2) : c) * 8;
                at = ch < p.rowsA ? ((unsigned)(u * 32 + row) * (unsigned)p.rowsA + ch) * 2u : FAR;
            }
            dma16(rw, share + (u % SLOTS) * UNIT + q * 1024, at);
        }
    };
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) copy_unit(u);
    for_constant<UNITS>([&](auto U) {
        constexpr int u = U, newer = (UNITS - 1 - u < SLOTS - 1 ? UNITS - 1 - u : SLOTS - 1) * (UNIT / 1024);
        const unsigned base = share + (u % SLOTS) * UNIT;
        wait_vmcnt<newer>();
        if constexpr (FWD) {
            const int row = lane & 31;
#pragma unroll
            for (int k = 0; k < 4; ++k) wf[u / TC][u % TC * 4 + k] = lds_read16<0>(base + row * 128 + (((2 * k + (lane >> 5)) ^ ((row >> 1) & 7)) << 4));
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(wf[u / TC][u % TC * 4 + k]));
        } else {
            const int i16 = lane & 15, t = (lane >> 5) * 8 + (i16 >> 2), cl = ((lane >> 4) & 1) * 16 + (i16 & 3) * 4;
            u32x2 lo[AW][2], hi[AW][2];
#pragma unroll
            for (int aw = 0; aw < AW; ++aw)
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const unsigned ad = base + (k * 16 + t) * RB + (AW == 2 ? (unsigned)(aw ^ seg_swz<64>(t)) << 6 : 0u) + cl * 2;
                    lo[aw][k] = lds_read_tr<0>(ad);
                    hi[aw][k] = lds_read_tr<4 * RB>(ad);
                }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int aw = 0; aw < AW; ++aw)
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    asm volatile("" : "+v"(lo[aw][k]));
                    asm volatile("" : "+v"(hi[aw][k]));
                    wf[aw][u * 2 + k] = u32x4{lo[aw][k].x, lo[aw][k].y, hi[aw][k].x, hi[aw][k].y};
                }
        }
        if constexpr (u + SLOTS < UNITS) copy_unit(u + SLOTS);
    });
    __builtin_amdgcn_s_barrier();   // the ring is free

    const TileWalk tw = tile_walk(tiles);
    int tile = tw.first;
#pragma unroll
    for (int j = 0; j < NB - 1; ++j) copy_tile(tile + j * tw.stride, smem_base + j * D::BUF, tile + j * tw.stride < tw.end);

    // results: written by pixel fragment, read back 4 AW lanes to a pixel
    constexpr int LP = 4 * AW, RPI = 64 / LP;   // lanes per pixel, pixels per instruction
    const unsigned stg = smem_base + NB * D::BUF + wave * (AW * 2048);
    const int wpx = lane & 31, rpx = lane / LP, och = aw0 + (lane % LP) * 8;
    const unsigned wsw = AW == 2 ? wpx & 7 : (wpx >> 2) & 3;
    const unsigned stw = stg + wpx * (AW * 64) + (((unsigned)(lane >> 5) ^ wsw) << 4);
    const unsigned str = stg + rpx * (AW * 64) + (((unsigned)(lane % LP) ^ (AW == 2 ? rpx & 7 : (rpx >> 2) & 3)) << 4);
    const unsigned bad = lds_offset(bias_lds) + (wc * (AW * 32) + 4 * (lane >> 5)) * 4;
    // this lane's pixel of fragment f, 16-channel slice 0
    const unsigned col = smem_base + (wp * D::F * 32 + (lane & 31)) * 128 + (((unsigned)(lane >> 5) ^ ((unsigned)(lane >> 1) & 7u)) << 4);
    auto out_at = [&](int t, int f) {   // this lane's first output vector of fragment f; an offset past the tensor is dropped by the hardware
        const int pix = t * D::PIX + (wp * D::F + f) * 32 + rpx;
        return och < p.rowsA && t < tw.end ? ((unsigned)pix * (unsigned)p.rowsA + och) * 2u : FAR;
    };
    auto vec_at = [&](unsigned at, int i) { return at + (unsigned)(i * RPI) * (unsigned)p.rowsA * 2u; };
    u32x4 mk[D::F][2 * AW];
    if constexpr (MASK) {
#pragma unroll
        for (int f = 0; f < D::F; ++f)
#pragma unroll
            for (int i = 0; i < 2 * AW; ++i) mk[f][i] = __builtin_amdgcn_raw_buffer_load_b128(rx, vec_at(out_at(tile, f), i), 0, 0);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the bias, before the first barrier

    constexpr int PER = D::M * (MASK ? 2 : 1), STEADY = PER + (NB - 2) * (D::CP + PER);
    for (int it = 0; tile < tw.end; tile += tw.stride, ++it) {
        // of this wave's loads and stores after its share of this buffer: what the iterations since have issued
        if (it < NB - 1) wait_vmcnt<(NB - 2) * D::CP < 63 ? (NB - 2) * D::CP : 63>();
        else wait_vmcnt<STEADY < 63 ? STEADY : 63>();
        __builtin_amdgcn_s_barrier();   // all shares have landed; everyone has read the buffer before
        const int ahead = tile + (NB - 1) * tw.stride;
        copy_tile(ahead, smem_base + (it + NB - 1) % NB * D::BUF, ahead < tw.end);
        const unsigned cb = col + it % NB * D::BUF;
        f32x4 bv[AW][4];
        for_constant<D::F>([&](auto FR) {
            constexpr int f = FR;
            f32x16 acc[AW];
#pragma unroll
            for (int aw = 0; aw < AW; ++aw)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[aw][v] = 0.f;
            u32x4 fb[DEPTH + 1];
            auto read_b = [&](auto SL) {
                constexpr int sl = SL;
                fb[sl % (DEPTH + 1)] = lds_read16<sl / 4 * (D::PIX * 128) + f * 4096>(cb ^ (unsigned)((sl & 3) << 5));
            };
            for_constant<DEPTH>([&](auto SL) { read_b(SL); });
            for_constant<TC * 4>([&](auto SL) {
                constexpr int sl = SL, left = TC * 4 - 1 - sl, newer = left < DEPTH ? left : DEPTH;
                if constexpr (sl + DEPTH < TC * 4) read_b(std::integral_constant<int, sl + DEPTH>{});
                asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(newer));
                asm volatile("" : "+v"(fb[sl % (DEPTH + 1)]));
#pragma unroll
                for (int aw = 0; aw < AW; ++aw)
                    acc[aw] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, wf[aw][sl]),
                                                                      __builtin_bit_cast(bf16x8, fb[sl % (DEPTH + 1)]), acc[aw], 0, 0, 0);
            });
            // accumulator element v of lane l is channel 8*(v/4) + 4*(l/32) + v%4 of pixel l%32; the lanes l and l+32 swap halves of
            // two channel groups, after which each holds 8 consecutive channels of one group
#pragma unroll
            for (int aw = 0; aw < AW; ++aw) {
                if constexpr (FWD) {
                    if (p.flags & KF_BIAS) {
                        bv[aw][0] = __builtin_bit_cast(f32x4, lds_read16<0>(bad + aw * 128)); bv[aw][1] = __builtin_bit_cast(f32x4, lds_read16<32>(bad + aw * 128));
                        bv[aw][2] = __builtin_bit_cast(f32x4, lds_read16<64>(bad + aw * 128)); bv[aw][3] = __builtin_bit_cast(f32x4, lds_read16<96>(bad + aw * 128));
                        asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            asm volatile("" : "+v"(bv[aw][k]));
                            acc[aw][4 * k] += bv[aw][k].x; acc[aw][4 * k + 1] += bv[aw][k].y; acc[aw][4 * k + 2] += bv[aw][k].z; acc[aw][4 * k + 3] += bv[aw][k].w;
                        }
                    }
                    if (p.flags & KF_RELU) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[aw][v] = acc[aw][v] > 0.f ? acc[aw][v] : 0.f;
                    }
                }
#pragma unroll
                for (int gp = 0; gp < 2; ++gp) {
                    const int e = 8 * gp;
                    const unsigned a_lo = pack_bf16(acc[aw][e], acc[aw][e + 1]), a_hi = pack_bf16(acc[aw][e + 2], acc[aw][e + 3]);
                    const unsigned b_lo = pack_bf16(acc[aw][e + 4], acc[aw][e + 5]), b_hi = pack_bf16(acc[aw][e + 6], acc[aw][e + 7]);
                    const auto s0 = __builtin_amdgcn_permlane32_swap(a_lo, b_lo, false, false);
                    const auto s1 = __builtin_amdgcn_permlane32_swap(a_hi, b_hi, false, false);
                    lds_write16(stw ^ (unsigned)((aw * 4 + gp * 2) << 4), u32x4{s0[0], s1[0], s0[1], s1[1]});   // chunk aw * 4 + gp * 2 + l / 32
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            u32x4 o[2 * AW];
            for_constant<2 * AW>([&](auto I) { o[I] = lds_read16<I * 1024>(str); });
            asm volatile("s_waitcnt lgkmcnt(0)");
            const unsigned at = out_at(tile, f);
#pragma unroll
            for (int i = 0; i < 2 * AW; ++i) {
                asm volatile("" : "+v"(o[i]));
                if constexpr (MASK) o[i] = apply_mask(o[i], mk[f][i]);
                __builtin_amdgcn_raw_buffer_store_b128(o[i], rout, vec_at(at, i), 0, 0);
            }
            if constexpr (MASK) {
                const unsigned nx = out_at(tile + tw.stride, f);
#pragma unroll
                for (int i = 0; i < 2 * AW; ++i) mk[f][i] = __builtin_amdgcn_raw_buffer_load_b128(rx, vec_at(nx, i), 0, 0);
            }
        });
    }
#endif
}

typedef void (*PwFn)(const KArgs, int);
template <int PASS, int AW, int WC, bool OPT> PwFn pick_tc(int tc)
{
    switch (tc) {
    case 1: return k_pointwise<PASS, 1, AW, WC, OPT>;
    case 2: return k_pointwise<PASS, 2, AW, WC, OPT>;
    case 3: return k_pointwise<PASS, 3, AW, WC, OPT>;
    case 4: return k_pointwise<PASS, 4, AW, WC, OPT>;
    }
    if constexpr (AW == 1 && WC == 4)
        switch (tc) {
        case 5: return k_pointwise<PASS, 5, AW, WC, OPT>;
        case 6: return k_pointwise<PASS, 6, AW, WC, OPT>;
        case 7: return k_pointwise<PASS, 7, AW, WC, OPT>;
        case 8: return k_pointwise<PASS, 8, AW, WC, OPT>;
        }
    return nullptr;
}
// variant 0: 64 channels per block, 1: 128, 2: 256
template <int PASS, bool OPT> PwFn pick_pw(int v, int tc)
{
    return v == 0 ? pick_tc<PASS, 1, 2, OPT>(tc) : v == 1 ? pick_tc<PASS, 1, 4, OPT>(tc) : pick_tc<PASS, 2, 4, OPT>(tc);
}
PwFn pick_pw(int pass, int v, int tc, bool opt)
{
    if (pass == PASS_FWD) return opt ? pick_pw<PASS_FWD, true>(v, tc) : pick_pw<PASS_FWD, false>(v, tc);
    return opt ? pick_pw<PASS_DGRAD, true>(v, tc) : pick_pw<PASS_DGRAD, false>(v, tc);
}
template <int TC, int AW, int WC> void shape(int *pix, int *lds) { *pix = Pw<TC, AW, WC>::PIX; *lds = Pw<TC, AW, WC>::LDS; }
template <int AW, int WC> bool shape_tc(int tc, int *pix, int *lds)
{
    switch (tc) {
    case 1: shape<1, AW, WC>(pix, lds); return true;
    case 2: shape<2, AW, WC>(pix, lds); return true;
    case 3: shape<3, AW, WC>(pix, lds); return true;
    case 4: shape<4, AW, WC>(pix, lds); return true;
    }
    if constexpr (AW == 1 && WC == 4)
        switch (tc) {
        case 5: shape<5, AW, WC>(pix, lds); return true;
        case 6: shape<6, AW, WC>(pix, lds); return true;
        case 7: shape<7, AW, WC>(pix, lds); return true;
        case 8: shape<8, AW, WC>(pix, lds); return true;
        }
    return false;
}
bool pw_shape(int v, int tc, int *pix, int *lds)
{
    return v == 0 ? shape_tc<1, 2>(tc, pix, lds) : v == 1 ? shape_tc<1, 4>(tc, pix, lds) : shape_tc<2, 4>(tc, pix, lds);
}

}  // namespace

hipError_t pw_init()
{
    for (int pass = 0; pass < 2; ++pass)
        for (int v = 0; v < 3; ++v)
            for (int tc = 1; tc <= 8; ++tc)
                for (int opt = 0; opt < 2; ++opt) {
                    int pix, lds;
                    if (!pw_shape(v, tc, &pix, &lds)) continue;
                    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(pick_pw(pass, v, tc, opt != 0)), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
                    if (e != hipSuccess) return e;
                }
    return hipSuccess;
}

// force_splits: blocks per channel tile (0: two per CU over all channel tiles)
bool pw_plan(const ConvGeom &g, int pass, int variant, int force_splits, GemmPlan *pl)
{
    if (pass == PASS_WGRAD || variant < 0 || variant > 2 || g.R != 1 || g.S != 1) return false;
    const bool fwd = pass == PASS_FWD;
    if (!fwd && (g.sh != 1 || g.sw != 1 || g.ph != 0 || g.pw != 0)) return false;
    const int red = fwd ? g.C : g.K, rowsA = fwd ? g.K : g.C;
    const long long rowsB = fwd ? (long long)g.N * g.Ho * g.Wo : (long long)g.N * g.H * g.W;
    int pix, lds;
    if (red % 64 != 0 || rowsA % 8 != 0 || red > 512 || !pw_shape(variant, red / 64, &pix, &lds)) return false;
    // 32-bit offsets, also of the tiles that a block asks for past its last
    const long long in = (long long)g.N * g.H * g.W * g.C * 2, out = (long long)g.N * g.Ho * g.Wo * g.K * 2, w = (long long)g.K * g.C * 2;
    if (in >= 0x7fffffffLL || out >= 0x7fffffffLL || w >= 0x7fffffffLL) return false;
    pl->variant = variant; pl->TA = 64 << variant; pl->TB = pix; pl->BK = 64;
    pl->vecA = pl->vecB = true; pl->fast = true; pl->dma = true; pl->halo = false; pl->phase = pl->fill = false; pl->wstrip = false; pl->wwin = false;
    pl->win = false; pl->pw = true; pl->pw_gather = fwd && (g.sh != 1 || g.sw != 1 || g.ph != 0 || g.pw != 0);
    pl->tilesA = (rowsA + pl->TA - 1) / pl->TA;
    pl->tilesB = (int)((rowsB + pix - 1) / pix);
    pl->steps_total = pl->steps_per_split = red / 64;
    pl->splits = 1;
    pl->blocks = force_splits > 1 ? force_splits : 0;
    return true;
}

void pw_kernel_name(int pass, const GemmPlan &pl, bool masked, char *name, size_t name_bytes)
{
    snprintf(name, name_bytes, "k_pointwise<%d, %d, %d, %d, %s>", pass, pl.steps_total, pl.variant == 2 ? 2 : 1, pl.variant == 0 ? 2 : 4,
             (pass == PASS_FWD ? pl.pw_gather : masked) ? "true" : "false");
}

int pw_blocks(const GemmPlan &pl)
{
    int blocks = pl.blocks > 0 ? pl.blocks : std::max(512 / pl.tilesA, 8);
    if (blocks > 8) blocks = blocks / 8 * 8;   // whole eighths: the channel tiles of a pixel tile on one compute die
    return std::min(blocks, pl.tilesB);
}

hipError_t pw_launch(const ConvArgs &a, hipStream_t st)
{
    KArgs p{};
    int pix, lds;
    const bool fwd = a.pass == PASS_FWD;
    const GemmPlan &pl = a.plan;
    if (!pw_shape(pl.variant, pl.steps_total, &pix, &lds)) return hipErrorInvalidValue;
    p.g = a.g;
    p.rowsA = fwd ? a.g.K : a.g.C; p.rowsB = fwd ? a.g.N * a.g.Ho * a.g.Wo : a.g.N * a.g.H * a.g.W; p.red = pl.steps_total * 64;
    p.tilesA = pl.tilesA; p.tilesB = pl.tilesB; p.steps_total = p.steps_per_split = pl.steps_total; p.splits = 1;
    p.flags = a.flags;
    p.x = a.x; p.w = a.w; p.dy = a.dy; p.bias = a.bias; p.out = a.out;
    hipLaunchKernelGGL(pick_pw(a.pass, pl.variant, pl.steps_total, fwd ? pl.pw_gather : (a.flags & KF_MASK_IN) != 0), dim3((unsigned)pw_blocks(pl), (unsigned)pl.tilesA), dim3(256),
                       (size_t)lds, st, p, pl.tilesB);
    dp_trace_main_kernel_done(st);
    return hipGetLastError();
}
