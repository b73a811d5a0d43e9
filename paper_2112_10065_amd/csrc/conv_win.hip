// Forward and backward-data of unit-stride layers with one window of pixels for all taps, for grids of few tiles.
//
// out[u][a] = sum over taps t and reduction channels c of src[u + o(t)][c] * w(t, c, a), for pixel slots u: an image row takes P slots and an
// image HP slot rows, as many as source and output need and the source's zero padding; slots without a source pixel hold zeros, so no
// tap needs a mask.  Forward: src = x, o = (r - pad_h) * P + s - pad_w; backward-data: src = dy, the mirrored offsets and filter.
// A block owns 32 WA output channels and 32 FB slots.  Per 64 reduction channels it copies the window of source slots that its taps reach once
// (TB + (R-1) P + S - 1 slots of 128 bytes, two buffers), where a tiled kernel copies the pixels once per tap; small grids are bound by that
// traffic out of the L2.
// Twelve waves, three per SIMD: WA of them over the channels, CBP over channel blocks and G = 12 / (WA CBP) over the taps.  A wave's weights are
// its own (32 channels of its taps), so it streams them through two 4 KB buffers in LDS that only it waits for; the waves meet once
// per channel block, for the window.  (With the weights shared and a barrier per tap the waves go through copying, LDS reads and matrix
// instructions in step, one after the other.)  The sums of the tap and channel groups meet in
// LDS at the end, in group order: the chip is filled by tiles alone, without a reduction split, partials in memory and a second kernel.
// Where a copy's data lies depends on the tile only: all offsets are computed before the loop, steps ride in the scalar offset.
// Measured (us, before: the best of the other kernels with their reduction kernel): 512 -> 512 on 28 x 28, 8 samples, forward 39.1 -> 34.5, masked
// backward-data 41.7 -> 36.6; 4 samples 28.2 -> 24.0 and 29.6 -> 25.2; 512 -> 512 on 14 x 14, 8 samples 22.5 -> 15.6 and 25.6 -> 17.9; 288 -> 384 on
// 35 x 35, 4 samples 32.4 -> 18.4 and 23.3 -> 19.5.  Tiles of 96 channels (three waves side by side, four tap groups) for channel counts that 64 and 128
// divide badly, or that fill the chip better so: backward-data 192 -> 80 on 73 x 73, 4 samples 23.6 -> 14.5; forward 272 -> 96 there 25.3 -> 19.4,
// 384 -> 288 on 26 x 26, 11 samples 28.3 -> 21.6.  What bounds it (counters at 8 samples): waits for copies and LDS reads.  On 28 x 28, 512 -> 512
// the matrix cores are busy for 0.52 of the time and the waves wait at counters and barriers for 0.42 of theirs; on 14 x 14 0.3 and 0.5, where the fixed
// part of a launch (3 - 7 us of the fitted price: first copies, sums, stores) is most of it.
#include "dma_common.h"
#include <cstdio>

namespace {

constexpr int kWaves = 12, kThreads = 64 * kWaves, kMaxWindowCopies = 3, kLdsBytes = 160 * 1024, kSlot = 4096, kWeightBytes = kWaves * 2 * kSlot;

struct WinArgs {
    int P, HP;                 // slots per image row, slot rows per image
    int first;                 // first slot of a tile's window, relative to the tile's first slot
    int Hs, Ws, Hd, Wd;        // source and output image
    int CR, ncb;               // reduction channels, blocks of 64 of them
    int wrows;                 // window rows in LDS
};

// the fragments of one 16-channel slice: FA times 32 output channels, FB times 32 slots; backward-data reads the weights through the
// transpose read, in two halves
template <bool DG, int FA, int FB> struct Frags {
    u32x4 a, b[FB];
    u32x2 lo[FA], hi[FA];
    DEVFN void landed()
    {
        asm volatile("s_waitcnt lgkmcnt(0)");
        if constexpr (DG) {
#pragma unroll
            for (int i = 0; i < FA; ++i) { asm volatile("" : "+v"(lo[i])); asm volatile("" : "+v"(hi[i])); }
        } else
            asm volatile("" : "+v"(a));
#pragma unroll
        for (int j = 0; j < FB; ++j) asm volatile("" : "+v"(b[j]));
    }
    // the wave's slice K of the weight slot at byte offset sa and of the window; `pix`: this lane's address of its first slice
    template <int K> DEVFN void read(const unsigned (&fa)[4], unsigned sa, unsigned pix)
    {
        if constexpr (DG) {
            constexpr int ROW = FA * 64;   // bytes of a reduction row
#pragma unroll
            for (int i = 0; i < FA; ++i) {
                lo[i] = lds_read_tr<K * 16 * ROW>(fa[i] + sa);
                hi[i] = lds_read_tr<K * 16 * ROW + 4 * ROW>(fa[i] + sa);
            }
        } else
            a = lds_read16<0>(fa[K] + sa);
        const unsigned ad = pix ^ (K << 5);   // the swizzle is an exclusive-or of the chunk, a slice is two chunks
        b[0] = lds_read16<0>(ad);
        if constexpr (FB > 1) b[1] = lds_read16<4096>(ad);
        if constexpr (FB > 2) b[2] = lds_read16<8192>(ad);
        if constexpr (FB > 3) b[3] = lds_read16<12288>(ad);
    }
    DEVFN bf16x8 weights(int i) const
    {
        if constexpr (DG) return __builtin_bit_cast(bf16x8, u32x4{lo[i].x, lo[i].y, hi[i].x, hi[i].y});
        else return __builtin_bit_cast(bf16x8, a);
    }
};

// Backward-data with tiles of two fragments' width and height: the waves go in pairs that share 64 channels and take two of the four slices each.
// A wave's weights are then 32 reduction rows of 128 bytes instead of 64 of 64 (copies of 64-byte rows run at half the rate), and four
// fragment reads serve four matrix instructions instead of three two.
template <bool DG, int WA, int FB> constexpr int win_fa() { return DG && WA % 2 == 0 && FB == 2 ? 2 : 1; }

// SAVED (backward-data): dy counts where the saved output p.ymask is positive.  The window then goes through registers, dy and the saved output side by
// side, and is masked on its way to LDS: once per window, in the place of a pass over dy in memory and the launch of it.
// The kernel takes 5 - 16 % longer for it, the pass 2.8 us and 0.4 us per MB of dy (with it, us): 192 -> 64 on 48 x 48,
// 7 samples 17.4 -> 13.1, 128 -> 64 on 29 x 29, 14 samples 13.4 -> 10.0; all passes of 80 -> 192 on 73 x 73, 4 samples 64.5 -> 60.7.
template <bool DG, int WA, int CBP, int FB, bool SAVED>
__global__ __launch_bounds__(kThreads) void k_conv_win(const KArgs p, const WinArgs q)
{
#if __HIP_DEVICE_COMPILE__   // the host pass only needs the launch stub (and silently drops it when it sees this body)
    constexpr int TA = 32 * WA, TB = 32 * FB, G = kWaves / (WA * CBP), FA = win_fa<DG, WA, FB>(), SL = 4 / FA, WCH = WA / FA, KG = G * CBP * FA, IW = kMaxWindowCopies;
    static_assert(G * WA * CBP == kWaves, "twelve waves");
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const ConvGeom &g = p.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // four tap groups would meet the four SIMDs one to one, and the group with a tap more would be one SIMD's alone: each row of waves shifts by one
    const int grp = G == 4 ? (wave + wave / 4) % 4 : wave % G, wc = wave / G % WCH, sp = wave / G / WCH % FA, cbp = wave / G / WA;   // taps, channels, slices, channel block
    const int tile = logical_block(blockIdx.x, gridDim.x), tb = tile / p.tilesA, a0 = (tile - tb * p.tilesA) * TA, u0 = tb * TB;
    const int RS = g.R * g.S, RSC = RS * g.C, win_bytes = q.wrows * 128, rounds = (q.ncb + CBP - 1) / CBP;
    const int each = RS / G, more = RS - G * each, tap0 = grp * each + min(grp, more), nt = each + (grp < more ? 1 : 0);   // this wave's taps
    int *rowpix = reinterpret_cast<int *>(smem + kWeightBytes + 2 * CBP * win_bytes);   // [TB] output pixel of a tile row, -1 for none
    float *bias_lds = reinterpret_cast<float *>(rowpix + TB);                           // [TA]
    const unsigned lds0 = lds_offset(smem), lds_win = lds0 + kWeightBytes, lds_a = lds0 + wave * 2 * kSlot;
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(p.w, (size_t)g.K * RSC * 2), rs = make_rsrc(DG ? p.dy : p.x, (size_t)g.N * q.Hs * q.Ws * q.CR * 2);

    // slot -> image position: a few hundred slots behind a uniform first one; one scalar division, then reciprocals (exact below 2^21; win_args keeps P and HP under half of that)
    const float rP = 1.0f / (float)q.P, rHP = 1.0f / (float)q.HP;
    auto place = [&](int first, int row, int &n, int &h, int &w) {
        const int img = q.HP * q.P;
        int n0 = first / img, rem = first - n0 * img;
        if (rem < 0) { rem += img; --n0; }
        const int h0 = rem / q.P, w0 = rem - h0 * q.P + row, up = (int)(((float)w0 + 0.5f) * rP), h1 = h0 + up, un = (int)(((float)h1 + 0.5f) * rHP);
        n = n0 + un; h = h1 - un * q.HP; w = w0 - up * q.P;
    };
    // window copies: eight slots of 128 bytes each, copy 12 i + wave; chunk c of window row r sits at position c ^ ((r >> 1) & 7), which makes
    // 16 consecutive rows conflict-free wherever they start
    const int ncopies = q.wrows / 8, iw = (ncopies - wave + kWaves - 1) / kWaves, tail = q.CR - 64 * (q.ncb - 1);   // tail: channels of the last block
    unsigned voffW[IW];
#pragma unroll
    for (int i = 0; i < IW; ++i) {
        const int row = (i * kWaves + wave) * 8 + lane / 8, c = (lane % 8) ^ ((row >> 1) & 7);
        int n, h, w;
        place(u0 + q.first, row, n, h, w);
        voffW[i] = n >= 0 && n < g.N && h < q.Hs && w < q.Ws ? (unsigned)(((n * q.Hs + h) * q.Ws + w) * q.CR + c * 8) * 2u : OOR;
    }
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(SAVED ? p.ymask : p.dy, (size_t)g.N * q.Hs * q.Ws * q.CR * 2);
    constexpr int HELD = CBP > 1 ? 2 : 3;   // copies of a wave per window: LDS holds no more
    u32x4 hg[SAVED ? CBP * HELD : 1], hy[SAVED ? CBP * HELD : 1];
    auto issue_windows = [&](int round) {   // the CBP windows of a round; a channel block past the last is not read
#pragma unroll
        for (int b = 0; b < CBP; ++b) {
            const int cb = round * CBP + b;
            const unsigned dst = lds_win + ((round & 1) * CBP + b) * win_bytes + wave * 1024;
#pragma unroll
            for (int i = 0; i < (SAVED ? HELD : IW); ++i) {
                if (!SAVED && i >= iw) break;   // SAVED: always as many loads, those past the window's end out of range
                const int row = (i * kWaves + wave) * 8 + lane / 8, c = (lane % 8) ^ ((row >> 1) & 7);
                const bool out = cb >= q.ncb || (cb == q.ncb - 1 && c * 8 >= tail) || (SAVED && i >= iw);
                if constexpr (SAVED) {
                    hg[b * HELD + i] = __builtin_amdgcn_raw_buffer_load_b128(rs, out ? OOR : voffW[i], cb < q.ncb ? cb * 128 : 0, 0);
                    hy[b * HELD + i] = __builtin_amdgcn_raw_buffer_load_b128(ry, out ? OOR : voffW[i], cb < q.ncb ? cb * 128 : 0, 0);
                } else
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void)(size_t)(dst + i * kWaves * 1024), 16, out ? OOR : voffW[i], cb < q.ncb ? cb * 128 : 0, 0, 0);
            }
        }
    };
    auto store_windows = [&](int round) {   // SAVED: what issue_windows asked for
#pragma unroll
        for (int b = 0; b < CBP; ++b)
#pragma unroll
            for (int i = 0; i < HELD; ++i) {
                if (i >= iw) break;
                const u32x4 v = apply_mask(hg[b * HELD + i], hy[b * HELD + i]);
                asm volatile("ds_write_b128 %0, %1" ::"v"(lds_win + ((round & 1) * CBP + b) * win_bytes + (i * kWaves + wave) * 1024 + lane * 16), "v"(v) : "memory");
            }
    };
    // this wave's weights of one tap and channel block, four copies.  Forward: 32 rows (output channels) of 64 reduction channels; backward-data:
    // reduction rows of 32 FA input channels, for the transpose read (four 64-byte rows meet all banks, 128-byte rows are swizzled)
    unsigned voffA[4];
    bool inA[4];   // the copy's reduction channels exist in the last channel block
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (DG) {
            constexpr int CPR = FA * 4;   // chunks per row
            const int tl = i * (64 / CPR) + lane / CPR, t = sp * (64 / FA) + tl, col = a0 + wc * 32 * FA + ((lane % CPR) ^ (seg_swz<32 * FA>(tl) << 2)) * 8;
            voffA[i] = col < g.C ? ((unsigned)t * RSC + col) * 2u : OOR;
            inA[i] = t < tail;
        } else {
            const int row = i * 8 + lane / 8, c = (lane % 8) ^ ((row >> 1) & 7), k = a0 + wc * 32 + row;
            voffA[i] = k < g.K ? ((unsigned)k * RSC + c * 8) * 2u : OOR;
            inA[i] = c * 8 < tail;
        }
    }
    const int nsteps = cbp < q.ncb ? ((q.ncb - 1 - cbp) / CBP + 1) * nt : 0;
    int is = 0, is_cb = cbp, is_j = 0;   // the next step to copy: number, channel block, tap of this wave's
    auto issue_weights = [&]() {
        const bool last = is_cb == q.ncb - 1;
        const int tap = DG ? RS - 1 - (tap0 + is_j) : tap0 + is_j;
        const int soff = DG ? (is_cb * 64 * RSC + tap * g.C) * 2 : (tap * g.C + is_cb * 64) * 2;
        const unsigned dst = lds_a + (is & 1) * kSlot;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void)(size_t)(dst + i * 1024), 16, last && !inA[i] ? OOR : voffA[i], soff, 0, 0);
        ++is;
        if (++is_j == nt) { is_j = 0; is_cb += CBP; }
    };
    issue_windows(0);
    if (nsteps > 0) issue_weights();
    if (nsteps > 1) issue_weights();

    if (tid < TB) {
        int n, h, w;
        place(u0, tid, n, h, w);
        rowpix[tid] = n < g.N && h < q.Hd && w < q.Wd ? (n * q.Hd + h) * q.Wd + w : -1;
    }
    if (!DG && (p.flags & KF_BIAS) && tid < TA) bias_lds[tid] = a0 + tid < p.rowsA ? p.bias[a0 + tid] : 0.f;

    f32x16 acc[FA][FB];
#pragma unroll
    for (int i = 0; i < FA; ++i)
#pragma unroll
        for (int j = 0; j < FB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    unsigned fa[4];
    if constexpr (DG) {
        const int i16 = lane & 15, tl = (lane >> 5) * 8 + (i16 >> 2), cl = ((lane >> 4) & 1) * 16 + (i16 & 3) * 4;
#pragma unroll
        for (int i = 0; i < FA; ++i) fa[i] = lds_a + tl * FA * 64 + ((i ^ seg_swz<32 * FA>(tl)) << 6) + cl * 2;
    } else {
        const int r = lane & 31;
#pragma unroll
        for (int k = 0; k < 4; ++k) fa[k] = lds_a + r * 128 + (((2 * k + (lane >> 5)) ^ ((r >> 1) & 7)) << 4);
    }
    Frags<DG, FA, FB> s0, s1;
    auto multiply = [&](const Frags<DG, FA, FB> &s) {
#pragma unroll
        for (int i = 0; i < FA; ++i)
#pragma unroll
            for (int j = 0; j < FB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(s.weights(i), __builtin_bit_cast(bf16x8, s.b[j]), acc[i][j], 0, 0, 0);
    };
    // this lane's address of a tap's first slice in the window at `win`
    auto pixels = [&](unsigned win, int off) {
        const unsigned row = (unsigned)((lane & 31) + off);
        return win + row * 128u + ((((unsigned)lane >> 5) ^ (unsigned)(2 * SL * sp) ^ ((row >> 1) & 7u)) << 4);
    };

    if constexpr (SAVED) {
        store_windows(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    // Copies complete in order.  Behind the weights of step s the wave has issued at most those of step s + 1 and, in a round's first two
    // steps, the next round's windows (issued at the round's start).
    const int r0 = tap0 / g.S, c0 = tap0 - r0 * g.S;
    const int iwb = SAVED ? 0 : iw * CBP;   // loads to registers are the compiler's to count: the waits below take them as landed, which costs little
    wait_copies(4 * min(2, nsteps));
    __builtin_amdgcn_s_barrier();
    int s = 0;
    for (int round = 0; round < rounds; ++round) {
        const bool next = round + 1 < rounds;
        if constexpr (SAVED) wait_copies(s + 1 < nsteps ? 4 : 0);   // the weights of step s, before loads that are not counted
        if (next) issue_windows(round + 1);
        if (round * CBP + cbp < q.ncb && nt > 0) {
            const unsigned win = lds_win + ((round & 1) * CBP + cbp) * win_bytes;
            int tr = r0, ts = c0;
            if constexpr (!SAVED) wait_copies((s + 1 < nsteps ? 4 : 0) + (next ? iwb : 0));
            s0.template read<0>(fa, (s & 1) * kSlot, pixels(win, tr * q.P + ts));
            for (int j = 0; j < nt; ++j, ++s) {
                const unsigned sa = (s & 1) * kSlot, pix = pixels(win, tr * q.P + ts);
                if (++ts == g.S) { ts = 0; ++tr; }
                s0.landed();
                s1.template read<1>(fa, sa, pix);
                multiply(s0);
                s1.landed();
                if constexpr (SL == 4) {
                    s0.template read<SL == 4 ? 2 : 0>(fa, sa, pix);
                    multiply(s1);
                    s0.landed();
                    s1.template read<SL == 4 ? 3 : 0>(fa, sa, pix);
                    multiply(s0);
                    s1.landed();
                }
                // in a round's last step: the loads have had the round to land, and what is younger is waited for below in any case
                if constexpr (SAVED)
                    if (next && j + 1 == nt) store_windows(round + 1);
                // the slot has been read: it takes step s + 2
                if (s + 2 < nsteps) issue_weights();
                if (j + 1 < nt) {
                    wait_copies((s + 2 < nsteps ? 4 : 0) + (j == 0 && next ? iwb : 0));
                    s0.template read<0>(fa, sa ^ kSlot, pixels(win, tr * q.P + ts));
                }
                multiply(s1);
            }
        }
        else if (SAVED && next) store_windows(round + 1);
        if (next) {
            if constexpr (SAVED) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            wait_copies(4 * max(0, min(min(2, nt), nsteps - s + nt - 2)));   // the next round's windows have landed: at most this many weight copies are younger
            __builtin_amdgcn_s_barrier();
        }
    }

    // Epilogue: the saved input of a masked tile is requested first; then the groups' sums through LDS
    __syncthreads();
    constexpr int CPR = TA / 8, TOTAL = TB * CPR, ITERS = (TOTAL + kThreads - 1) / kThreads, LSO = TA + 8;
    const size_t out_bytes = (size_t)p.rowsB * p.rowsA * 2;
    const __amdgpu_buffer_rsrc_t rin = make_rsrc(p.x, out_bytes), rout = make_rsrc(p.out, out_bytes);
    unsigned voffO[ITERS];
#pragma unroll
    for (int i = 0; i < ITERS; ++i) {
        const int id = tid + i * kThreads, rp = id < TOTAL ? rowpix[id / CPR] : -1, col = a0 + (id % CPR) * 8;
        voffO[i] = rp >= 0 && col < p.rowsA ? ((unsigned)rp * (unsigned)p.rowsA + col) * 2u : OOR;
    }
    const bool mask = DG && (p.flags & KF_MASK_IN);
    u32x4 xm[ITERS];
    if (mask)
#pragma unroll
        for (int i = 0; i < ITERS; ++i) xm[i] = __builtin_amdgcn_raw_buffer_load_b128(rin, voffO[i], 0, 0);
    // Every wave leaves its sums, two fragments at a time (one, of an odd number); all threads add the groups' in order and stage the finished values.
    const int kg = (cbp * FA + sp) * G + grp;
    constexpr int NF = FA * FB, FP = NF % 2 != 0 ? 1 : 2, QUADS = WCH * FP * 4 * 64;   // fragments per pass, groups of four values per pass
    f32x4 *sum = reinterpret_cast<f32x4 *>(smem);                                  // [group][channel wave][fragment][quad][lane]
    bf16_t *stage = reinterpret_cast<bf16_t *>(smem + KG * QUADS * 16);
#pragma unroll
    for (int f0 = 0; f0 < NF; f0 += FP) {
        if (f0 > 0) __syncthreads();
#pragma unroll
        for (int f = 0; f < FP; ++f)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const f32x16 &c = acc[(f0 + f) / FB][(f0 + f) % FB];
                sum[kg * QUADS + ((wc * FP + f) * 4 + v) * 64 + lane] = f32x4{c[4 * v], c[4 * v + 1], c[4 * v + 2], c[4 * v + 3]};
            }
        __syncthreads();
        for (int id = tid; id < QUADS; id += kThreads) {
            f32x4 o = sum[id];
#pragma unroll
            for (int k = 1; k < KG; ++k) o += sum[k * QUADS + id];
            const int l = id & 63, v = (id >> 6) & 3, f = f0 + (id >> 8) % FP, w = (id >> 8) / FP;
            const int ch = (w * FA + f / FB) * 32 + 8 * v + 4 * (l >> 5), row = f % FB * 32 + (l & 31);
            if (!DG && (p.flags & KF_BIAS)) o += *reinterpret_cast<const f32x4 *>(bias_lds + ch);
            if (!DG && (p.flags & KF_RELU)) { o.x = fmaxf(o.x, 0.f); o.y = fmaxf(o.y, 0.f); o.z = fmaxf(o.z, 0.f); o.w = fmaxf(o.w, 0.f); }
            *reinterpret_cast<u32x2 *>(stage + row * LSO + ch) = u32x2{pack_bf16(o.x, o.y), pack_bf16(o.z, o.w)};
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITERS; ++i) {
        const int id = min(tid + i * kThreads, TOTAL - 1);   // past the tile the offset is out of range
        u32x4 v = *reinterpret_cast<const u32x4 *>(stage + (id / CPR) * LSO + (id % CPR) * 8);
        if (mask) v = apply_mask(v, xm[i]);
        __builtin_amdgcn_raw_buffer_store_b128(v, rout, voffO[i], 0, 0);
    }
#endif
}

typedef void (*WinFn)(const KArgs, const WinArgs);
struct WinVariant { int WA, CBP, FB; };
const WinVariant kWin[] = {{4, 1, 4}, {2, 1, 2}, {1, 2, 1}, {2, 2, 2}, {4, 1, 2}, {2, 1, 4}, {3, 1, 2}, {3, 1, 3}, {3, 1, 4}};
constexpr int kNumWin = 9;
template <bool DG, bool SAVED = false> WinFn pick(int v)
{
    switch (v) {
    case 0: return k_conv_win<DG, 4, 1, 4, SAVED>;
    case 1: return k_conv_win<DG, 2, 1, 2, SAVED>;
    case 2: return k_conv_win<DG, 1, 2, 1, SAVED>;
    case 3: return k_conv_win<DG, 2, 2, 2, SAVED>;
    case 4: return k_conv_win<DG, 4, 1, 2, SAVED>;
    case 5: return k_conv_win<DG, 2, 1, 4, SAVED>;
    case 6: return k_conv_win<DG, 3, 1, 2, SAVED>;
    case 7: return k_conv_win<DG, 3, 1, 3, SAVED>;
    default: return k_conv_win<DG, 3, 1, 4, SAVED>;
    }
}

// the slot layout of a layer and the LDS it takes; false if the kernel does not run it
bool win_args(const ConvGeom &g, bool dg, const WinVariant &d, WinArgs *q, long long *slots, size_t *lds)
{
    const int RS = g.R * g.S, TA = 32 * d.WA, TB = 32 * d.FB;
    if (g.sh != 1 || g.sw != 1 || g.C % 8 != 0 || g.K % 8 != 0 || RS < 3 || RS > 32) return false;
    // 32-bit offsets; a slot without a source pixel is marked by an offset past any tensor
    const long long in = (long long)g.N * g.H * g.W * g.C * 2, out = (long long)g.N * g.Ho * g.Wo * g.K * 2;
    if (in >= 0x7fffffffLL || out >= 0x7fffffffLL || (long long)g.K * RS * g.C * 2 >= 0x7fffffffLL) return false;
    const int pw = dg ? g.S - 1 - g.pw : g.pw, ph = dg ? g.R - 1 - g.ph : g.ph;
    q->Hs = dg ? g.Ho : g.H; q->Ws = dg ? g.Wo : g.W; q->Hd = dg ? g.H : g.Ho; q->Wd = dg ? g.W : g.Wo;
    q->P = q->Ws + (pw > 0 ? pw : 0);
    if (q->Wd > q->P) q->P = q->Wd;
    q->HP = q->Hs + (ph > 0 ? ph : 0);
    if (q->Hd > q->HP) q->HP = q->Hd;
    q->first = -ph * q->P - pw;
    q->CR = dg ? g.K : g.C;
    q->ncb = (q->CR + 63) / 64;
    *slots = (long long)g.N * q->HP * q->P;
    const long long wrows = (TB + (long long)(g.R - 1) * q->P + g.S - 1 + 7) / 8 * 8;
    if (q->P >= 1 << 20 || q->HP >= 1 << 20) return false;   // the kernel divides by reciprocals
    if (*slots >= 0x3fffffffLL || wrows > (d.CBP > 1 ? 2 : kMaxWindowCopies) * kWaves * 8) return false;   // no plan that LDS holds
    q->wrows = (int)wrows;
    const int sums = kWaves * (d.FB % 2 != 0 ? 1 : 2) * kSlot + TB * (TA + 8) * 2, tiles = kWeightBytes + 2 * d.CBP * q->wrows * 128, extra = (TB + TA) * 4;
    if (sums > tiles || tiles + extra > kLdsBytes) return false;   // the row map and the bias behind the tiles outlive the sums
    *lds = (size_t)tiles + extra;
    return true;
}

}  // namespace

hipError_t win_init()
{
    for (int v = 0; v < kNumWin; ++v)
        for (WinFn k : {pick<false>(v), pick<true>(v), pick<true, true>(v)}) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

bool win_plan(const ConvGeom &g, int pass, int variant, GemmPlan *pl)
{
    WinArgs q;
    long long slots;
    size_t lds;
    if (variant < 0 || variant >= kNumWin || pass == PASS_WGRAD || !win_args(g, pass == PASS_DGRAD, kWin[variant], &q, &slots, &lds)) return false;
    const WinVariant &d = kWin[variant];
    pl->variant = variant; pl->TA = 32 * d.WA; pl->TB = 32 * d.FB; pl->BK = 64;
    pl->vecA = pl->vecB = true; pl->fast = true; pl->dma = true; pl->halo = false; pl->phase = pl->fill = false; pl->wstrip = false; pl->wwin = false; pl->win = true;
    pl->tilesA = ((pass == PASS_FWD ? g.K : g.C) + pl->TA - 1) / pl->TA;
    pl->tilesB = (int)((slots + pl->TB - 1) / pl->TB);
    pl->steps_total = pl->steps_per_split = g.R * g.S * q.ncb;
    pl->splits = 1;
    return true;
}

bool win_work(const ConvGeom &g, int pass, int variant, int *rounds, int *rows)
{
    WinArgs q;
    long long slots;
    size_t lds;
    if (!win_args(g, pass == PASS_DGRAD, kWin[variant], &q, &slots, &lds)) return false;
    *rounds = (q.ncb + kWin[variant].CBP - 1) / kWin[variant].CBP;
    *rows = kWin[variant].CBP * q.wrows;
    return true;
}

void win_kernel_name(int pass, const GemmPlan &pl, bool saved, char *name, size_t name_bytes)
{
    const WinVariant &d = kWin[pl.variant];
    snprintf(name, name_bytes, "k_conv_win<%s, %d, %d, %d, %s>", pass == PASS_DGRAD ? "true" : "false", d.WA, d.CBP, d.FB, pass == PASS_DGRAD && saved ? "true" : "false");
}

hipError_t win_launch(const ConvArgs &a, hipStream_t st)
{
    KArgs p;
    WinArgs q;
    long long slots;
    size_t lds;
    const bool dg = a.pass == PASS_DGRAD;
    if (!win_args(a.g, dg, kWin[a.plan.variant], &q, &slots, &lds)) return hipErrorInvalidValue;
    p.g = a.g;
    p.rowsA = dg ? a.g.C : a.g.K; p.rowsB = a.g.N * q.Hd * q.Wd; p.red = a.g.R * a.g.S * q.CR;
    p.tilesA = a.plan.tilesA; p.tilesB = a.plan.tilesB;
    p.steps_total = p.steps_per_split = a.plan.steps_total; p.splits = 1;
    p.flags = a.flags;
    p.x = a.x; p.w = a.w; p.dy = a.dy; p.ymask = dg ? a.ymask : nullptr; p.bias = a.bias; p.out = a.out; p.partial = nullptr; p.dbp = nullptr;
    p.tickets = nullptr;
    p.ph_on = 0;
    const WinFn kern = !dg ? pick<false>(a.plan.variant) : p.ymask != nullptr ? pick<true, true>(a.plan.variant) : pick<true>(a.plan.variant);
    hipLaunchKernelGGL(kern, dim3((unsigned)(p.tilesA * p.tilesB)), dim3(kThreads), lds, st, p, q);
    dp_trace_main_kernel_done(st);
    return hipGetLastError();
}
