// Filter gradient of unit-stride layers with all taps of a block fed from one window of x.
//
// dW[k][r][s][c] = sum over pixels m of dy[m][k] * x[m + (r - pad_h, s - pad_w)][c] (pairs outside the image contribute nothing).
// The reduction runs over pixel SLOTS: an image row takes P = W + pad_w of them and an image HP = H + pad_h slot rows (or as many as
// dy needs), the slots behind a row's and an image's last pixel hold zeros.  With that padding tap (r, s) of slot u is slot
// u + (r - pad_h) * P + (s - pad_w) for every pixel, taps outside the image meet a zero slot, and no operand needs a mask.
// A block owns 64 output channels, 32 input channels and up to nine taps.  A chunk of the reduction is T slots: dy
// and the window of x that the taps reach from there (T + span slots, 64 bytes each), copied once for all taps, where a kernel with one
// column tile per tap copies every x slot once per tap: 128 + 64 (T + span) / T bytes per slot for 64 x 288 outputs, against 384 for 64 x 128.
// Twelve waves, three per SIMD: wave (g, pg) multiplies every fourth 16-slot slice (pg) by a third of the taps (g), 2 x 3 tiles of
// 32 x 32 in 96 accumulators; five fragment reads serve six matrix instructions.  The four slice groups' sums meet in LDS at the end, in
// group order, so that a block needs no partials in memory for them: a 512 x 512 x 3 x 3 gradient fills the chip with two splits.
// Measured with the reduction kernel (us; the pipelined tiles with one column tile per tap before): 512 -> 512 on 28 x 28, 8 samples 47.4 -> 40.5,
// 32 samples 124 -> 112; 128 -> 128 on 112 x 112, 8 samples 48.0 -> 39.1, 32 samples 150 -> 112 (1.06 PFLOP/s).  What is left (counters, four layers of
// 14 x 14 to 112 x 112 at 8 samples): the matrix cores are busy for 0.50 of the time, the waves wait at counters and barriers for 0.40 of theirs; and the fixed part of the fitted price, 6.8 us (first copies, the slice groups' sums, the stores), which is why short layers keep the other kernels.
// Both operands are reduction-major in LDS and go through the LDS transpose read; x rows are 64 bytes, so the four rows one read touches
// are 256 consecutive bytes wherever a tap starts, and the taps differ by an address offset only.
// Output: fp32 dW, or fp32 partials [split][k][r][s][c] for the split-reduce kernel.
#include "dma_common.h"
#include <cstdio>

namespace {

constexpr int kWaves = 12, kTables = 4, kMaxStages = 3, kTapBlocks = 4, kTapsPerBlock = 9;
constexpr int dy_copies(int T) { return T / 8; }   // copies of one KB
constexpr int lane_copies(int T) { return T == 128 ? 5 : 6; }   // most copies of a wave per chunk
constexpr int kLdsBytes = 160 * 1024, kSumBytes = 3 * 3 * 4 * 3 * 64 * 16;   // the sums of three slice groups for one half of the tiles

struct WinGeom {
    int P, HP;                        // slots per image row, slot rows per image
    int tilesC, tapBlocks;
    int nxi, ns;                      // x copies (16 slots each) per chunk, stages
    int dn, dh, dw;                   // T slots as images, slot rows and slots
    int first[kTapBlocks];            // first slot of the x window of a chunk that starts at slot 0, per tap block
    int tap[kTapBlocks + 1];          // first tap of a block
    short at[kTapBlocks * kTapsPerBlock];   // the slot of a tap in its block's window
};

constexpr int ROWA = 128, ROWX = 64;   // bytes per slot in LDS

// the fragments of one 16-slot slice: two of dy, one of x per tap
template <int NTP, bool ROW> struct Slice {
    u32x2 alo[2], ahi[2], blo[NTP], bhi[NTP];
    template <int J> DEVFN void read(const unsigned (&fa)[2], const unsigned (&fx)[3], unsigned sb)   // slice J of the stage at byte offset sb
    {
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            alo[f] = lds_read_tr<J * 64 * ROWA>(fa[f] + sb);
            ahi[f] = lds_read_tr<J * 64 * ROWA + 4 * ROWA>(fa[f] + sb);
        }
#pragma unroll
        for (int j = 0; j < NTP; j += ROW ? 2 : 1) {
            blo[j] = lds_read_tr<J * 64 * ROWX>(fx[j] + sb);
            bhi[j] = lds_read_tr<J * 64 * ROWX + 4 * ROWX>(fx[j] + sb);
        }
    }
    DEVFN void landed()
    {
        asm volatile("s_waitcnt lgkmcnt(0)");
#pragma unroll
        for (int f = 0; f < 2; ++f) { asm volatile("" : "+v"(alo[f])); asm volatile("" : "+v"(ahi[f])); }
#pragma unroll
        for (int j = 0; j < NTP; j += ROW ? 2 : 1) { asm volatile("" : "+v"(blo[j])); asm volatile("" : "+v"(bhi[j])); }
    }
    DEVFN bf16x8 x(int j) const   // ROW: the middle tap's eight pixels are one behind the first tap's, the last of them is in the third tap's
    {
        if (ROW && j == 1)
            return __builtin_bit_cast(bf16x8, u32x4{__builtin_amdgcn_alignbit(blo[0].y, blo[0].x, 16), __builtin_amdgcn_alignbit(bhi[0].x, blo[0].y, 16),
                                                    __builtin_amdgcn_alignbit(bhi[0].y, bhi[0].x, 16), __builtin_amdgcn_alignbit(bhi[2].y, bhi[0].y, 16)});
        return __builtin_bit_cast(bf16x8, u32x4{blo[j].x, blo[j].y, bhi[j].x, bhi[j].y});
    }
};

// dW[row .. row + 3][tap][col] from the slots first .. last - 1, only the pixels that the tap pairs: what the product does not give where a pixel is
// infinite or NaN.  Row by row of the image, so that the sums stay as short as the product's; a sum that is all NaN stays so.  Costs
// what a plain loop costs, and only where the product is NaN.
DEVFN f32x4 sum_in_range(const KArgs &p, const WinGeom &q, int first, int last, int row, int tap, int col)
{
    const ConvGeom &g = p.g;
    const int r = tap / g.S - g.ph, s = tap % g.S - g.pw, line0 = first / q.P;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    int n = line0 / q.HP, h = line0 - n * q.HP;
    for (int at = line0 * q.P; at < last && n < g.N; at += q.P) {   // `at`: the slot of the row's first pixel
        const int hx = h + r;
        if (h < g.Ho && hx >= 0 && hx < g.H) {
            const int w0 = max(max(0, first - at), -s), w1 = min(min(g.Wo, last - at), g.W - s);
            const bf16_t *dy = p.dy + ((size_t)(n * g.Ho + h) * g.Wo) * g.K + row, *x = p.x + ((size_t)(n * g.H + hx) * g.W + s) * g.C + col;
            f32x4 line = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
            for (int w = w0; w < w1; ++w) {
                const u32x2 d = *reinterpret_cast<const u32x2 *>(dy + (size_t)w * g.K);
                const float v = __uint_as_float((unsigned)*reinterpret_cast<const unsigned short *>(x + (ptrdiff_t)w * g.C) << 16);
                line.x = fmaf(__uint_as_float(d.x << 16), v, line.x); line.y = fmaf(__uint_as_float(d.x & 0xffff0000u), v, line.y);
                line.z = fmaf(__uint_as_float(d.y << 16), v, line.z); line.w = fmaf(__uint_as_float(d.y & 0xffff0000u), v, line.w);
            }
            sum += line;
            if (sum.x != sum.x && sum.y != sum.y && sum.z != sum.z && sum.w != sum.w) break;
        }
        if (++h == q.HP) { h = 0; ++n; }
    }
    return sum;
}

struct Arguments { KArgs p; WinGeom q; };   // the kernel's arguments as they lie in memory

// the sums of this lane that `nan` marks (bit 3 f + j: half f of the channels, tap j of the wave) once more
template <int T> DEVFN void sum_again(const KArgs &p, const WinGeom &q, unsigned nan, int grp, int pg, int lane)
{
    const ConvGeom &g = p.g;
    const int id = logical_block(blockIdx.x, gridDim.x), ncol = q.tilesC * q.tapBlocks, tiles = p.tilesA * ncol;
    const int split = id / tiles, tile = id - split * tiles, rest = tile / p.tilesA, ct = rest % q.tilesC, tb = rest / q.tilesC;
    const int first = split * p.steps_per_split, steps = min(p.steps_per_split, p.steps_total - first);
    const int ntap = q.tap[tb + 1] - q.tap[tb], each = ntap / 3, tap = q.tap[tb] + grp * each + min(grp, ntap - 3 * each);
    float *dst = p.splits > 1 ? p.partial + (size_t)split * p.rowsA * p.rowsB : reinterpret_cast<float *>(p.out);
    for (; nan != 0; nan &= nan - 1) {
        const int e = __ffs(nan) - 1, f = e / 3, t = tap + e - 3 * f, row = (tile - rest * p.tilesA) * 64 + f * 32 + 8 * pg + 4 * (lane >> 5), col = ct * 32 + (lane & 31);
        if (col >= g.C || row >= p.rowsA) continue;
        const f32x4 v = sum_in_range(p, q, first * T, (first + steps) * T, row, t, col);
#pragma unroll
        for (int i = 0; i < 4; ++i) dst[(size_t)(row + i) * p.rowsB + (size_t)t * g.C + col] = v[i];
    }
}

template <int T, bool DB, bool ROW>
__global__ __launch_bounds__(64 * kWaves) void k_wgrad_win(const KArgs p, const WinGeom q)
{
    constexpr int A_BYTES = T * ROWA, QM = lane_copies(T), JN = T / 64, DYI = dy_copies(T);
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const ConvGeom &g = p.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), grp = wave % 3, pg = wave / 3;
    // split-major: an XCD gets neighbouring tiles of one split (or whole splits), whose blocks read the same slots
    const int id = logical_block(blockIdx.x, gridDim.x), ncol = q.tilesC * q.tapBlocks, tiles = p.tilesA * ncol;
    const int split = id / tiles, tile = id - split * tiles, rest = tile / p.tilesA, ct = rest % q.tilesC, tb = rest / q.tilesC;
    const int k0 = (tile - rest * p.tilesA) * 64, c0 = ct * 32;
    const int kbeg = split * p.steps_per_split, nsteps = min(p.steps_per_split, p.steps_total - kbeg);
    // this wave's taps: a third of the tap block's, which has at least three
    const int tap0 = q.tap[tb], ntap = q.tap[tb + 1] - tap0, each = ntap / 3, more = ntap - 3 * each;
    const int tap = tap0 + grp * each + min(grp, more), nt = each + (grp < more ? 1 : 0);
    const int xfirst = q.first[tb];

    // Copies of a chunk: dy first (8 slots of 128 bytes each), then x (16 slots of 64 bytes), dealt over the waves; copy i fills the
    // stage's i-th KB.  Where a slot's data lies is worked out once per slot and chunk: thread t < T follows dy slot t, the threads behind
    // them the slots of the x window, and leaves the byte offset (all ones for a slot without data) in a table that the copying lanes read.
    // Slots before the first and behind the last image are out of the tensor's range by their offset.
    const __amdgpu_buffer_rsrc_t rdy = make_rsrc(p.dy, (size_t)p.red * g.K * 2), rx = make_rsrc(p.x, (size_t)g.N * g.H * g.W * g.C * 2);
    const int cnt = (DYI + q.nxi - wave + kWaves - 1) / kWaves, entries = T + q.nxi * 16;
    const unsigned lds0 = lds_offset(smem), stage_bytes = (unsigned)(DYI + q.nxi) * 1024u, ring = q.ns * stage_bytes, tab0 = lds0 + ring;
    const unsigned tab_bytes = (unsigned)entries * 4u, tab_ring = kTables * tab_bytes;
    const bool my_dy = wave < T / 64;
    const int Hk = my_dy ? g.Ho : g.H, Wk = my_dy ? g.Wo : g.W, E = (my_dy ? g.K : g.C) * 2;
    const unsigned mv_hw = (unsigned)q.dh << 16 | (unsigned)q.dw, row_hw = 0x10000u - (unsigned)q.P, img_hw = (unsigned)q.HP << 16;
    const unsigned mv_off = (unsigned)((q.dn * Hk + q.dh) * Wk + q.dw) * E, row_off = (unsigned)(Wk - q.P) * E, img_off = (unsigned)((Hk - q.HP) * Wk) * E;
    unsigned hw, off;   // slot row * 65536 + slot within it; byte offset
    {
        // the first slot's position by scalar division, this thread's few hundred slots behind it by the reciprocal (exact below 2^21)
        const int first = kbeg * T + (my_dy ? 0 : xfirst), img = q.HP * q.P;
        int n = first / img, rem = first - n * img;
        if (rem < 0) { rem += img; --n; }
        const int h0 = rem / q.P, w0 = rem - h0 * q.P + (my_dy ? tid : tid - T);
        const int up = (int)(((float)w0 + 0.5f) * (1.0f / (float)q.P)), w = w0 - up * q.P, h1 = h0 + up;
        const int un = (int)(((float)h1 + 0.5f) * (1.0f / (float)q.HP)), h = h1 - un * q.HP;
        hw = (unsigned)h << 16 | (unsigned)w;
        off = (unsigned)((((n + un) * Hk + h) * Wk + w) * E);
    }
    auto fill_table = [&](unsigned tb_) {   // the next chunk's entries at byte offset tb_ of the tables
        const unsigned e = (hw & 0xffffu) < (unsigned)Wk && hw < (unsigned)Hk << 16 ? off : OOR;
        if (tid < entries) asm volatile("ds_write_b32 %0, %1" ::"v"(tab0 + tb_ + tid * 4u), "v"(e) : "memory");
        hw += mv_hw;
        const bool c1 = (hw & 0xffffu) >= (unsigned)q.P;
        hw += c1 ? row_hw : 0u;
        const bool c2 = hw >= img_hw;
        hw -= c2 ? img_hw : 0u;
        off += mv_off + (c1 ? row_off : 0u) + (c2 ? img_off : 0u);
    };
    // 128-byte rows: the second 64-byte segment comes first in slots 2 and 3 of four, so that the four slots of a transpose read meet all banks
    const int col_dy = k0 + ((lane % 8) ^ ((lane >> 4 & 1) << 2)) * 8, col_x = c0 + (lane % 4) * 8;
    const unsigned add_dy = col_dy < g.K ? col_dy * 2u : OOR, add_x = col_x < g.C ? col_x * 2u : OOR;
    const unsigned my_tab_dy = tab0 + (wave * 8 + lane / 8) * 4, my_tab_x = tab0 + (T + (wave - DYI) * 16 + lane / 4) * 4;
    auto is_dy = [&](int i) { return (i + 1) * kWaves <= DYI || (i * kWaves < DYI && wave < DYI - i * kWaves); };
    unsigned src[QM];
    auto read_table = [&](unsigned tb_) {
#pragma unroll
        for (int i = 0; i < QM; ++i) {
            if (i >= cnt) break;
            const unsigned at = is_dy(i) ? my_tab_dy + i * kWaves * 32 : my_tab_x + i * kWaves * 64;
            asm volatile("ds_read_b32 %0, %1" : "=v"(src[i]) : "v"(at + tb_));
        }
    };
    auto issue = [&](unsigned sb) {   // copies of the chunk whose table entries have been read into the stage at byte offset sb
        unsigned dst = lds0 + sb + wave * 1024;
#pragma unroll
        for (int i = 0; i < QM; ++i, dst += kWaves * 1024) {
            if (i >= cnt) break;
            asm volatile("" : "+v"(src[i]));
            if (is_dy(i)) dma16(rdy, dst, __builtin_elementwise_add_sat(src[i], add_dy));
            else dma16(rx, dst, __builtin_elementwise_add_sat(src[i], add_x));
        }
    };

    f32x16 acc[2][3];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[f][j][v] = 0.f;
    // bias gradient: the column sums of the two dy fragments belong to the first two column tiles' first waves (or, with a single column
    // tile, to its first two), four slice groups each
    const int dbf = !DB ? -1 : rest == 0 && grp == 0 ? 0 : (ncol > 1 ? rest == 1 && grp == 0 : grp == 1) ? 1 : -1;
    f32x4 accdb = {0.f, 0.f, 0.f, 0.f};
    unsigned db_one = __builtin_bit_cast(u32x4, colsum_selector(lane)).x;

    // transpose reads: lane l points at slot 16 * pg + 8 * (l >> 5) + (l & 15) / 4 (and four slots further for the second half), channels
    // 16 * ((l >> 4) & 1) + 4 * (l & 3) .. +3; the second slice of the wave is 64 slots further
    unsigned fa[2], fx[3];
    {
        const int i16 = lane & 15, t = pg * 16 + (lane >> 5) * 8 + (i16 >> 2), cl = ((lane >> 4) & 1) * 16 + (i16 & 3) * 4;
#pragma unroll
        for (int f = 0; f < 2; ++f) fa[f] = lds0 + t * ROWA + ((f ^ ((t >> 1) & 1)) << 6) + cl * 2;
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            fx[j] = lds0 + A_BYTES + (t + q.at[tap + min(j, nt - 1)]) * ROWX + cl * 2;
        }
    }

    // `taps` of the three tap tiles are in use
    unsigned nan = 0;   // sums with a NaN: bit 3 f + j
    auto run = [&](auto taps) {
        constexpr int NTP = decltype(taps)::value;
        Slice<NTP, ROW> s0, s1;   // the wave's two slices of a chunk
        auto multiply = [&](const Slice<NTP, ROW> &s) {
            bf16x8 a[2];
#pragma unroll
            for (int f = 0; f < 2; ++f) a[f] = __builtin_bit_cast(bf16x8, u32x4{s.alo[f].x, s.alo[f].y, s.ahi[f].x, s.ahi[f].y});
#pragma unroll
            for (int jj = 0; jj < NTP; ++jj) {
                const int j = ROW ? (jj * 2) % 3 : jj;   // the middle tap last: its operand is made meanwhile
                const bf16x8 b = s.x(j);
#pragma unroll
                for (int f = 0; f < 2; ++f) acc[f][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[f], b, acc[f][j], 0, 0, 0);
            }
            if (DB && dbf >= 0) {
                asm volatile("" : "+v"(db_one));   // the operand's four equal words are made here: kept, they would cost three more registers
                const bf16x8 sel = __builtin_bit_cast(bf16x8, u32x4{db_one, db_one, db_one, db_one});
                if (dbf == 0) accdb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], sel, accdb, 0, 0, 0);
                else accdb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], sel, accdb, 0, 0, 0);
            }
        };
        static_assert(JN % 2 == 0, "the two fragment buffers alternate over the slices");

        // Every stage is filled ahead; the hand-over to the next chunk comes before the last slice is multiplied: by then the wave has read
        // all it needs of the stage, which takes chunk i + ns.  The tables are one chunk further.
        for (int s = 0; s <= q.ns; ++s) fill_table(s * tab_bytes);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        for (int s = 0; s < q.ns; ++s)
            if (s < nsteps) {
                read_table(s * tab_bytes);
                asm volatile("s_waitcnt lgkmcnt(0)");
                issue(s * stage_bytes);
            }
        wait_copies(min(q.ns - 1, nsteps - 1) * cnt);
        __builtin_amdgcn_s_barrier();
        s0.template read<0>(fa, fx, 0u);
        unsigned sb = 0, tb_ = q.ns * tab_bytes;   // the stage of chunk i, the table of chunk i + ns
        for (int i = 0; i < nsteps; ++i) {
            const unsigned sn = sb + stage_bytes == ring ? 0u : sb + stage_bytes, tn = tb_ + tab_bytes == tab_ring ? 0u : tb_ + tab_bytes;
            const bool more_copies = i + q.ns < nsteps;
            for_constant<JN / 2>([&](auto pair) {
                constexpr int J = 2 * decltype(pair)::value;
                s0.landed();
                s1.template read<J + 1>(fa, fx, sb);
                multiply(s0);
                s1.landed();
                if constexpr (J + 2 < JN) s0.template read<J + 2 < JN ? J + 2 : 0>(fa, fx, sb);
                else if (i + 1 < nsteps) {
                    wait_copies((min(i + q.ns, nsteps) - i - 2) * cnt);   // chunk i + 1 has landed, younger ones may be in flight
                    __builtin_amdgcn_s_barrier();
                    s0.template read<0>(fa, fx, sn);
                    if (more_copies) read_table(tb_);
                }
                multiply(s1);
            });
            if (more_copies) {
                fill_table(tn);   // done before the next barrier: the wait below and the one for the next slice cover it
                s0.landed();
                issue(sb);
            }
            sb = sn;
            tb_ = tn;
        }

        // The slice groups' sums: group pg finishes accumulators 4 pg .. 4 pg + 3 of every tile (rows 8 pg + 4 (l >> 5) + 0..3), adding
        // in group order; one half of the output channels at a time.
        f32x4 *sum = reinterpret_cast<f32x4 *>(smem);
        float *dst = (p.splits > 1 ? p.partial + (size_t)split * p.rowsA * p.rowsB : reinterpret_cast<float *>(p.out));
        const int col = c0 + (lane & 31);
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            __syncthreads();
#pragma unroll
            for (int j = 0; j < NTP; ++j)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq)
                    if (gq != pg)
                        sum[(((grp * 3 + j) * 4 + gq) * 3 + (pg < gq ? pg : pg - 1)) * 64 + lane] =
                            f32x4{acc[f][j][4 * gq], acc[f][j][4 * gq + 1], acc[f][j][4 * gq + 2], acc[f][j][4 * gq + 3]};
            __syncthreads();
#pragma unroll
            for (int j = 0; j < NTP; ++j) {
                const f32x4 *in = sum + ((grp * 3 + j) * 4 + pg) * 3 * 64 + lane;
                const f32x4 a = in[0], b = in[64], c = in[128];
                f32x4 v;
                switch (pg) {
                case 0: v = f32x4{acc[f][j][0], acc[f][j][1], acc[f][j][2], acc[f][j][3]} + a; v += b; v += c; break;
                case 1: v = a + f32x4{acc[f][j][4], acc[f][j][5], acc[f][j][6], acc[f][j][7]}; v += b; v += c; break;
                case 2: v = a + b; v += f32x4{acc[f][j][8], acc[f][j][9], acc[f][j][10], acc[f][j][11]}; v += c; break;
                default: v = a + b; v += c; v += f32x4{acc[f][j][12], acc[f][j][13], acc[f][j][14], acc[f][j][15]};
                }
                const int row = k0 + f * 32 + 8 * pg + 4 * (lane >> 5);
                float *d = dst + (size_t)row * p.rowsB + (size_t)(tap + j) * g.C + col;
                nan |= __builtin_isunordered(v[0], v[1]) | __builtin_isunordered(v[2], v[3]) ? 1u << (3 * f + j) : 0u;
                if (col < g.C && row < p.rowsA)   // c_out in whole 8s
#pragma unroll
                    for (int e = 0; e < 4; ++e) d[(size_t)e * p.rowsB] = v[e];
            }
        }
    };
    if (ROW || nt == 3) run(std::integral_constant<int, 3>());
    else if (nt == 2) run(std::integral_constant<int, 2>());
    else run(std::integral_constant<int, 1>());

    if constexpr (DB) {
        f32x4 *sum = reinterpret_cast<f32x4 *>(smem);
        __syncthreads();
        if (dbf >= 0 && pg > 0) sum[(dbf * 3 + pg - 1) * 64 + lane] = accdb;
        __syncthreads();
        if (dbf >= 0 && pg == 0) {
            for (int s = 0; s < 3; ++s) accdb += sum[(dbf * 3 + s) * 64 + lane];
            store_colsum_fragment(accdb, p.dbp + (size_t)split * p.rowsA, k0 + dbf * 32, p.rowsA, lane);
        }
    }

    // An infinite or NaN pixel also meets the zeros of padding slots, and zero times infinity is NaN: those sums are made again (the check is not measurable; 8 x 28 x 28, 512 -> 512 with one such pixel at an edge 46 us -> 1.2 - 2.3 ms, all NaN 71 us).
    // The arguments are read and the block's place is worked out again: kept, they would cost the loop scalar registers that it does not have.
    if (__builtin_expect(nan == 0, 1)) return;
    const Arguments *args = (const Arguments *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    sum_again<T>(args->p, args->q, nan, grp, pg, lane);
}

// the slot layout of a layer, false if the kernel does not take it
bool win_geom(const ConvGeom &g, int T, WinGeom *q, long long *slots)
{
    const int RS = g.R * g.S;
    if (g.sh != 1 || g.sw != 1 || g.C % 8 != 0 || g.K % 8 != 0 || RS < 3 || RS > kTapBlocks * kTapsPerBlock) return false;
    // offsets and slot numbers are 32-bit, and a slot before the first image must be out of range by its (negative) offset
    if ((long long)g.N * g.H * g.W * g.C * 2 >= 0x7fffffffLL || (long long)g.N * g.Ho * g.Wo * g.K * 2 >= 0x7fffffffLL) return false;
    q->P = g.W + g.pw > g.Wo ? g.W + g.pw : g.Wo;
    q->HP = g.H + g.ph > g.Ho ? g.H + g.ph : g.Ho;
    *slots = (long long)g.N * q->HP * q->P;
    if (*slots >= 0x3fffffffLL || q->P >= 0x8000 || q->HP >= 0x4000) return false;
    q->tilesC = (g.C + 31) / 32;
    q->tapBlocks = (RS + kTapsPerBlock - 1) / kTapsPerBlock;
    q->nxi = 0;
    for (int b = 0; b < q->tapBlocks; ++b) {
        long long lo = 0, hi = 0;
        const int t0 = b * RS / q->tapBlocks, t1 = (b + 1) * RS / q->tapBlocks;
        for (int t = t0; t < t1; ++t) {
            const long long o = (long long)(t / g.S - g.ph) * q->P + (t % g.S - g.pw);
            if (t == t0 || o < lo) lo = o;
            if (t == t0 || o > hi) hi = o;
        }
        const long long copies = (T + hi - lo + 15) / 16;
        if (copies + dy_copies(T) > lane_copies(T) * kWaves || T + copies * 16 > 64 * kWaves || lo < -0x3fffffffLL) return false;
        q->first[b] = (int)lo;
        q->tap[b] = t0;
        q->tap[b + 1] = t1;
        for (int t = t0; t < t1; ++t) q->at[t] = (short)((long long)(t / g.S - g.ph) * q->P + (t % g.S - g.pw) - lo);
        if (copies > q->nxi) q->nxi = (int)copies;
    }
    q->ns = (kLdsBytes - kTables * (T + q->nxi * 16) * 4) / 1024 / (dy_copies(T) + q->nxi);
    if (q->ns < 2) return false;
    if (q->ns > kMaxStages) q->ns = kMaxStages;
    q->dn = T / (q->HP * q->P);
    q->dh = (T - q->dn * q->HP * q->P) / q->P;
    q->dw = T - (q->dn * q->HP + q->dh) * q->P;
    return true;
}

typedef void (*WinKernel)(const KArgs, const WinGeom);
WinKernel pick_win(int T, bool db, bool row)
{
    if (!row) return k_wgrad_win<128, false, false>;
    if (T == 256) return db ? k_wgrad_win<256, true, true> : k_wgrad_win<256, false, true>;
    return db ? k_wgrad_win<128, true, true> : k_wgrad_win<128, false, true>;
}

}  // namespace

hipError_t wwin_init()
{
    for (int v = 0; v < 8; ++v) {
        const WinKernel k = pick_win(v & 4 ? 128 : 256, v & 1, v & 2);
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

bool wwin_plan(const ConvGeom &g, int slots_per_chunk, int force_splits, GemmPlan *pl)
{
    WinGeom q;
    long long slots;
    const bool row = g.R == 3 && g.S == 3;   // a wave's three taps are a filter row
    if ((slots_per_chunk != 128 && !row) || !win_geom(g, slots_per_chunk, &q, &slots)) return false;
    pl->variant = slots_per_chunk == 128 ? 17 : 18; pl->TA = 64; pl->TB = 32 * kTapsPerBlock; pl->BK = slots_per_chunk;
    pl->vecA = pl->vecB = true; pl->fast = true; pl->dma = true; pl->halo = false; pl->phase = false; pl->wstrip = false; pl->wwin = true;
    pl->row_taps = row;
    pl->tilesA = (g.K + 63) / 64;
    pl->tilesB = q.tilesC * q.tapBlocks;
    pl->steps_total = (int)((slots + slots_per_chunk - 1) / slots_per_chunk);
    const long long tiles = (long long)pl->tilesA * pl->tilesB;
    int splits = force_splits > 0 ? force_splits : (int)(256 / tiles > 0 ? 256 / tiles : 1);
    if (splits > pl->steps_total) splits = pl->steps_total;
    pl->steps_per_split = (pl->steps_total + splits - 1) / splits;
    pl->splits = (pl->steps_total + pl->steps_per_split - 1) / pl->steps_per_split;
    return true;
}

void wwin_kernel_name(const GemmPlan &pl, char *name, size_t name_bytes) { snprintf(name, name_bytes, pl.row_taps ? "k_wgrad_win<%d, true, true>" : "k_wgrad_win<%d, false, false>", pl.BK); }

hipError_t wwin_launch(const ConvArgs &a, hipStream_t st)
{
    KArgs p;
    WinGeom q;
    long long slots;
    const int T = a.plan.BK;
    if (!win_geom(a.g, T, &q, &slots)) return hipErrorInvalidValue;
    p.g = a.g;
    p.rowsA = a.g.K; p.rowsB = a.g.R * a.g.S * a.g.C; p.red = a.g.N * a.g.Ho * a.g.Wo;
    p.tilesA = a.plan.tilesA; p.tilesB = a.plan.tilesB;
    p.steps_total = a.plan.steps_total; p.steps_per_split = a.plan.steps_per_split; p.splits = a.plan.splits;
    p.flags = a.flags;
    p.x = a.x; p.w = nullptr; p.dy = a.dy; p.ymask = nullptr; p.bias = nullptr; p.out = a.out; p.partial = a.partial;
    p.dbp = p.splits > 1 ? a.db_partial : a.db_out;
    p.tickets = nullptr;
    p.ph_on = 0;
    const bool row = a.plan.row_taps, db = row && (p.flags & KF_DB) && p.dbp != nullptr;
    const int stages = q.ns * (dy_copies(T) + q.nxi) * 1024 + kTables * (T + q.nxi * 16) * 4;
    const WinKernel kern = pick_win(T, db, row);
    hipLaunchKernelGGL(kern, dim3((unsigned)(p.splits * p.tilesA * p.tilesB)), dim3(64 * kWaves),
                       stages > kSumBytes ? stages : kSumBytes, st, p, q);
    dp_trace_main_kernel_done(st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.splits <= 1) return e;
    return launch_split_reduce(a, p.rowsA, p.rowsB, st, db);
}
