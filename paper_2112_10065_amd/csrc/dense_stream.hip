// Dense (fully connected) forward at per-GPU batch <= 32, bound by reading the weights once (paper section 3.1: the
// small-batch regime leaves these layers with a few hundred flops per weight byte at most).
//
// y[n][o] = sum_i x[n][i] * W[o][i]: every weight is used N <= 32 times, so the kernel is a stream over W.  What the
// memory system rewards (measured): a wave-wide load that touches at most 8 rows with 128 contiguous bytes each, several
// such loads in flight per wave, eight or more waves per compute unit, and no block barrier in the stream.  So:
//   * a block owns 16 output rows (one 16x16x32 matrix-instruction tile of W rows x samples) and its 8 waves split the
//     input features among them; the waves' partial sums meet in LDS at the end (added in wave order), so there is no
//     second kernel and no partial sum in memory;
//   * every wave runs its own NS-stage pipeline of direct-to-LDS loads (two loads of 8 rows x 128 bytes per 64-feature
//     step) into its own LDS stages and reads the fragments back 16-byte chunk-swizzled (chunk c of row r sits at
//     position c ^ (r % 8)), waiting on its own load counter only;
//   * the activations (N rows, shared by all blocks, resident in L2) come straight from memory into registers, issued
//     together with the weight loads of the same step so that the in-order load counter never waits for a young load.
// Bias and ReLU are applied after the waves' sums are added.
#include "dma_common.h"
#include <algorithm>
#include <type_traits>

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4v;

// the weights are read once per pass: non-temporal, so that the stream does not push the step's activations out of the caches
DEVFN void dma16_soff(__amdgpu_buffer_rsrc_t r, unsigned lds_base, unsigned voff, unsigned soff)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void)(size_t)lds_base, 16, voff, soff, 0, 2);
}
// 16 bytes per lane into registers, invisible to the compiler's wait placement (it would drain the whole pipeline once per
// trip of the unrolled loop): the caller waits on the load counter and then ties the registers to that wait
template <int OFF> DEVFN u32x4 load16_async(u32x4 rsrc, unsigned voff, unsigned soff)
{
    u32x4 v;
    asm volatile("buffer_load_dwordx4 %0, %1, %2, %3 offen offset:%4" : "=v"(v) : "v"(voff), "s"(rsrc), "s"(soff), "n"(OFF) : "memory");
    return v;
}
DEVFN u32x4 raw_rsrc(const void *p, size_t bytes)   // the words of make_rsrc's descriptor
{
    const unsigned long long a = (unsigned long long)p;
    return u32x4{(unsigned)a, (unsigned)(a >> 32) & 0xffffu, (unsigned)bytes, 0x00020000u};
}

constexpr int DF_NS = 5, DF_WAVES = 8, DF_STAGE = 2048;

template <int NB>   // groups of 16 samples: 1 (N <= 16) or 2 (N <= 32)
__global__ __launch_bounds__(64 * DF_WAVES) void k_dense_fwd(int N, int C, int K, unsigned flags, const bf16_t *x, const bf16_t *w, const float *bias,
                                                             bf16_t *y)
{
    constexpr int D = DF_NS - 1, P = 2 + 2 * NB;   // prefetch distance in steps; memory instructions per step
    static_assert((D - 1) * P < 64, "the load counter has six bits");
    __shared__ __attribute__((aligned(1024))) char lds[DF_WAVES * DF_NS * DF_STAGE];
    static_assert(sizeof(lds) >= DF_WAVES * NB * 64 * sizeof(f32x4v), "the waves' sums fit the stages");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g0 = blockIdx.x * 16;
    const int steps = C / 64, spw = (steps + DF_WAVES - 1) / DF_WAVES;
    const int sbeg = min(wave * spw, steps), nst = min(sbeg + spw, steps) - sbeg;
    __amdgpu_buffer_rsrc_t rw = make_rsrc(w, (size_t)K * C * 2);
    const u32x4 rx = raw_rsrc(x, (size_t)N * C * 2);
    const unsigned base = lds_offset(lds) + wave * (DF_NS * DF_STAGE);

    unsigned voffW[2], voffX[NB];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = 8 * j + (lane >> 3), c = (lane & 7) ^ (row & 7);
        voffW[j] = g0 + row < K ? ((unsigned)(g0 + row) * C + c * 8) * 2u : OOR;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int n = 16 * b + (lane & 15);
        voffX[b] = n < N ? ((unsigned)n * C + (lane >> 4) * 8) * 2u : OOR;
    }
    // fragment of W for matrix instruction s of a step: row l%16, features 32*s + 8*(l/16) .. +7, i.e. chunk 4*s + l/16
    unsigned fa[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) fa[s] = base + (lane & 15) * 128 + (((4 * s + (lane >> 4)) ^ (lane & 7)) << 4);

    u32x4 xr[DF_NS][NB][2];
    auto issue = [&](int i, int stage) {   // loads of step i (relative to sbeg) into `stage`
        const unsigned soff = (unsigned)(sbeg + i) * 128u;
#pragma unroll
        for (int j = 0; j < 2; ++j) dma16_soff(rw, base + stage * DF_STAGE + j * 1024, voffW[j], soff);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            xr[stage][b][0] = load16_async<0>(rx, voffX[b], soff);
            xr[stage][b][1] = load16_async<64>(rx, voffX[b], soff);
        }
    };
    f32x4v acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4v{0.f, 0.f, 0.f, 0.f};

#pragma unroll
    for (int u = 0; u < D; ++u)
        if (u < nst) issue(u, u);
    for (int i0 = 0; i0 < nst; i0 += DF_NS) {
#pragma unroll
        for (int u = 0; u < DF_NS; ++u) {
            const int i = i0 + u;
            if (i < nst) {
                const int younger = min(D - 1, nst - 1 - i);
                if (younger == D - 1) wait_vmcnt<(D - 1) * P>();
                else if (D >= 3 && younger == D - 2) wait_vmcnt<(D >= 3 ? D - 2 : 0) * P>();
                else if (D >= 4 && younger == D - 3) wait_vmcnt<(D >= 4 ? D - 3 : 0) * P>();
                else wait_vmcnt<0>();
                if (i + D < nst) issue(i + D, (u + D) % DF_NS);   // the stage of step i - 1, whose reads have returned
                u32x4 a[2];
                a[0] = lds_read16<0>(fa[0] + u * DF_STAGE);
                a[1] = lds_read16<0>(fa[1] + u * DF_STAGE);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                asm volatile("" : "+v"(a[0]), "+v"(a[1]));
#pragma unroll
                for (int b = 0; b < NB; ++b) asm volatile("" : "+v"(xr[u][b][0]), "+v"(xr[u][b][1]));   // landed with the step's weight loads
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[s]), __builtin_bit_cast(bf16x8, xr[u][b][s]), acc[b], 0, 0, 0);
            }
        }
    }
    wait_vmcnt<0>();
    __syncthreads();   // every wave is done with its stages: they give way to the sums
    f32x4v *red = reinterpret_cast<f32x4v *>(lds);   // [wave][group][lane]
#pragma unroll
    for (int b = 0; b < NB; ++b) red[(wave * NB + b) * 64 + lane] = acc[b];
    __syncthreads();
    if (tid < 64 * NB) {
        const int b = tid >> 6;
        f32x4v s = red[b * 64 + lane];
#pragma unroll
        for (int wv = 1; wv < DF_WAVES; ++wv) s += red[(wv * NB + b) * 64 + lane];
        // element v of lane l: output row g0 + 4*(l/16) + v, sample 16*b + l%16
        const int n = 16 * b + (lane & 15), o = g0 + 4 * (lane >> 4);
        if (n < N) {
            float v[4] = {s[0], s[1], s[2], s[3]};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if ((flags & KF_BIAS) && o + e < K) v[e] += bias[o + e];
                if (flags & KF_RELU) v[e] = fmaxf(v[e], 0.f);
            }
            bf16_t *dst = y + (size_t)n * K + o;
            if (o + 4 <= K && (K & 3) == 0) *reinterpret_cast<u32x2 *>(dst) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
            else
                for (int e = 0; e < 4; ++e) if (o + e < K) dst[e] = (bf16_t)f32_to_bf16(v[e]);
        }
    }
}

// ---------------------------------------------------------------------------------------
// Backward-data of the same layers: dx[n][i] = sum_o dy[n][o] * W[o][i], again one pass over W.  A block owns 64 input
// features (128 contiguous bytes of every weight row) and its 8 waves split the output rows, the reduction, among
// them.  A step is 16 weight rows: two direct-to-LDS loads of 8 rows x 128 bytes into the wave's own stage, rows as they
// come from memory (the two 64-byte halves of a row swapped on odd row pairs); the matrix instruction wants the
// reduction contiguous per lane, which the LDS transpose read delivers.  The gradient operand (sample l%32, output rows
// 8*(l/32) .. +7 of the step) is 16 contiguous bytes of dy and goes from memory straight into registers, issued with the
// step's weight loads.  The waves' sums meet in LDS; the backward of the ReLU in front of the layer (mask by the saved
// input) and the conversion ride in that last pass.
// ---------------------------------------------------------------------------------------
constexpr int DG_NS = 4, DG_STAGE = 2048;
template <int OFF> DEVFN u32x2 lds_read_tr_off(unsigned addr)
{
    u32x2 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
__global__ __launch_bounds__(64 * DF_WAVES) void k_dense_dgrad(int N, int C, int K, unsigned flags, const bf16_t *dy, const bf16_t *w, const bf16_t *xin,
                                                               void *dx)
{
    constexpr int D = DG_NS - 1, P = 3;   // prefetch distance in steps; memory instructions per step
    __shared__ __attribute__((aligned(1024))) char lds[DF_WAVES * DG_NS * DG_STAGE];   // 64 KiB: the stages, then the waves' sums
    static_assert(sizeof(lds) >= DF_WAVES * 2 * 64 * sizeof(f32x16), "the waves' sums fit the stages");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = blockIdx.x * 64;
    const int steps = (K + 15) / 16, spw = (steps + DF_WAVES - 1) / DF_WAVES;
    const int sbeg = min(wave * spw, steps), nst = min(sbeg + spw, steps) - sbeg;
    __amdgpu_buffer_rsrc_t rw = make_rsrc(w, (size_t)K * C * 2);
    const u32x4 rdy = raw_rsrc(dy, (size_t)N * K * 2);
    const unsigned base = lds_offset(lds) + wave * (DG_NS * DG_STAGE);

    // weight loads: lane l of load j fills 16-byte position l%8 of stage row 8*j + l/8 with global chunk (l%8) ^ 4*swz(row); rows
    // past the last output and chunks past the last input feature fetch zeros (the range check of the buffer covers the end only)
    unsigned voffW[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int t = 8 * j + (lane >> 3), c = (lane & 7) ^ (seg_swz<64>(t) << 2);
        voffW[j] = i0 + c * 8 < C ? ((unsigned)t * C + i0 + c * 8) * 2u : OOR;
    }
    const unsigned voffY = (lane & 31) < N ? ((unsigned)(lane & 31) * K + (lane >> 5) * 8) * 2u : OOR;
    // transpose-read addresses of the two 32-feature fragments: lane l of a 16-lane group points at stage row 8*(l>>5) + (l&15)/4
    // (+4 for the second half), features 16*((l>>4)&1) + 4*(l&3) .. +3 of the fragment
    const int i16 = lane & 15, tl = (lane >> 5) * 8 + (i16 >> 2), cl = ((lane >> 4) & 1) * 16 + (i16 & 3) * 4;
    unsigned fa[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) fa[i] = base + tl * 128 + (((i ^ seg_swz<64>(tl)) << 6) | (cl << 1));

    u32x4 yr[DG_NS];
    auto issue = [&](int i, int stage) {
        const int o0 = (sbeg + i) * 16;
        // rows of the step past K: the buffer's range check sees offsets past the end of W only for the very last rows, so mask here
        const unsigned soff = (unsigned)o0 * (unsigned)C * 2u;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const bool live = o0 + 8 * j + (lane >> 3) < K;
            dma16_soff(rw, base + stage * DG_STAGE + j * 1024, live ? voffW[j] : OOR, soff);
        }
        // eight output rows per lane: a chunk that straddles K is cut by the buffer's range check only at the very end of dy, so mask
        const bool ylive = o0 + (lane >> 5) * 8 + 8 <= K;
        yr[stage] = load16_async<0>(rdy, ylive ? voffY : OOR, (unsigned)o0 * 2u);
    };
    f32x16 acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;

#pragma unroll
    for (int u = 0; u < D; ++u)
        if (u < nst) issue(u, u);
    for (int it0 = 0; it0 < nst; it0 += DG_NS) {
#pragma unroll
        for (int u = 0; u < DG_NS; ++u) {
            const int it = it0 + u;
            if (it < nst) {
                const int younger = min(D - 1, nst - 1 - it);
                if (younger == D - 1) wait_vmcnt<(D - 1) * P>();
                else if (D >= 3 && younger == D - 2) wait_vmcnt<(D >= 3 ? D - 2 : 0) * P>();
                else wait_vmcnt<0>();
                if (it + D < nst) issue(it + D, (u + D) % DG_NS);   // the stage of step it - 1, whose reads have returned
                u32x2 lo[2], hi[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    lo[i] = lds_read_tr_off<0>(fa[i] + u * DG_STAGE);
                    hi[i] = lds_read_tr_off<512>(fa[i] + u * DG_STAGE);
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                asm volatile("" : "+v"(lo[0]), "+v"(hi[0]), "+v"(lo[1]), "+v"(hi[1]), "+v"(yr[u]));
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, u32x4{lo[i].x, lo[i].y, hi[i].x, hi[i].y}),
                                                                     __builtin_bit_cast(bf16x8, yr[u]), acc[i], 0, 0, 0);
            }
        }
    }
    wait_vmcnt<0>();
    __syncthreads();   // every wave is done with its stages: they give way to the sums
    f32x4v *red = reinterpret_cast<f32x4v *>(lds);   // [wave][fragment][group of four registers][lane]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int gq = 0; gq < 4; ++gq)
            red[((wave * 2 + i) * 4 + gq) * 64 + lane] = f32x4v{acc[i][4 * gq], acc[i][4 * gq + 1], acc[i][4 * gq + 2], acc[i][4 * gq + 3]};
    __syncthreads();
    {
        // wave w adds group w%4 of fragment w/4 over the eight waves, in wave order: registers 4*gq .. +3 of lane l are
        // features 32*i + 8*gq + 4*(l/32) .. +3 of sample l%32
        const int i = wave >> 2, gq = wave & 3;
        f32x4v s = red[((0 * 2 + i) * 4 + gq) * 64 + lane];
#pragma unroll
        for (int wv = 1; wv < DF_WAVES; ++wv) s += red[((wv * 2 + i) * 4 + gq) * 64 + lane];
        const int n = lane & 31, f = i0 + 32 * i + 8 * gq + 4 * (lane >> 5);
        if (n < N && f < C) {
            float v[4] = {s[0], s[1], s[2], s[3]};
            const size_t o = (size_t)n * C + f;
            if (flags & KF_MASK_IN)
                for (int e = 0; e < 4; ++e) if (f + e < C) v[e] = mask1f(v[e], xin[o + e]);
            if (flags & KF_OUT_F32) {
                float *dst = reinterpret_cast<float *>(dx) + o;
                if (f + 4 <= C && (C & 3) == 0) *reinterpret_cast<f32x4 *>(dst) = f32x4{v[0], v[1], v[2], v[3]};
                else
                    for (int e = 0; e < 4; ++e) if (f + e < C) dst[e] = v[e];
            } else {
                bf16_t *dst = reinterpret_cast<bf16_t *>(dx) + o;
                if (f + 4 <= C && (C & 3) == 0) *reinterpret_cast<u32x2 *>(dst) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
                else
                    for (int e = 0; e < 4; ++e) if (f + e < C) dst[e] = (bf16_t)f32_to_bf16(v[e]);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------
// Filter gradient of the same layers: dW[o][i] = sum_n dy[n][o] * x[n][i] with N <= 32 is an outer product that writes
// K*C fp32 once and reads next to nothing, so it is a store stream.  A wave owns one 64 x 64 tile of dW: it copies its
// dy tile [32 samples][64 outputs] and its x tile [32 samples][64 inputs] into its own LDS (direct-to-LDS loads, rows of
// samples the batch does not have fetch zeros), reads both through the LDS transpose read (samples are the reduction),
// multiplies (one 16-sample slice, two beyond 16 samples) and stores its sums, non-temporally when the gradient is large.
// No barrier, no row tables, no partial sums.  The bias gradient (dy fragments times ones) is added by the waves of the
// first input tile.
// ---------------------------------------------------------------------------------------
template <bool NT>
__global__ __launch_bounds__(64 * DF_WAVES) void k_dense_wgrad(int N, int C, int K, const bf16_t *x, const bf16_t *dy, float *dw, float *db)
{
    __shared__ __attribute__((aligned(1024))) char lds[DF_WAVES * 8192];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int o0 = blockIdx.x * 64, i0 = (blockIdx.y * DF_WAVES + wave) * 64;
    if (i0 >= C) return;   // no barrier follows
    __amdgpu_buffer_rsrc_t rdy = make_rsrc(dy, (size_t)N * K * 2);
    __amdgpu_buffer_rsrc_t rx = make_rsrc(x, (size_t)N * C * 2);
    const unsigned base = lds_offset(lds) + wave * 8192;
    // lane l of load j fills 16-byte position l%8 of tile row (sample) 8*j + l/8 with global chunk (l%8) ^ 4*swz(row)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int t = 8 * j + (lane >> 3), c = (lane & 7) ^ (seg_swz<64>(t) << 2);
        const bool row = t < N;
        dma16(rdy, base + j * 1024, row && o0 + c * 8 < K ? ((unsigned)t * K + o0 + c * 8) * 2u : OOR);
        dma16(rx, base + 4096 + j * 1024, row && i0 + c * 8 < C ? ((unsigned)t * C + i0 + c * 8) * 2u : OOR);
    }
    const int i16 = lane & 15, tl = (lane >> 5) * 8 + (i16 >> 2), cl = ((lane >> 4) & 1) * 16 + (i16 & 3) * 4;
    unsigned fa[2];   // fragment f of either tile: sample rows tl (+4), columns 32*f + cl .. +3
#pragma unroll
    for (int f = 0; f < 2; ++f) fa[f] = base + tl * 128 + (((f ^ seg_swz<64>(tl)) << 6) | (cl << 1));
    f32x16 acc[2][2], accdb[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
#pragma unroll
        for (int v = 0; v < 16; ++v) accdb[a][v] = 0.f;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    }
    const bool do_db = db != nullptr && i0 == 0;
    wait_vmcnt<0>();
    auto slice = [&](auto ks_tag) {
        constexpr int KS = decltype(ks_tag)::value;
        u32x2 alo[2], ahi[2], blo[2], bhi[2];
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            alo[f] = lds_read_tr_off<KS * 2048>(fa[f]);
            ahi[f] = lds_read_tr_off<KS * 2048 + 512>(fa[f]);
            blo[f] = lds_read_tr_off<4096 + KS * 2048>(fa[f]);
            bhi[f] = lds_read_tr_off<4096 + KS * 2048 + 512>(fa[f]);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        asm volatile("" : "+v"(alo[0]), "+v"(ahi[0]), "+v"(alo[1]), "+v"(ahi[1]), "+v"(blo[0]), "+v"(bhi[0]), "+v"(blo[1]), "+v"(bhi[1]));
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const bf16x8 av = __builtin_bit_cast(bf16x8, u32x4{alo[a].x, alo[a].y, ahi[a].x, ahi[a].y});
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, __builtin_bit_cast(bf16x8, u32x4{blo[b].x, blo[b].y, bhi[b].x, bhi[b].y}), acc[a][b], 0, 0, 0);
            if (do_db) accdb[a] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, ones_bf16(), accdb[a], 0, 0, 0);
        }
    };
    slice(std::integral_constant<int, 0>{});
    if (N > 16) slice(std::integral_constant<int, 1>{});
    // element v of lane l: output row 8*(v/4) + 4*(l/32) + v%4 of its fragment, input column l%32
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int o = o0 + 32 * a + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            if (o >= K) continue;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int i = i0 + 32 * b + (lane & 31);
                if (i >= C) continue;
                if (NT) __builtin_nontemporal_store(acc[a][b][v], dw + (size_t)o * C + i);
                else dw[(size_t)o * C + i] = acc[a][b][v];
            }
        }
    if (do_db) {
#pragma unroll
        for (int a = 0; a < 2; ++a) store_db_fragment(accdb[a], db, o0 + 32 * a, K, lane);
    }
}

// ---------------------------------------------------------------------------------------
// Forward and backward-data of the same layers in one pass over W, for calls that ask for both (the incoming gradient is an input of such a
// call, so neither waits for the other).  Apart, each streams W: 42 + 47 us on 25088 x 4096 at two samples; together 50
// (4096 x 4096: 21 -> 9.7, 1024 x 1024: 11.8 -> 7.5).
// A block owns 16 * RT output rows and a range of 64-feature column units, its waves take one unit after the other and walk down the
// rows, 16 at a time (two direct-to-LDS loads of 8 rows x 128 bytes, NS stages per wave, no block barrier in the stream).  A
// stage feeds both products: read by rows it is the weight operand of the forward tile (16 outputs x samples, one accumulator per row
// tile, kept over all units of the wave), through the transpose read the operand of the gradient of the unit's 64 inputs (kept down the
// column, stored per unit).  The 16-byte chunk c of row r sits at c ^ (r % 8), which both reads accept.  The block's
// dy rows wait in LDS in fragment order, the unit's x fragments in registers.  y is then summed over the waves (in wave order) and leaves as
// one partial per column range, dx as one per row range; k_dense_both_sum adds them in order and applies bias, ReLU and mask.
// RT = 32 keeps the partials of dx few (16 * samples / 4096 of the weight bytes each way); layers too small to give every wave of
// the chip a unit that way take RT = 8, those with fewer such units than CUs RT = 2: there the chain of a wave's row tiles is the time.
// Both kernels, two passes apart / RT = 8 / RT = 2: 512 x 184, 16 samples 7.8 / 9.4 / 8.1 us; 1024 x 160, 16 samples 8.3 / 9.7 / 8.1; over 140
// drawn layers under 256 units RT = 2 is 0.97 - 1.4 times as fast as the passes apart, RT = 8 0.83 - 1.3; at 500 units the two are even.
// ---------------------------------------------------------------------------------------
constexpr int DB_NS = 6;
template <int RT, bool Y>   // Y: also the forward product
__global__ __launch_bounds__(64 * DF_WAVES) void k_dense_both(int N, int C, int K, int units_per_block, const bf16_t *x, const bf16_t *dy, const bf16_t *w,
                                                              float *ypart, float *dxpart)
{
    constexpr int D = DB_NS - 1, STAGE = 2048, DYB = RT * 512, TG = RT < 8 ? RT : 8;   // TG: row tiles whose sums meet in LDS at a time
    static_assert(DF_WAVES * DB_NS * STAGE >= DF_WAVES * 8 * 64 * (int)sizeof(f32x4v), "the waves' sums of eight row tiles fit the stages");
    static_assert(RT % 2 == 0 && RT % TG == 0, "dy is fetched two row tiles at a time; whole groups of tiles are summed");
    __shared__ __attribute__((aligned(1024))) char lds[DF_WAVES * DB_NS * STAGE + DYB];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int o0 = blockIdx.x * RT * 16, nst = min(RT, (K - o0 + 15) / 16);
    const int units = C / 64, ubeg = blockIdx.y * units_per_block, uend = min(ubeg + units_per_block, units);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(w, (size_t)K * C * 2), rx = make_rsrc(x, (size_t)N * C * 2), rdy = make_rsrc(dy, (size_t)N * K * 2);
    const unsigned base = lds_offset(lds) + wave * (DB_NS * STAGE), dybase = lds_offset(lds) + DF_WAVES * DB_NS * STAGE;

    // dy fragments of the block's rows: 16-byte chunk (step, half h, sample) at step*512 + (h*16 + sample)*16 holds rows 16*step + 8*h .. +7
    // (K is whole chunks); one load fills two steps
#pragma unroll
    for (int q = 0; q < RT / 2; q += DF_WAVES) {
        const int pair = q + wave;
        if (pair < RT / 2) {
            const int o = o0 + pair * 32 + (lane >> 4) * 8, n = lane & 15;
            dma16(rdy, dybase + pair * 1024, n < N && o < K ? ((unsigned)n * K + o) * 2u : OOR);
        }
    }
    // weight loads: lane l of load j fills 16-byte position l%8 of stage row 8*j + l/8 with global chunk (l%8) ^ (row%8)
    unsigned voffW[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = 8 * j + (lane >> 3), c = (lane & 7) ^ (row & 7);
        voffW[j] = ((unsigned)(o0 + row) * C + c * 8) * 2u;
    }
    // by rows: row l%16, features 32*s + 8*(l/16) .. +7; transposed: row 8*(l>>5) + (l&15)/4 (+4: chunk ^ 4), features 32*i + 16*((l>>4)&1) + 4*(l&3) .. +3
    unsigned fr[2], ft[2], ft4[2];
    const int i16 = lane & 15, tl = (lane >> 5) * 8 + (i16 >> 2), cl = ((lane >> 4) & 1) * 16 + (i16 & 3) * 4;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        fr[s] = base + i16 * 128 + (((4 * s + (lane >> 4)) ^ (lane & 7)) << 4);
        const int col = 32 * s + cl, ch = col >> 3;
        ft[s] = base + tl * 128 + ((ch ^ (tl & 7)) << 4) + (col & 7) * 2;
        ft4[s] = base + (tl + 4) * 128 + ((ch ^ ((tl + 4) & 7)) << 4) + (col & 7) * 2;
    }
    const unsigned fdy = dybase + ((lane >> 5) * 16 + i16) * 16;   // lanes of samples 16 .. 31 repeat 0 .. 15, their columns are not stored
    const unsigned voffX = i16 < N ? ((unsigned)i16 * C + (lane >> 4) * 8) * 2u : OOR;

    f32x4v accy[Y ? RT : 1];
#pragma unroll
    for (int t = 0; t < (Y ? RT : 1); ++t) accy[t] = f32x4v{0.f, 0.f, 0.f, 0.f};
    bool first = true;
    for (int u = ubeg + wave; first || u < uend; u += DF_WAVES) {
        const bool live = u < uend;   // a wave without a unit still meets the barrier below
        const unsigned ucol = (unsigned)u * 128u;
        u32x4 xf[2];
        auto issue = [&](int step, int stage) {
            const unsigned soff = (unsigned)(step * 16) * (unsigned)C * 2u + ucol;
            int row = o0 + (lane >> 3);
            asm volatile("" : "+v"(row));   // computed here and not kept for all steps across the units
#pragma unroll
            for (int j = 0; j < 2; ++j) dma16_soff(rw, base + stage * STAGE + j * 1024, row + step * 16 + 8 * j < K ? voffW[j] : OOR, soff);
        };
        if (live) {
#pragma unroll
            for (int s = 0; s < 2; ++s) if (Y) xf[s] = __builtin_amdgcn_raw_buffer_load_b128(rx, i16 < N ? voffX + ucol + s * 64 : OOR, 0, 0);
#pragma unroll
            for (int t = 0; t < D; ++t)
                if (t < nst) issue(t, t);
        }
        if (first) {   // this wave's dy chunks have landed (they are older than the loads above), then everybody's
            if (live && nst >= D) wait_vmcnt<2 * D>(); else wait_vmcnt<0>();
            __builtin_amdgcn_s_barrier();
            first = false;
        }
        if (!live) break;
        f32x16 accx[2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) accx[i][v] = 0.f;
        for_constant<RT>([&](auto tc) {   // stage and fragment offsets are instruction immediates
            constexpr int t = decltype(tc)::value, st = (t % DB_NS) * STAGE;
            if (t < nst) {
                constexpr int P = 2;
                if (nst - 1 - t >= D - 1) wait_vmcnt<(D - 1) * P>();
                else if (nst - 1 - t == D - 2) wait_vmcnt<(D - 2) * P>();
                else if (nst - 1 - t == D - 3) wait_vmcnt<(D - 3) * P>();
                else wait_vmcnt<0>();
                if (t + D < nst) issue(t + D, (t + D) % DB_NS);   // the stage of step t - 1, whose reads have returned
                u32x4 a[2], yf;
                u32x2 lo[2], hi[2];
#pragma unroll
                for (int s = 0; s < 2; ++s) if (Y) a[s] = lds_read16<st>(fr[s]);
#pragma unroll
                for (int s = 0; s < 2; ++s) { lo[s] = lds_read_tr_off<st>(ft[s]); hi[s] = lds_read_tr_off<st>(ft4[s]); }
                yf = lds_read16<t * 512>(fdy);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if constexpr (Y) asm volatile("" : "+v"(a[0]), "+v"(a[1]));
                asm volatile("" : "+v"(yf), "+v"(lo[0]), "+v"(hi[0]), "+v"(lo[1]), "+v"(hi[1]));
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    if constexpr (Y) accy[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[s]), __builtin_bit_cast(bf16x8, xf[s]), accy[t], 0, 0, 0);
                    accx[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, u32x4{lo[s].x, lo[s].y, hi[s].x, hi[s].y}),
                                                                      __builtin_bit_cast(bf16x8, yf), accx[s], 0, 0, 0);
                }
            }
        });
        // element v of lane l: feature 32*i + 8*(v/4) + 4*(l/32) + v%4 of the unit, sample l%32
        if ((lane & 31) < N) {
            float *dst = dxpart + ((size_t)blockIdx.x * N + (lane & 31)) * C + u * 64 + 4 * (lane >> 5);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq)
                    *reinterpret_cast<f32x4v *>(dst + 32 * i + 8 * gq) = f32x4v{accx[i][4 * gq], accx[i][4 * gq + 1], accx[i][4 * gq + 2], accx[i][4 * gq + 3]};
        }
    }
    if constexpr (!Y) return;
    // y: the eight waves' sums of TG row tiles at a time; wave v adds tile v in wave order
    f32x4v *red = reinterpret_cast<f32x4v *>(lds);   // [wave][tile][lane]
#pragma unroll
    for (int t0 = 0; t0 < RT; t0 += TG) {
        __syncthreads();   // the stages (or the tiles before) have been read
#pragma unroll
        for (int t = 0; t < TG; ++t) red[(wave * TG + t) * 64 + lane] = accy[Y ? t0 + t : 0];
        __syncthreads();
        if (wave >= TG) continue;
        f32x4v s = red[wave * 64 + lane];
#pragma unroll
        for (int wv = 1; wv < DF_WAVES; ++wv) s += red[(wv * TG + wave) * 64 + lane];
        // element v of lane l: output row 4*(l/16) + v of the tile, sample l%16
        const int o = o0 + (t0 + wave) * 16 + 4 * (lane >> 4);
        if (i16 < N && o < K) *reinterpret_cast<f32x4v *>(ypart + ((size_t)blockIdx.y * N + i16) * K + o) = s;
    }
}

// dx and y from the partials of k_dense_both: thread (group of four, part) adds every eighth partial, the eight parts are added in
// order; blocks 0 .. nbx - 1 take dx, the others y
__global__ __launch_bounds__(256) void k_dense_both_sum(int N, int C, int K, int nbx, int row_parts, int col_parts, unsigned flags_y, unsigned flags_dx,
                                                        const float *dxpart, const float *ypart, const float *bias, const bf16_t *xin, bf16_t *y, void *dx)
{
    __shared__ f32x4v sm[8][32];
    const bool is_dx = (int)blockIdx.x < nbx;
    const int width = is_dx ? C : K, parts = is_dx ? row_parts : col_parts;
    const float *src = is_dx ? dxpart : ypart;
    const int q = threadIdx.x & 31, part = threadIdx.x >> 5, total = N * width;
    const int e = ((is_dx ? blockIdx.x : blockIdx.x - nbx) * 32 + q) * 4;
    f32x4v s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
    if (e < total) {
        int b = part;
        for (; b + 8 < parts; b += 16) {
            s0 += *reinterpret_cast<const f32x4v *>(src + (size_t)b * total + e);
            s1 += *reinterpret_cast<const f32x4v *>(src + (size_t)(b + 8) * total + e);
        }
        if (b < parts) s0 += *reinterpret_cast<const f32x4v *>(src + (size_t)b * total + e);
    }
    sm[part][q] = s0 + s1;
    __syncthreads();
    if (part != 0 || e >= total) return;
    f32x4v s = sm[0][q];
#pragma unroll
    for (int i = 1; i < 8; ++i) s += sm[i][q];
    float v[4] = {s[0], s[1], s[2], s[3]};
    if (is_dx) {
        if (flags_dx & KF_MASK_IN) {
            const u32x2 xm = *reinterpret_cast<const u32x2 *>(xin + e);
            const bf16_t xv[4] = {(bf16_t)xm.x, (bf16_t)(xm.x >> 16), (bf16_t)xm.y, (bf16_t)(xm.y >> 16)};
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = mask1f(v[i], xv[i]);
        }
        if (flags_dx & KF_OUT_F32) *reinterpret_cast<f32x4v *>(reinterpret_cast<float *>(dx) + e) = f32x4v{v[0], v[1], v[2], v[3]};
        else *reinterpret_cast<u32x2 *>(reinterpret_cast<bf16_t *>(dx) + e) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        return;
    }
    const int o = e % K;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (flags_y & KF_BIAS) v[i] += bias[o + i];
        if (flags_y & KF_RELU) v[i] = fmaxf(v[i], 0.f);
    }
    *reinterpret_cast<u32x2 *>(y + e) = u32x2{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
}

}  // namespace

// shapes the fused pass takes: at most 16 samples (one matrix tile; beyond that the partials of dx outweigh the second read of W), input
// features in whole units, output features in whole 8s
bool dense_both_shape(const ConvGeom &g)
{
    return g.R == 1 && g.S == 1 && g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0 && g.H == 1 && g.W == 1 && g.N <= 16 && g.C % 64 == 0 && g.C >= 512 &&
           g.K % 8 == 0 && (unsigned long long)g.K * g.C * 2 < (1ull << 32);
}
// Backward-data alone: against the pipelined tiles and their split reduction it pays where the weights are many and the partials of dx few.
// Measured new / old: 25088 x 4096 2 samples 35.0 / 37.7 us, 16 samples 44.2 / 40.6; 4096 x 4096 2 samples 7.9 / 13.7, 8 samples 9.8 / 14.0;
// 12800 x 2048 2 samples 11.3 / 14.0, 16 samples 20.4 / 14.6; 8192 x 512 7.0 / 6.8; 1024 x 1024 7.3 / 6.9
bool dense_dgrad_split_shape(const ConvGeom &g)
{
    return dense_both_shape(g) && g.K % 64 == 0 && g.N <= 8 && g.K >= 1024 && (long long)g.K * g.C >= (4 << 20);
}
static void dense_both_split(const ConvGeom &g, int *rt, int *row_parts, int *units_per_block, int *col_parts)
{
    const int units = g.C / 64;
    // 32: a unit for every wave of one block per CU; 2: never without y, see dense_dgrad_split_shape
    *rt = (long long)((g.K + 511) / 512) * units >= 2048 ? 32 : (long long)((g.K + 127) / 128) * units >= 256 ? 8 : 2;
    *row_parts = (g.K + *rt * 16 - 1) / (*rt * 16);
    int cp = std::max(1, 256 / *row_parts);
    if (cp > (units + DF_WAVES - 1) / DF_WAVES) cp = (units + DF_WAVES - 1) / DF_WAVES;
    *units_per_block = (units + cp - 1) / cp;
    *col_parts = (units + *units_per_block - 1) / *units_per_block;
}
size_t dense_both_partial_bytes(const ConvGeom &g, bool with_y)
{
    int rt, rp, upb, cp;
    dense_both_split(g, &rt, &rp, &upb, &cp);
    return ((size_t)rp * g.N * g.C + (with_y ? (size_t)cp * g.N * g.K : 0)) * sizeof(float);
}
hipError_t dense_both(const ConvGeom &g, const bf16_t *x, const bf16_t *dy, const bf16_t *w, float *partial, bool with_y, hipStream_t st)
{
    int rt, rp, upb, cp;
    dense_both_split(g, &rt, &rp, &upb, &cp);
    float *ypart = partial + (size_t)rp * g.N * g.C;
    const dim3 grid((unsigned)rp, (unsigned)cp), block(64 * DF_WAVES);
    auto *kernel = rt == 32 ? (with_y ? k_dense_both<32, true> : k_dense_both<32, false>) : rt == 2 ? k_dense_both<2, true> :
                   (with_y ? k_dense_both<8, true> : k_dense_both<8, false>);
    hipLaunchKernelGGL(kernel, grid, block, 0, st, g.N, g.C, g.K, upb, x, dy, w, ypart, partial);
    return hipGetLastError();
}
hipError_t dense_both_sum(const ConvGeom &g, unsigned flags_y, unsigned flags_dx, const float *partial, const float *bias, const bf16_t *xin, bf16_t *y,
                          void *dx, hipStream_t st)
{
    int rt, rp, upb, cp;
    dense_both_split(g, &rt, &rp, &upb, &cp);
    const int nbx = (g.N * g.C / 4 + 31) / 32, nby = y != nullptr ? (g.N * g.K / 4 + 31) / 32 : 0;
    hipLaunchKernelGGL(k_dense_both_sum, dim3((unsigned)(nbx + nby)), dim3(256), 0, st, g.N, g.C, g.K, nbx, rp, cp, flags_y, flags_dx, partial,
                       partial + (size_t)rp * g.N * g.C, bias, xin, y, dx);
    return hipGetLastError();
}
const char *dense_both_name(const ConvGeom &g, bool with_y)
{
    int rt, rp, upb, cp;
    dense_both_split(g, &rt, &rp, &upb, &cp);
    return rt == 32 ? (with_y ? "k_dense_both<32, true>" : "k_dense_both<32, false>") : rt == 2 ? "k_dense_both<2, true>" : (with_y ? "k_dense_both<8, true>" : "k_dense_both<8, false>");
}

// shapes the streaming dense forward takes: a 1x1 layer over at most 16 pixel rows (beyond that the activation operand, which
// every block re-reads, outweighs the weights), input features in whole 64-feature steps
bool dense_fwd_stream_shape(const ConvGeom &g)
{
    const long long rows = (long long)g.N * g.Ho * g.Wo;
    return g.R == 1 && g.S == 1 && g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0 && rows <= 16 && g.C % 64 == 0 && g.C >= 64 * DF_WAVES &&
           (unsigned long long)g.K * g.C * 2 < (1ull << 32);
}

hipError_t dense_fwd_stream(const ConvGeom &g, unsigned flags, const bf16_t *x, const bf16_t *w, const float *bias, bf16_t *y, hipStream_t st)
{
    const int rows = g.N * g.Ho * g.Wo, blocks = (g.K + 15) / 16;
    if (rows <= 16) hipLaunchKernelGGL(k_dense_fwd<1>, dim3((unsigned)blocks), dim3(64 * DF_WAVES), 0, st, rows, g.C, g.K, flags, x, w, bias, y);
    else hipLaunchKernelGGL(k_dense_fwd<2>, dim3((unsigned)blocks), dim3(64 * DF_WAVES), 0, st, rows, g.C, g.K, flags, x, w, bias, y);
    return hipGetLastError();
}

// shapes the streaming dense backward-data takes: a 1x1 layer over at most 32 pixel rows whose output features do not come in whole
// 64-row reduction steps, which keeps the pipelined tile kernels away (the classifier layer with its 1000 outputs); input and output
// features in whole 8-element chunks (16-byte loads), enough output rows to give every wave of a block a few steps.  Where the
// pipelined kernels do run they are as fast (measured on 25088 x 4096 and 4096 x 4096: both forms read the 128-byte column strips
// of W at about 4 TB/s), so they keep those shapes.
bool dense_dgrad_stream_shape(const ConvGeom &g)
{
    const long long rows = (long long)g.N * g.H * g.W;
    return g.R == 1 && g.S == 1 && g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0 && rows <= 32 && g.C % 8 == 0 && g.K % 8 == 0 &&
           g.K % 64 != 0 && g.K >= 16 * DF_WAVES && (unsigned long long)g.K * g.C * 2 < (1ull << 32);
}

hipError_t dense_dgrad_stream(const ConvGeom &g, unsigned flags, const bf16_t *dy, const bf16_t *w, const bf16_t *xin, void *dx, hipStream_t st)
{
    const int rows = g.N * g.H * g.W, blocks = (g.C + 63) / 64;
    hipLaunchKernelGGL(k_dense_dgrad, dim3((unsigned)blocks), dim3(64 * DF_WAVES), 0, st, rows, g.C, g.K, flags, dy, w, xin, dx);
    return hipGetLastError();
}

// shapes the streaming dense filter gradient takes: a 1x1 layer over at most 32 pixel rows, features in whole 8-element chunks,
// a gradient of 4 to 128 MB (measured: 4096 x 4096 28 -> 21 us and 4096 x 1000 19 -> 14 us against the pipelined tile kernel,
// which in turn writes the 411 MB of the 25088 x 4096 layer 15 us faster with its 128 x 128 tiles)
bool dense_wgrad_stream_shape(const ConvGeom &g)
{
    const long long rows = (long long)g.N * g.Ho * g.Wo, elems = (long long)g.K * g.C;
    return g.R == 1 && g.S == 1 && g.sh == 1 && g.sw == 1 && g.ph == 0 && g.pw == 0 && rows <= 32 && g.C % 8 == 0 && g.K % 8 == 0 &&
           elems >= (1 << 20) && elems <= (32 << 20);
}

hipError_t dense_wgrad_stream(const ConvGeom &g, const bf16_t *x, const bf16_t *dy, float *dw, float *db, hipStream_t st)
{
    const int rows = g.N * g.Ho * g.Wo;
    const dim3 grid((unsigned)((g.K + 63) / 64), (unsigned)((g.C + 64 * DF_WAVES - 1) / (64 * DF_WAVES)));
    if ((size_t)g.K * g.C * 4 >= ((size_t)32 << 20)) hipLaunchKernelGGL(k_dense_wgrad<true>, grid, dim3(64 * DF_WAVES), 0, st, rows, g.C, g.K, x, dy, dw, db);
    else hipLaunchKernelGGL(k_dense_wgrad<false>, grid, dim3(64 * DF_WAVES), 0, st, rows, g.C, g.K, x, dy, dw, db);
    return hipGetLastError();
}

const char *dense_fwd_stream_name(const ConvGeom &g) { return g.N * g.Ho * g.Wo <= 16 ? "k_dense_fwd<1>" : "k_dense_fwd<2>"; }
const char *dense_wgrad_stream_name(const ConvGeom &g) { return (size_t)g.K * g.C * 4 >= ((size_t)32 << 20) ? "k_dense_wgrad<true>" : "k_dense_wgrad<false>"; }
