// Device helpers shared by the kernels that fill LDS with direct-to-LDS buffer loads: buffer
// resources, the 16-byte copy, explicit waits, and LDS fragment reads as inline assembly (the compiler
// would otherwise wait for every outstanding copy before any LDS read it can see).
#pragma once
#include "tile_common.h"
#include <utility>
#include <type_traits>

namespace {

constexpr unsigned OOR = 0xFFFFFFFFu;
typedef __attribute__((address_space(3))) void *lds_void;

DEVFN __amdgpu_buffer_rsrc_t make_rsrc(const void *p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(unsigned)bytes, 0x00020000);
}
// 16 bytes per lane from the buffer straight into LDS at lds_base + lane*16 (lds_base wave-uniform)
DEVFN void dma16(__amdgpu_buffer_rsrc_t r, unsigned lds_base, unsigned voff)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void)(size_t)lds_base, 16, voff, 0, 0, 0);
}
// the same copy with the non-temporal hint: for operands that are read exactly once (allocating them in the caches
// would push out dirty lines that then have to be written back in the middle of the stream)
DEVFN void dma16_nt(__amdgpu_buffer_rsrc_t r, unsigned lds_base, unsigned voff)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void)(size_t)lds_base, 16, voff, 0, 0, 2);
}
DEVFN unsigned lds_offset(const void *p) { return (unsigned)(size_t)(__attribute__((address_space(3))) const char *)p; }

// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>): a loop whose index is a constant expression in the body
template <typename F, int... I> DEVFN void for_constant_impl(F &&f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, typename F> DEVFN void for_constant(F &&f) { for_constant_impl(f, std::make_integer_sequence<int, N>{}); }

template <int N> DEVFN void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// the same for a count known only at run time (uniform); counts not listed wait for everything
DEVFN void wait_copies(int n)
{
    switch (n) {
    case 12: wait_vmcnt<12>(); break;
    case 11: wait_vmcnt<11>(); break;
    case 10: wait_vmcnt<10>(); break;
    case 9: wait_vmcnt<9>(); break;
    case 8: wait_vmcnt<8>(); break;
    case 7: wait_vmcnt<7>(); break;
    case 6: wait_vmcnt<6>(); break;
    case 5: wait_vmcnt<5>(); break;
    case 4: wait_vmcnt<4>(); break;
    case 3: wait_vmcnt<3>(); break;
    case 2: wait_vmcnt<2>(); break;
    case 1: wait_vmcnt<1>(); break;
    default: wait_vmcnt<0>();
    }
}

template <int OFF> DEVFN u32x4 lds_read16(unsigned addr)
{
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}


// issue the fragment reads of one 16-wide reduction slice (blocks of 32 rows are BS bytes apart)
template <int FA, int FB, int BS>
DEVFN void read_frags(u32x4 (&a)[FA], u32x4 (&b)[FB], unsigned pa, unsigned pb)
{
    if constexpr (FA >= 1) a[0] = lds_read16<0>(pa);
    if constexpr (FA >= 2) a[1] = lds_read16<BS>(pa);
    if constexpr (FA >= 3) a[2] = lds_read16<2 * BS>(pa);
    if constexpr (FA >= 4) a[3] = lds_read16<3 * BS>(pa);
    if constexpr (FB >= 1) b[0] = lds_read16<0>(pb);
    if constexpr (FB >= 2) b[1] = lds_read16<BS>(pb);
    if constexpr (FB >= 3) b[2] = lds_read16<2 * BS>(pb);
    if constexpr (FB >= 4) b[3] = lds_read16<3 * BS>(pb);
}
// The reads are invisible to the compiler: wait until at most N newer LDS reads are outstanding,
// with the fragments as operands so that no matrix instruction using them is scheduled earlier.
template <int N, int FA, int FB>
DEVFN void wait_frags(u32x4 (&a)[FA], u32x4 (&b)[FB])
{
    static_assert(N >= 0 && N < 16, "lgkmcnt is a 4-bit counter");
    asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N));
    // volatile statements keep their order; the empty ones make the fragments depend on the wait
#pragma unroll
    for (int i = 0; i < FA; ++i) asm volatile("" : "+v"(a[i]));
#pragma unroll
    for (int j = 0; j < FB; ++j) asm volatile("" : "+v"(b[j]));
}

// Valid-tap mask of a pixel row: bit r*S+s is set iff 0 <= hb + sg*r < Hlim and 0 <= wb + sg*s < Wlim.
DEVFN unsigned tap_mask(int hb, int wb, int sg, int R, int S, int Hlim, int Wlim)
{
    unsigned smask = 0;
    for (int s = 0; s < S; ++s) smask |= ((unsigned)(wb + sg * s) < (unsigned)Wlim) ? 1u << s : 0u;
    unsigned mask = 0;
    for (int r = 0; r < R; ++r) mask |= ((unsigned)(hb + sg * r) < (unsigned)Hlim) ? smask << (r * S) : 0u;
    return mask;
}

// Tiles of a persistent block.  Consecutive block ids go round-robin to the 8 XCDs, each with an L2 of its own: XCD x (blocks x,
// x + 8, ...) walks one contiguous eighth of the tile list, its blocks side by side, so that tiles that share halo pixels (left /
// right neighbours, and the row of tiles above / below) run on one XCD at about the same time and the second reader of a halo pixel
// finds it in that L2.  (Dealing the tiles out block by block over the whole chip, every halo pixel was fetched from memory again: L2
// hit rate 0.09 on conv1_2, and the copies of a CU are bound by its ~64 outstanding misses.)  Other counts of blocks than whole eighths, which the
// 3x3 kernels take with 3, 5, 6 or 7 channel tiles, are dealt out that way all the same.
struct TileWalk { int first, end, stride; };
DEVFN TileWalk tile_walk(int tiles)
{
    const int nb = gridDim.x;
    if ((nb & 7) != 0) return {(int)blockIdx.x, tiles, nb};
    const int x = blockIdx.x & 7;
    return {(int)((long long)tiles * x / 8) + (int)(blockIdx.x >> 3), (int)((long long)tiles * (x + 1) / 8), nb >> 3};
}

template <int T> DEVFN int seg_swz(int t)
{
    constexpr int SPR = T / 32, RPS = T >= 128 ? 1 : 128 / T;   // segments per row, rows per 256 bytes
    return (t / RPS) & (SPR >= 4 ? 3 : SPR - 1);
}

DEVFN void lds_write16(unsigned addr, u32x4 v) { asm volatile("ds_write_b128 %0, %1" ::"v"(addr), "v"(v) : "memory"); }

template <int OFF> DEVFN u32x2 lds_read_tr(unsigned addr)
{
    u32x2 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}


}  // namespace
