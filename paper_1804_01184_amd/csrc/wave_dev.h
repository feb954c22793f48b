// Device helpers shared by the batched kernels: buffer accesses, row offsets,
// whole-wave shifts and the horizontal differences built on them.
#pragma once

#include "fwi2d_internal.h"

namespace fwi {

namespace {

constexpr int WAVE = 64;
constexpr int HALO = 3;

// Buffer accesses: a uniform resource per record group, a uniform byte
// offset for the row (scalar offset) and a per-lane byte offset for the
// column.  A lane offset of kOOB lies past every resource, so its loads
// return 0 (ghost cells outside the grid, cells without an absorbing-layer
// split, rows past the band) and its stores are dropped (halo lanes).  The
// host keeps every resource and every row offset below 2^31 bytes, and
// every resource is followed by at least kSlack allocated bytes (the lane
// holding the last grid column may read past it; those values are masked).
using rsrc_t = __amdgpu_buffer_rsrc_t;
constexpr unsigned kOOB = 0x80000000u;
constexpr int kRsrcWord3 = 0x00020000;
constexpr unsigned kSlack = 16;
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ inline rsrc_t res(const float *p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, (short)0, (int)(bytes + kSlack), kRsrcWord3);
}
// (the buffer builtins move raw 32-bit words: bit casts, not conversions)
__device__ inline float bld(rsrc_t r, unsigned voff, unsigned soff)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0));
}
__device__ inline void bst(rsrc_t r, unsigned voff, unsigned soff, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)voff, (int)soff, 0);
}
// Vector components are copied to scalars before the bit cast: a bit cast
// of a component expression (x.y) is not lowered to that component.
template <int C>
__device__ inline void vld(rsrc_t r, unsigned voff, unsigned soff, float (&o)[C])
{
    if constexpr (C == 1) {
        o[0] = bld(r, voff, soff);
    } else if constexpr (C == 2) {
        const u32x2 x = __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const unsigned e = x[c];
            o[c] = __builtin_bit_cast(float, e);
        }
    } else {
        const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const unsigned e = x[c];
            o[c] = __builtin_bit_cast(float, e);
        }
    }
}
template <int C>
__device__ inline void vst(rsrc_t r, unsigned voff, unsigned soff, const float (&v)[C])
{
    if constexpr (C == 1) {
        bst(r, voff, soff, v[0]);
    } else if constexpr (C == 2) {
        u32x2 x;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float e = v[c];
            x[c] = __builtin_bit_cast(unsigned, e);
        }
        __builtin_amdgcn_raw_buffer_store_b64(x, r, (int)voff, (int)soff, 0);
    } else {
        u32x4 x;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float e = v[c];
            x[c] = __builtin_bit_cast(unsigned, e);
        }
        __builtin_amdgcn_raw_buffer_store_b128(x, r, (int)voff, (int)soff, 0);
    }
}

// by-value min / max (reference-returning overloads applied to kernel
// arguments would force a private copy of the argument struct)
__device__ inline int imin(int a, int b) { return a < b ? a : b; }

// Read-only tables seen through the constant address space: a load at a
// uniform index becomes a scalar load, which keeps the per-row table values
// off the vector memory path (the kernels' stores would otherwise stop the
// compiler from proving the tables unchanged inside the row loops).
typedef const __attribute__((address_space(4))) float cfloat;
__device__ inline cfloat *ctab(const float *p) { return (cfloat *)p; }
typedef const __attribute__((address_space(4))) unsigned cuint;
typedef const __attribute__((address_space(4))) int cint;
__device__ inline int imax(int a, int b) { return a > b ? a : b; }
__device__ inline int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ inline int xcd_item(int b, int nb)
{
    int q = nb >> 3;
    if (b >= (q << 3))
        return b;
    return (b & 7) * q + (b >> 3);
}

// Neighbour exchange by whole-wave DPP shifts (register moves, no LDS):
// lane l receives the value of lane l + 1 (shift left) or l - 1 (shift
// right); the end lanes, which have no such neighbour, receive 0, and only
// halo lanes ever use it.
constexpr int kDppWaveShl1 = 0x130, kDppWaveShr1 = 0x138;
template <int CTRL>
__device__ inline float wave_shift(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL,
                                                              0xf, 0xf, true));
}
__device__ inline float from_right(float v) { return wave_shift<kDppWaveShl1>(v); }
__device__ inline float from_left(float v) { return wave_shift<kDppWaveShr1>(v); }

// Fourth-order staggered differences of a row held C columns per lane
// (without the 1/h factor).  Forward: at j + 1/2 from the nodes j-1 .. j+2;
// backward: at node j from the half nodes j-3/2 .. j+1/2 (stored at j-2 .. j+1).
template <int C>
__device__ inline void dfwd(const float (&v)[C], float (&d)[C])
{
    const float r0 = from_right(v[0]);                          // column C
    const float r1 = C >= 2 ? from_right(v[C >= 2 ? 1 : 0]) : from_right(r0);  // column C+1
    const float l1 = from_left(v[C - 1]);                       // column -1
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const float p1 = c + 1 < C ? v[c + 1 < C ? c + 1 : 0] : r0;
        const float p2 = c + 2 < C ? v[c + 2 < C ? c + 2 : 0] : (c + 2 == C ? r0 : r1);
        const float m1 = c >= 1 ? v[c >= 1 ? c - 1 : 0] : l1;
        d[c] = kC1 * (p1 - v[c]) + kC2 * (p2 - m1);
    }
}
template <int C>
__device__ inline void dbwd(const float (&v)[C], float (&d)[C])
{
    const float l1 = from_left(v[C - 1]);                                      // column -1
    const float l2 = C >= 2 ? from_left(v[C >= 2 ? C - 2 : 0]) : from_left(l1);  // column -2
    const float r0 = from_right(v[0]);                                         // column C
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const float m1 = c >= 1 ? v[c >= 1 ? c - 1 : 0] : l1;
        const float m2 = c >= 2 ? v[c >= 2 ? c - 2 : 0] : (c == 1 ? l1 : l2);
        const float p1 = c + 1 < C ? v[c + 1 < C ? c + 1 : 0] : r0;
        d[c] = kC1 * (v[c] - m1) + kC2 * (p1 - m2);
    }
}

__device__ inline bool row_ok(const Geo &g, int i) { return (unsigned)i < (unsigned)g.Nz; }

// Byte offset of row i (uniform).
__device__ inline unsigned rowb(const Geo &g, int i) { return 4u * (unsigned)i * (unsigned)g.Nx; }

// Split (absorbing-layer) index of row i: uniform row base + lane part.  On
// the top and bottom strips every column has a split (full rows); on middle
// rows only the side columns.  With no layer every lane part is kOOB.
struct ZRow {
    unsigned base;
    bool full;
};
__device__ inline ZRow zrow(const Geo &g, int i)
{
    const bool top = i < g.npml, bot = i >= g.Nz - g.npml;
    ZRow z;
    z.full = top || bot;
    const int fr = top ? i : i - (g.Nz - 2 * g.npml);
    z.base = z.full ? 4u * (unsigned)fr * (unsigned)g.Nx
                    : 4u * (unsigned)(2 * g.npml * g.Nx + (i - g.npml) * 2 * g.npml);
    return z;
}
// Select between two lane values.  The empty asm makes both operands
// values first, so the choice is not turned into a choice between two
// addresses of the wave geometry (which would keep it in scratch memory).
__device__ inline unsigned pick(bool c, unsigned a, unsigned b)
{
    asm("" : "+v"(a), "+v"(b));
    return c ? a : b;
}

}  // namespace

}  // namespace fwi
