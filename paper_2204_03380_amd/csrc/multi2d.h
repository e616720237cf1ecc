// Device helpers of the 2-D kernels that take several time steps per launch
// (and, where they apply, of the 3-D kernels): addressing without guards,
// table access through the scalar cache, cache-bypassing access, lane shifts
// with zero ends, source nodes held in lanes.
#pragma once

#include "stencil.h"

namespace rtm {
namespace {

__device__ __forceinline__ float dpp_shr1z(float src)
{
    // wave_shr:1 - lane i receives lane i-1; lane 0 receives zero.
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(src), 0x138, 0xf, 0xf, true));
}

__device__ __forceinline__ float dpp_shl1z(float src)
{
    // wave_shl:1 - lane i receives lane i+1; lane 63 receives zero.
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(src), 0x130, 0xf, 0xf, true));
}

// exchange_row with zeros beyond the strip ends.
template <int VEC>
__device__ __forceinline__ void exchange_row0(const float (&c)[VEC], float (&ext)[VEC + 8])
{
    constexpr int K = 4 / VEC;
    float L[VEC], Rr[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) ext[4 + j] = L[j] = Rr[j] = c[j];
#pragma unroll
    for (int k = 1; k <= K; ++k)
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            L[j] = dpp_shr1z(L[j]);
            Rr[j] = dpp_shl1z(Rr[j]);
            ext[4 - k * VEC + j] = L[j];
            ext[4 + VEC + (k - 1) * VEC + j] = Rr[j];
        }
}

typedef __attribute__((address_space(1))) char gchar;
__device__ __forceinline__ const gfloat *at(const gfloat *f, int64_t bytes)
{
    return (const gfloat *)((const gchar *)f + bytes);
}
__device__ __forceinline__ gfloat *at(gfloat *f, int64_t bytes) { return (gfloat *)((gchar *)f + bytes); }
__device__ __forceinline__ const gfloat *at(const gfloat *f, unsigned bytes)
{
    return (const gfloat *)((const gchar *)f + bytes);
}
__device__ __forceinline__ gfloat *at(gfloat *f, unsigned bytes) { return (gfloat *)((gchar *)f + bytes); }

// Byte offset of a row that advances by one row at a time and stays on the
// stored rows [-4, NZr + 4): rows outside them are read from the zero halo
// instead, so that no load needs a guard.
struct RowAt {
    int64_t off;
    unsigned r;  // row + 4
    __device__ __forceinline__ void start(int row, unsigned pitch4, int NZr)
    {
        r = (unsigned)(row + kRadius);
        off = (int64_t)min(max(row, -kRadius), NZr + kRadius - 1) * pitch4;
    }
    __device__ __forceinline__ void next(unsigned pitch4, int NZr)
    {
        off += r < (unsigned)(NZr + 2 * kRadius - 1) ? pitch4 : 0u;
        ++r;
    }
};

// Is lo <= r < lo + n?
__device__ __forceinline__ bool in_rows(int r, int lo, unsigned n) { return (unsigned)(r - lo) < n; }

// Entries of the shot and tile tables, which no kernel writes, read through
// the scalar cache (their index is uniform), so that everything derived from
// them stays in scalar registers.
typedef __attribute__((address_space(4))) const ShotDev ShotEntry;
typedef __attribute__((address_space(4))) const Tile2D TileEntry;

// Access to values that a launch touches once (new levels, imaging sums; in
// the 3-D kernels also the older level and D').  NT leaves them out of the way
// in the L2, whose lines then last until the neighbouring tiles have read the
// halo rows they share.
template <int VEC, bool NT>
__device__ __forceinline__ void ld_once(const gfloat *p, float (&v)[VEC])
{
    if constexpr (!NT) {
        ldv<VEC>(p, v);
    } else if constexpr (VEC == 4) {
        const f4v t = __builtin_nontemporal_load((const gf4v *)p);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else if constexpr (VEC == 2) {
        const f2v t = __builtin_nontemporal_load((const gf2v *)p);
        v[0] = t.x; v[1] = t.y;
    } else {
        v[0] = __builtin_nontemporal_load(p);
    }
}

template <int VEC, bool NT>
__device__ __forceinline__ void st_once(gfloat *p, const float (&v)[VEC])
{
    if constexpr (!NT)
        stv<VEC>(p, v);
    else if constexpr (VEC == 4)
        __builtin_nontemporal_store(f4v{v[0], v[1], v[2], v[3]}, (gf4v *)p);
    else if constexpr (VEC == 2)
        __builtin_nontemporal_store(f2v{v[0], v[1]}, (gf2v *)p);
    else
        __builtin_nontemporal_store(v[0], p);
}

// The value again, opaque to the compiler: the 64-bit extension of a byte
// offset then stays next to its use, where it folds into the access (a
// scalar address plus a 32-bit vector offset).
__device__ __forceinline__ unsigned here(unsigned v)
{
    asm("" : "+v"(v));
    return v;
}

// Source nodes of the strip, one per lane, loaded before the march: lanes
// 8 (s - 1) .. 8 (s - 1) + 7 hold the list of step s (at most four nodes)
// with its signal value, so that a row with a source waits for no load.
struct SrcLane {
    int z, x, slot;
    float val, wsum;
};

template <int T>
__device__ __forceinline__ void src_range(TileEntry &t, int s, int &beg, int &end)
{
    beg = s == T ? t.sbeg : (s == 1 ? t.s1beg : t.s2beg);
    end = s == T ? t.send : (s == 1 ? t.s1end : t.s2end);
}

template <int T>
__device__ __forceinline__ void rec_range(TileEntry &t, int s, int &beg, int &end)
{
    beg = s == T ? t.rbeg : (s == 1 ? t.r1beg : t.r2beg);
    end = s == T ? t.rend : (s == 1 ? t.r1end : t.r2end);
}

// wav: the wavelet at step one's time; dir: +1 forward, -1 reverse.
template <int T>
__device__ __forceinline__ SrcLane src_load(TileEntry &t, const InjEnt *__restrict__ ents,
                                            const Contrib *__restrict__ cont, const float *wav, int dir, int lane,
                                            bool want_sum)
{
    SrcLane s{-(1 << 30), 0, 0, 0.f, 0.f};
    const int step = (lane >> 3) + 1;
    if (step > T) return s;
    int beg, end;
    src_range<T>(t, step, beg, end);
    const int e = beg + (lane & 7);
    if (e >= end) return s;
    const InjEnt E = ents[e];
    s.z = E.z;
    s.x = E.x;
    s.slot = E.slot;
    s.val = inj_sum(E, cont, wav + dir * (step - 1));
    if (want_sum)
        for (int c = E.cbeg; c < E.cend; ++c) s.wsum += cont[c].w;
    return s;
}

// Source terms of step s in row r: add(column offset j, value) at the lane
// that holds the node.
template <int VEC, class F>
__device__ __forceinline__ void src_row(const SrcLane &src, int s, int r, int x, F add)
{
    #pragma unroll 1
    for (int e = 0; e < 4; ++e) {
        const int l = 8 * (s - 1) + e;
        if (__builtin_amdgcn_readlane(src.z, l) != r) continue;
        const int sx = __builtin_amdgcn_readlane(src.x, l);
        const float val = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(src.val), l));
#pragma unroll
        for (int j = 0; j < VEC; ++j)
            if (sx == x + j) add(j, val, l);
    }
}

}  // namespace
}  // namespace rtm
