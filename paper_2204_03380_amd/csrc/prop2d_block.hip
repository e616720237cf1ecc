// 2-D propagation of small jobs for gfx950: two or three time steps per
// launch, one workgroup per block of rows.
//
// A marching strip (prop2d_multi.hip) is a serial chain of rows.  When a job
// has few strips per CU, that chain is the launch: 27 rows for nine owned
// ones.  Here a workgroup of NW wavefronts owns a block of NW * RW rows by
// 64 * VEC columns, RW consecutive rows per wavefront, kept in registers:
//  - every load of the launch is issued at the start (one memory latency);
//  - step one takes its neighbour rows from memory with the same loads;
//  - later steps take the four rows above and below a wavefront's own from
//    an LDS copy of the level (double-buffered: one barrier per step);
//  - x-neighbours come from the adjacent lanes through DPP.
// Blocks overlap as the marching strips do: T steps own the inner
// 64 VEC - 8 (T - 1) columns and NW RW - 8 (T - 1) rows.  Step s is exact on
// the rows and columns within 4 (T - s) of the owned ones; wavefronts with
// none of these rows sit the step out.  Every cell's arithmetic is the
// one-step kernels', operation for operation.
//
// What bounds it: the latency of the launch, of the table reads and of the
// one round of loads; with several rounds of blocks per CU, the vector
// instructions (a block of 48 rows computes 40 rows a step on average for
// its 32, on 128 columns for 112).  us per step, blocks against marching
// strips: 201 x 201 with a 40-cell band forward 1.8 against 3.5, reverse 3.2
// against 6.1; 1574 x 534 2.95 against 4.6, 6.1 against 8.8; 4 shots of
// 2301 x 751 forward 13.9 against 15.0.  Shapes (VEC/NW/RW) measured on 201 x
// 201 (forward): 1/8/4 1.88, 2/16/2 2.28, 1/16/4 2.50, 2/16/3 2.76; on 800 x
// 450: 2/12/3 2.47, 1/8/4 2.73, 2/16/3 2.85; on 1574 x 534: 2/16/3 2.95,
// 2/8/4 3.06, 2/12/3 3.38, 2/16/4 3.53, 1/8/4 3.72.
#include "multi2d.h"


namespace rtm {
namespace {

// The kernels' shape Z: VEC floats per lane, NW wavefronts, RW rows each.

// What a wavefront needs to know about its block.  Field pointers point at
// column xs of padded row 0.  Rows and columns outside the stored ones are
// read from the zero halo instead (their values are zero and stay zero), so
// no load needs a guard.
struct Blk {
    unsigned pitch4;
    int xs, x, NZr, z0, z1, r0, lane, w;
    unsigned lx, hx, cx;  // byte offsets as in the marching kernels
    int s0;       // rows [s0, s0 + sn) hold the block's source nodes
    unsigned sn;
    bool own, ends;
    __device__ __forceinline__ int64_t row(int r) const
    {
        return (int64_t)min(max(r, -kRadius), NZr + kRadius - 1) * pitch4;
    }
};

template <class Z, int T>
__device__ __forceinline__ Blk make_blk(ShotEntry &S, TileEntry &t)
{
    Blk B;
    const int NX = S.L.NX;
    B.pitch4 = (unsigned)S.L.pitch * 4u;
    B.NZr = S.L.NZr;
    B.lane = threadIdx.x & 63;
    B.w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    B.xs = t.x0;
    B.z0 = t.z0;
    B.z1 = t.z1;
    B.r0 = t.z0 - 4 * (T - 1) + B.w * Z::RW;
    B.x = B.xs + B.lane * Z::VEC;
    B.lx = (unsigned)(min(B.x, (NX + Z::VEC - 1) / Z::VEC * Z::VEC) - B.xs) * 4u;
    B.hx = B.lane == 0 ? 0u : (unsigned)(min(B.xs + 64 * Z::VEC, (NX + 3) & ~3) - B.xs + 4) * 4u;
    B.cx = (unsigned)(B.lane * Z::VEC) * 4u;
    B.own = B.x >= B.xs + 4 * (T - 1) && B.x + Z::VEC <= B.xs + 64 * Z::VEC - 4 * (T - 1) && B.x < NX;
    B.ends = ((B.lane + 1) & 63) <= 1;
    B.s0 = 0;
    B.sn = 0;
    return B;
}

template <int T>
__device__ __forceinline__ SrcLane blk_sources(Blk &B, TileEntry &t, const InjEnt *__restrict__ ents,
                                               const Contrib *__restrict__ cont, const float *wav, int dir,
                                               bool want_sum)
{
    if (t.s1end == t.s1beg) return SrcLane{-(1 << 30), 0, 0, 0.f, 0.f};
    const SrcLane src = src_load<T>(t, ents, cont, wav, dir, B.lane, want_sum);
    // the first step's list holds every node of the others; sorted by row
    B.s0 = __builtin_amdgcn_readlane(src.z, 0);
    B.sn = (unsigned)(__builtin_amdgcn_readlane(src.z, t.s1end - t.s1beg - 1) + 1 - B.s0);
    return src;
}

template <int N, int VEC>
__device__ __forceinline__ void blk_load(const Blk &B, const gfloat *f, int r, float (&q)[N][VEC])
{
#pragma unroll
    for (int i = 0; i < N; ++i) ldv<VEC>(at(at(f, B.row(r + i)), here(B.lx)), q[i]);
}

// Strip-end halo of the wavefront's own rows (meaningful in lanes 0 and 63).
template <int RW>
__device__ __forceinline__ void blk_load_ends(const Blk &B, const gfloat *f, f4v (&h)[RW])
{
#pragma unroll
    for (int i = 0; i < RW; ++i) h[i] = f4v{0.f, 0.f, 0.f, 0.f};
    if (B.ends) {
#pragma unroll
        for (int i = 0; i < RW; ++i) h[i] = *(const gf4v *)at(at(f, B.row(B.r0 + i)) - 4, here(B.hx));
    }
}

// Does step s of T need any row of this wavefront?
template <class Z>
__device__ __forceinline__ bool blk_active(const Blk &B, int left)
{
    return B.r0 + Z::RW > B.z0 - 4 * left && B.r0 < B.z1 + 4 * left;  // left = T - s
}

// Laplacian sum of own row i; q holds rows r0 - 4 .. r0 + RW + 3.
template <int N, int VEC>
__device__ __forceinline__ void blk_lap(const float (&q)[N][VEC], int i, bool first, const f4v &h, int lane, float (&lap)[VEC])
{
    float ext[VEC + 8];
    if (first) {
        float hl[4], hr[4];
        halo_split(h, lane, hl, hr);
        exchange_row<VEC>(q[i + 4], hl, hr, ext);
    } else {
        exchange_row0<VEC>(q[i + 4], ext);
    }
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        const float c = q[i + 4][j], c2 = c + c;
        float l = d2(c2, ext[3 + j], ext[5 + j], ext[2 + j], ext[6 + j], ext[1 + j], ext[7 + j], ext[j], ext[8 + j]);
        l += d2(c2, q[i + 3][j], q[i + 5][j], q[i + 2][j], q[i + 6][j], q[i + 1][j], q[i + 7][j], q[i][j], q[i + 8][j]);
        lap[j] = l;
    }
}

// LDS copy of a level: the block's rows and four more on each side (never
// written; what a step reads there only reaches rows it does not need).
template <class Z>
struct BlkRows {
    float row[Z::NW * Z::RW + 8][64 * Z::VEC];
};

template <class Z>
__device__ __forceinline__ void blk_publish(BlkRows<Z> &L, const Blk &B, const float (&q)[Z::RW + 8][Z::VEC])
{
#pragma unroll
    for (int i = 0; i < Z::RW; ++i)
#pragma unroll
        for (int j = 0; j < Z::VEC; ++j) L.row[4 + B.w * Z::RW + i][B.lane * Z::VEC + j] = q[4 + i][j];
}

// Rows above and below the wavefront's own.
template <class Z>
__device__ __forceinline__ void blk_neighbours(const BlkRows<Z> &L, const Blk &B, float (&q)[Z::RW + 8][Z::VEC])
{
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < Z::VEC; ++j) {
            q[i][j] = L.row[B.w * Z::RW + i][B.lane * Z::VEC + j];
            q[Z::RW + 4 + i][j] = L.row[B.w * Z::RW + Z::RW + 4 + i][B.lane * Z::VEC + j];
        }
}

template <class Z>
__device__ __forceinline__ void blk_own(const BlkRows<Z> &L, const Blk &B, float (&q)[Z::RW + 8][Z::VEC])
{
#pragma unroll
    for (int i = 0; i < Z::RW; ++i)
#pragma unroll
        for (int j = 0; j < Z::VEC; ++j) q[4 + i][j] = L.row[4 + B.w * Z::RW + i][B.lane * Z::VEC + j];
}

// Adds the source of step s to the wavefront's rows v (row r0 first).
template <int RW, int VEC>
__device__ __forceinline__ void src_add(const SrcLane &src, int s, const Blk &B, const float (&d)[RW][VEC], float (&v)[RW][VEC])
{
#pragma unroll
    for (int i = 0; i < RW; ++i)
        if (in_rows(B.r0 + i, B.s0, B.sn))
            src_row<VEC>(src, s, B.r0 + i, B.x, [&](int j, float val, int) __attribute__((always_inline)) {
                v[i][j] = fmaf(d[i][j], val, v[i][j]);
            });
}

// A receiver node of the block, one per thread and step, loaded with the
// fields: its place in the LDS copy, signal sum and D'.
struct RecLane {
    int at;  // row * columns + column, -1: none
    float val, d;
};

template <class Z, int T>
__device__ __forceinline__ RecLane rec_make(const Blk &B, const InjEnt *__restrict__ ents,
                                            const Contrib *__restrict__ cont, const float *sig, const gfloat *Dp, int e,
                                            int end)
{
    RecLane R{-1, 0.f, 0.f};
    if (e >= end) return R;
    const InjEnt E = ents[e];
    R.at = (E.z - (B.z0 - 4 * (T - 1)) + 4) * (64 * Z::VEC) + (E.x - B.xs);
    R.d = at(Dp, (int64_t)E.z * B.pitch4)[E.x - B.xs];
    R.val = inj_sum(E, cont, sig);
    return R;
}

// Stores the owned cells of rows [lo, hi) of a level.
template <int N, int VEC>
__device__ __forceinline__ void blk_store(const Blk &B, gfloat *f, const float (&q)[N][VEC], int lo, int hi)
{
#pragma unroll
    for (int i = 0; i < N - 8; ++i) {
        const int r = B.r0 + i;
        if (r >= lo && r < hi && B.own) stv<VEC>(at(at(f, (int64_t)r * B.pitch4), here(B.cx)), q[4 + i]);
    }
}

}  // namespace

// Forward: levels n + 1 .. n + T of every block from n and n - 1; the last
// two are stored into the second field set.  Receivers as in the marching
// kernels: with three steps, level n + 1 is stored on the receiver rows, and
// the workgroups past the stencil slots record d^{n-2} (T = 3), d^{n-1} and
// d^n, one receiver task per wavefront.
template <class Z, int T>
__global__ __launch_bounds__(64 * Z::NW) void fwd2d_block_kernel(const ShotDev *__restrict__ shots,
                                                                 const Tile2D *__restrict__ tiles, int ntiles,
                                                                 int nslots, const InjEnt *__restrict__ ents,
                                                                 const Contrib *__restrict__ cont,
                                                                 const SampleTask *__restrict__ stasks, int nsample,
                                                                 int n)
{
    const int b = blockIdx.x;
    if (b >= nslots) {
        const int t = (b - nslots) * Z::NW + (int)(threadIdx.x >> 6);
        if (t >= T * nsample) return;
        const int g = t / nsample, level = n - (T - 1) + g;
        if (T == 3 && g == 0) {
            if (n >= 3) sample_body(shots, stasks[t], level, 6, (int)(threadIdx.x & 63));
        } else if (level >= 0) {
            sample_body(shots, stasks[t - g * nsample], level, level & 1, (int)(threadIdx.x & 63));
        }
        return;
    }
    const int t = xcd_tile(b, nslots);
    if (t >= ntiles) return;  // whole workgroup
    TileEntry &tile = *(TileEntry *)(uintptr_t)(tiles + t);
    ShotEntry &S = *(ShotEntry *)(uintptr_t)(shots + tile.shot);
    __shared__ BlkRows<Z> L[2];
    Blk B = make_blk<Z, T>(S, tile);
    const int64_t org = S.L.org + tile.x0;
    const gfloat *pc = gp(S.fld[n & 1] + org), *pm = gp(S.fld[(n + 1) & 1] + org);
    const gfloat *Dp = gp(S.Dp + org);

    constexpr int RW = Z::RW, VEC = Z::VEC;
    float q[RW + 8][VEC], old[RW][VEC], d[RW][VEC], v[RW][VEC];
    f4v h[RW];
    if (blk_active<Z>(B, T - 1)) {
        blk_load(B, pc, B.r0 - 4, q);
        blk_load_ends(B, pc, h);
        blk_load(B, pm, B.r0, old);
        blk_load(B, Dp, B.r0, d);
    }
    const SrcLane src = blk_sources<T>(B, tile, ents, cont, S.wav + n, 1, false);
#pragma unroll
    for (int s = 1; s <= T; ++s) {
        if (s > 1) {
            blk_publish<Z>(L[s & 1], B, q);
            __syncthreads();
        }
        if (!blk_active<Z>(B, T - s)) continue;
        if (s > 1) blk_neighbours<Z>(L[s & 1], B, q);
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            float lap[VEC];
            blk_lap(q, i, s == 1, h[i], B.lane, lap);
#pragma unroll
            for (int j = 0; j < VEC; ++j) v[i][j] = fmaf(d[i][j], lap[j], (q[4 + i][j] + q[4 + i][j]) - old[i][j]);
        }
        src_add(src, s, B, d, v);
#pragma unroll
        for (int i = 0; i < RW; ++i)
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                old[i][j] = q[4 + i][j];
                q[4 + i][j] = v[i][j];
            }
        if (T == 3 && s == 1 && nsample > 0)
            blk_store(B, gp(S.fld[2] + org), q, max(tile.z0, S.sz0), min(tile.z1, S.sz1));
        if (s >= T - 1) blk_store(B, gp(S.fld[4 + ((n + s) & 1)] + org), q, tile.z0, tile.z1);
    }
}

// Reverse: steps k .. k - T + 1 of the reconstruction and the receiver
// field, with the imaging sums (num, den read and written once per T steps)
// or the gradient sum (GRAD).  Receiver terms are added to the LDS copy of
// the new mu level by one thread per node, from which the owning wavefronts
// then take their rows back (only in blocks that hold receiver nodes).
template <class Z, int T, bool GRAD>
__global__ __launch_bounds__(64 * Z::NW) void rev2d_block_kernel(const ShotDev *__restrict__ shots,
                                                                 const Tile2D *__restrict__ tiles, int ntiles,
                                                                 int nslots, const InjEnt *__restrict__ ents,
                                                                 const Contrib *__restrict__ cont, int k,
                                                                 int reinject, float *__restrict__ wadj)
{
    const int t = xcd_tile(blockIdx.x, nslots);
    if (t >= ntiles) return;  // whole workgroup
    TileEntry &tile = *(TileEntry *)(uintptr_t)(tiles + t);
    ShotEntry &S = *(ShotEntry *)(uintptr_t)(shots + tile.shot);
    __shared__ BlkRows<Z> LP[2], LM[2];
    Blk B = make_blk<Z, T>(S, tile);
    const int64_t org = S.L.org + tile.x0;
    const gfloat *P0 = gp(S.fld[k & 1] + org), *P1 = gp(S.fld[(k + 1) & 1] + org);
    const gfloat *M0 = gp(S.fld[2 + ((k + 1) & 1)] + org), *M1 = gp(S.fld[2 + (k & 1)] + org);
    const gfloat *Dp = gp(S.Dp + org);
    gfloat *A0 = gp(S.acc0 + org);
    gfloat *A1 = GRAD ? nullptr : gp(S.acc1 + org);
    // rows and lanes whose sums this wavefront keeps
    constexpr int RW = Z::RW, VEC = Z::VEC;
    const bool alane = GRAD ? B.own : B.own && B.x + VEC > S.ix0 && B.x < S.ix1;
    const int alo = GRAD ? tile.z0 : max(tile.z0, S.iz0), ahi = GRAD ? tile.z1 : min(tile.z1, S.iz1);

    float qp[RW + 8][VEC], qm[RW + 8][VEC], op[RW][VEC], om[RW][VEC], d[RW][VEC], vp[RW][VEC], vm[RW][VEC], a[RW][VEC],
        c[RW][VEC];
    f4v hp[RW], hm[RW];
    if (blk_active<Z>(B, T - 1)) {
        blk_load(B, P0, B.r0 - 4, qp);
        blk_load(B, M0, B.r0 - 4, qm);
        blk_load_ends(B, P0, hp);
        blk_load_ends(B, M0, hm);
        blk_load(B, P1, B.r0, op);
        blk_load(B, M1, B.r0, om);
        blk_load(B, Dp, B.r0, d);
        blk_load(B, A0, B.r0, a);
        if constexpr (!GRAD) blk_load(B, A1, B.r0, c);
    }
    const SrcLane src = blk_sources<T>(B, tile, ents, cont, S.wav + k, -1, GRAD && wadj);
    const float *sig = S.sig + (int64_t)k * S.nrec;  // at time k; step s takes k - s + 1
    const int nrec = S.nrec;
    RecLane rec[T] = {};
    if (tile.r1end > tile.r1beg) {
#pragma unroll
        for (int s = 1; s <= T; ++s) {
            int eb, ee;
            rec_range<T>(tile, s, eb, ee);
            rec[s - 1] = rec_make<Z, T>(B, ents, cont, sig - (int64_t)(s - 1) * nrec, Dp, eb + (int)threadIdx.x, ee);
        }
    }
#pragma unroll
    for (int s = 1; s <= T; ++s) {
        const bool active = blk_active<Z>(B, T - s);
        if (active) {
            if (s > 1) {
                blk_neighbours<Z>(LP[s & 1], B, qp);
                blk_neighbours<Z>(LM[s & 1], B, qm);
            }
#pragma unroll
            for (int i = 0; i < RW; ++i) {
                float lp[VEC], lm[VEC];
                blk_lap(qp, i, s == 1, hp[i], B.lane, lp);
                blk_lap(qm, i, s == 1, hm[i], B.lane, lm);
#pragma unroll
                for (int j = 0; j < VEC; ++j) {
                    const float cp = qp[4 + i][j], cm = qm[4 + i][j];
                    if constexpr (GRAD) {
                        a[i][j] = fmaf(cm, d[i][j] * lp[j], a[i][j]);
                    } else {
                        a[i][j] = fmaf(cp, cm, a[i][j]);
                        c[i][j] = fmaf(cp, cp, c[i][j]);
                    }
                    vp[i][j] = fmaf(d[i][j], lp[j], (cp + cp) - op[i][j]);
                    vm[i][j] = fmaf(d[i][j], lm[j], (cm + cm) - om[i][j]);
                }
            }
            if constexpr (GRAD) {
#pragma unroll
                for (int i = 0; i < RW; ++i) {
                    if (!in_rows(B.r0 + i, B.s0, B.sn)) continue;
                    const bool mine = B.own && B.r0 + i >= tile.z0 && B.r0 + i < tile.z1;
                    src_row<VEC>(src, s, B.r0 + i, B.x, [&](int j, float val, int l) __attribute__((always_inline)) {
                        if (!mine) return;  // another block's
                        a[i][j] = fmaf(qm[4 + i][j], d[i][j] * val, a[i][j]);
                        if (wadj) {
                            const float wsum = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(src.wsum), l));
                            wadj[(int64_t)(k - s + 1) * kMaxNodes + __builtin_amdgcn_readlane(src.slot, l)] = wsum * qm[4 + i][j];
                        }
                    });
                }
            }
            if (reinject) src_add(src, s, B, d, vp);
#pragma unroll
            for (int i = 0; i < RW; ++i)
#pragma unroll
                for (int j = 0; j < VEC; ++j) {
                    op[i][j] = qp[4 + i][j];
                    om[i][j] = qm[4 + i][j];
                    qp[4 + i][j] = vp[i][j];
                    qm[4 + i][j] = vm[i][j];
                }
        }
        int rb, re;
        rec_range<T>(tile, s, rb, re);
        if (s < T) blk_publish<Z>(LP[(s + 1) & 1], B, qp);
        if (s < T || re > rb) {
            BlkRows<Z> &L = LM[(s + 1) & 1];
            blk_publish<Z>(L, B, qm);
            __syncthreads();
            if (re > rb) {
                float *lm = &L.row[0][0];
                if (rec[s - 1].at >= 0) lm[rec[s - 1].at] = fmaf(rec[s - 1].d, rec[s - 1].val, lm[rec[s - 1].at]);
                for (int e = rb + (int)threadIdx.x + 64 * Z::NW; e < re; e += 64 * Z::NW) {
                    const RecLane R = rec_make<Z, T>(B, ents, cont, sig - (int64_t)(s - 1) * nrec, Dp, e, re);
                    lm[R.at] = fmaf(R.d, R.val, lm[R.at]);
                }
                __syncthreads();
                blk_own<Z>(L, B, qm);
            }
        }
        if (active && s >= T - 1) {
            blk_store(B, gp(S.fld[4 + ((k - s) & 1)] + org), qp, tile.z0, tile.z1);
            blk_store(B, gp(S.fld[6 + ((k - s + 1) & 1)] + org), qm, tile.z0, tile.z1);
        }
    }
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int r = B.r0 + i;
        if (r >= alo && r < ahi && alane) {
            stv<VEC>(at(at(A0, (int64_t)r * B.pitch4), here(B.cx)), a[i]);
            if constexpr (!GRAD) stv<VEC>(at(at(A1, (int64_t)r * B.pitch4), here(B.cx)), c[i]);
        }
    }
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------

namespace {

template <int I>
struct Shape {
    static constexpr int VEC = kBlockShapes[I].vec, NW = kBlockShapes[I].waves, RW = kBlockShapes[I].rows;
};

template <class Z, int T>
void fwd_launch(const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots, const InjEnt *ents,
                const Contrib *cont, const SampleTask *stasks, int nsample, int n, hipStream_t st)
{
    const dim3 grid(nslots + (T * nsample + Z::NW - 1) / Z::NW), block(64 * Z::NW);
    hipLaunchKernelGGL((fwd2d_block_kernel<Z, T>), grid, block, 0, st, shots, tiles, ntiles, nslots, ents, cont, stasks,
                       nsample, n);
}

template <class Z, int T>
void rev_launch(bool grad, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots, const InjEnt *ents,
                const Contrib *cont, int k, int reinject, float *wadj, hipStream_t st)
{
    const dim3 grid(nslots), block(64 * Z::NW);
    if (grad)
        hipLaunchKernelGGL((rev2d_block_kernel<Z, T, true>), grid, block, 0, st, shots, tiles, ntiles, nslots, ents,
                           cont, k, reinject, wadj);
    else
        hipLaunchKernelGGL((rev2d_block_kernel<Z, T, false>), grid, block, 0, st, shots, tiles, ntiles, nslots, ents,
                           cont, k, reinject, wadj);
}

}  // namespace

#define RTM_SHAPES(CALL)                        \
    switch (shape) {                            \
    case 1: CALL(1); break;                     \
    case 2: CALL(2); break;                     \
    case 3: CALL(3); break;                     \
    default: return hipErrorInvalidValue;       \
    }                                           \
    return hipGetLastError();

hipError_t launch_fwd2d_block(int shape, int steps, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                              const InjEnt *ents, const Contrib *cont, const SampleTask *stasks, int nsample, int n,
                              hipStream_t st)
{
#define RTM_CALL(I)                                                                                     \
    if (steps == 3)                                                                                     \
        fwd_launch<Shape<I>, 3>(shots, tiles, ntiles, nslots, ents, cont, stasks, nsample, n, st);       \
    else                                                                                                \
        fwd_launch<Shape<I>, 2>(shots, tiles, ntiles, nslots, ents, cont, stasks, nsample, n, st)
    RTM_SHAPES(RTM_CALL)
#undef RTM_CALL
}

hipError_t launch_rev2d_block(int shape, int steps, bool grad, const ShotDev *shots, const Tile2D *tiles, int ntiles,
                              int nslots, const InjEnt *ents, const Contrib *cont, int k, int reinject, float *wadj,
                              hipStream_t st)
{
#define RTM_CALL(I)                                                                                           \
    if (steps == 3)                                                                                           \
        rev_launch<Shape<I>, 3>(grad, shots, tiles, ntiles, nslots, ents, cont, k, reinject, wadj, st);        \
    else                                                                                                      \
        rev_launch<Shape<I>, 2>(grad, shots, tiles, ntiles, nslots, ents, cont, k, reinject, wadj, st)
    RTM_SHAPES(RTM_CALL)
#undef RTM_CALL
}

}  // namespace rtm
