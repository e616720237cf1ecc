// 2-D propagation for gfx950, two or three time steps per launch: marching
// strips.
//
// One wavefront covers a strip of 64 * VEC columns and marches down the rows
// of its tile.  With T steps per launch a strip overlaps its neighbours by
// 8 (T - 1) columns and owns the inner 64 VEC - 8 (T - 1).  March step s
//  (1) advances the first level at row r1 = z0 - 4 (T - 1) + s on the whole
//      strip (the strip-end halo comes with one load by lanes 0 and 63);
//  (2) advances the second level four rows behind, exact on the columns 4
//      further in;
//  (3) with T = 3, the third level eight rows behind, exact on the owned
//      columns.
// Queue slot (S + i) mod 9 holds row r1 - 4 + i of every queue (S = s mod 9,
// a compile-time constant: the march is unrolled by nine), so step two's
// centre row sits in slot S and step three's in slot (S + 5) mod 9.  The
// first 9 (T - 1) march steps, where the later steps have no rows yet, are
// separate code: the main loop computes every step unconditionally, without
// register copies at the joins.  Only the last two levels are stored (with
// T = 3, modeling also stores level n + 1 on the rows that hold receiver
// nodes), so the level pairs and D' cross HBM once per T steps.  Every
// cell's arithmetic equals the one-step kernels', operation for operation.
//
// What bounds it.  A launch that fills the chip (48 shots of 2301 x 751) is
// bound by HBM traffic and, in the forward pass, by vector instructions at
// 88 % busy; hence the zero-guard addressing below (scalar row addresses, a
// 32-bit lane offset, clamped rows): 4442 vector instructions for 27 rows of
// fwd2d_multi<2, 3> against 2581 for 9 with guards and 64-bit lane addresses
// (forward 156.7 -> 149.9 us per step, reverse 413.7 -> 413.4).  Stores of new
// levels and the imaging sums that bypass the caches where the arrays exceed
// them (NT) take forward 150 -> 143 and reverse 413 -> 378: the traffic is
// nearly the same (240 shots, reverse: 31.0 -> 30.5 GB a launch), it moves at
// 5.6 instead of 5.2 TB/s.  Bypassing on the loads too, 146 and 391: strips
// overlap, and D' is shared by the shots.  With fewer
// than about four wavefronts per SIMD each row waits for its own loads, so
// P = 3 loads them three march steps ahead into a ring of registers
// (16 shots, forward: 64.3 -> 52.7 us per step, 55.3 without the ring; 2
// shots, reverse: 25.9 -> 20.6; the gradient of 12 windows: 24.8 -> 19.4).
// Jobs of few blocks take the block kernels (prop2d_block.hip) instead.
#include "multi2d.h"

namespace rtm {
// prop2d_block.hip
hipError_t launch_fwd2d_block(int shape, int steps, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                              const InjEnt *ents, const Contrib *cont, const SampleTask *stasks, int nsample, int n,
                              hipStream_t st);
hipError_t launch_rev2d_block(int shape, int steps, bool grad, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                              const InjEnt *ents, const Contrib *cont, int k, int reinject, float *wadj,
                              hipStream_t st);

namespace {

template <int VEC, int C>
__device__ __forceinline__ void lap_at(const float (&q)[9][VEC], const float (&ext)[VEC + 8], float (&lap)[VEC])
{
    constexpr int m1 = (C + 8) % 9, p1 = (C + 1) % 9, m2 = (C + 7) % 9, p2 = (C + 2) % 9, m3 = (C + 6) % 9,
                  p3 = (C + 3) % 9, m4 = (C + 5) % 9, p4 = (C + 4) % 9;
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        const float c = q[C][j], c2 = c + c;
        float l = d2(c2, ext[3 + j], ext[5 + j], ext[2 + j], ext[6 + j], ext[1 + j], ext[7 + j], ext[j], ext[8 + j]);
        l += d2(c2, q[m1][j], q[p1][j], q[m2][j], q[p2][j], q[m3][j], q[p3][j], q[m4][j], q[p4][j]);
        lap[j] = l;
    }
}

// What every marching strip knows of its tile.  Field pointers point at
// column xs of padded row 0.
struct Strip {
    unsigned pitch4;  // bytes per stored row
    // byte offsets from column xs, unsigned 32-bit so that an access takes a
    // scalar row address plus one vector register:
    unsigned lx;  // this lane's columns inside the stored ones
    unsigned hx;  // strip-end halo columns of lanes 0 and 63, from xs - 4
    unsigned cx;  // this lane's columns
    int x, xs, NZr, lane, z0, z1, r0;  // r0: row of march step 0
    unsigned zn;                       // z1 - z0
    bool own, ends;
};

template <int VEC, int T>
__device__ __forceinline__ Strip make_strip(ShotEntry &S, TileEntry &t)
{
    Strip C;
    const int NX = S.L.NX, xs = t.x0;
    C.pitch4 = (unsigned)S.L.pitch * 4u;
    C.NZr = S.L.NZr;
    C.lane = threadIdx.x;
    C.xs = xs;
    C.x = xs + C.lane * VEC;
    C.cx = (unsigned)(C.lane * VEC) * 4u;
    C.lx = (unsigned)(min(C.x, (NX + VEC - 1) / VEC * VEC) - xs) * 4u;
    C.hx = C.lane == 0 ? 0u : (unsigned)(min(xs + 64 * VEC, (NX + 3) & ~3) - xs + 4) * 4u;
    C.z0 = t.z0;
    C.z1 = t.z1;
    C.zn = (unsigned)(t.z1 - t.z0);
    C.r0 = t.z0 - 4 * (T - 1);
    C.own = C.x >= xs + 4 * (T - 1) && C.x + VEC <= xs + 64 * VEC - 4 * (T - 1) && C.x < NX;
    C.ends = ((C.lane + 1) & 63) <= 1;
    return C;
}

// Eight rows from row r on into slots 0 .. 7 of a queue.
template <int VEC>
__device__ __forceinline__ void strip_fill(const Strip &C, const gfloat *f, int r, float (&q)[9][VEC])
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        RowAt a;
        a.start(r + i, C.pitch4, C.NZr);
        ldv<VEC>(at(at(f, a.off), here(C.lx)), q[i]);
    }
}

// ---------------------------------------------------------------------------
// Forward
// ---------------------------------------------------------------------------

template <int VEC, int T>
struct FwdMulti {
    const gfloat *pc, *pm, *Dp;
    gfloat *wa, *wb, *mid;  // levels n + T - 1, n + T; n + 1 on rows [m0, m0 + mn)
    unsigned mn, sn;
    int m0, s0;  // [s0, s0 + sn): rows with source nodes
    Strip C;
};

// What a row of step one needs from memory, loaded P rows ahead.
template <int VEC>
struct FwdIn {
    float q[VEC], old[VEC], d[VEC];
    f4v h;
};

// Loads row r1 (ra: r1, rq: r1 + 4), then advances both.
template <int VEC, int T, bool AHEAD>
__device__ __forceinline__ void fwd_fetch(const FwdMulti<VEC, T> &K, RowAt &ra, RowAt &rq, FwdIn<VEC> &in)
{
    const unsigned lx = here(K.C.lx);
    ldv<VEC>(at(at(K.pc, rq.off), lx), in.q);
    ldv<VEC>(at(at(K.pm, ra.off), lx), in.old);
    ldv<VEC>(at(at(K.Dp, ra.off), lx), in.d);
    if constexpr (AHEAD)
        if (K.C.ends) in.h = *(const gf4v *)at(at(K.pc, ra.off) - 4, here(K.C.hx));
    ra.next(K.C.pitch4, K.C.NZr);
    rq.next(K.C.pitch4, K.C.NZr);
    if constexpr (!AHEAD)
        if (K.C.ends) in.h = *(const gf4v *)at(at(K.pc, ra.off) - 4, here(K.C.hx));
}

// March step s = 9 i + S (PH = min(i, 2)): step one of row r1 = r0 + s, step
// two of row r1 - 4 from s = 8 on, step three of row r1 - 8 from s = 16 on.
template <int VEC, int T, int P, bool NT, int PH, int S>
__device__ __forceinline__ void fwd_row(const FwdMulti<VEC, T> &K, float (&q1)[9][VEC], float (&q2)[9][VEC],
                                           float (&q3)[9][VEC], float (&qd)[9][VEC], FwdIn<VEC> (&in)[P > 0 ? P : 1],
                                           const SrcLane &src, RowAt &ra, RowAt &rq, int64_t &o1, int r1)
{
    constexpr int a0 = S % 9, a4 = (S + 4) % 9, a5 = (S + 5) % 9, a8 = (S + 8) % 9;
    const Strip &C = K.C;
    const int r2 = r1 - 4, r3 = r1 - 8;
    FwdIn<VEC> &I = in[P > 0 ? S % (P > 0 ? P : 1) : 0];
    const f4v h = I.h;
    if constexpr (P == 0) fwd_fetch<VEC, T, false>(K, ra, rq, I);
    float hl[4], hr[4], ext[VEC + 8], lap[VEC], v[VEC], d[VEC], old[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        q1[a8][j] = I.q[j];
        d[j] = I.d[j];
        old[j] = I.old[j];
    }
    halo_split(h, C.lane, hl, hr);
    exchange_row<VEC>(q1[a4], hl, hr, ext);
    if constexpr (P > 0) fwd_fetch<VEC, T, true>(K, ra, rq, I);
    lap_at<VEC, a4>(q1, ext, lap);
#pragma unroll
    for (int j = 0; j < VEC; ++j) v[j] = fmaf(d[j], lap[j], (q1[a4][j] + q1[a4][j]) - old[j]);
    if (in_rows(r1, K.s0, K.sn)) src_row<VEC>(src, 1, r1, C.x, [&](int j, float s, int) __attribute__((always_inline)) { v[j] = fmaf(d[j], s, v[j]); });
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        q2[a4][j] = v[j];
        qd[a4][j] = d[j];
    }
    if constexpr (T == 3) {
        if (in_rows(r1, K.m0, K.mn) && C.own) st_once<VEC, NT>(at(at(K.mid, o1), here(C.cx)), v);
    } else {
        if (in_rows(r1, C.z0, C.zn) && C.own) st_once<VEC, NT>(at(at(K.wa, o1), here(C.cx)), v);
    }
    if constexpr (PH > 0 || S == 8) {
        exchange_row0<VEC>(q2[a0], ext);
        lap_at<VEC, a0>(q2, ext, lap);
#pragma unroll
        for (int j = 0; j < VEC; ++j) v[j] = fmaf(qd[a0][j], lap[j], (q2[a0][j] + q2[a0][j]) - q1[a0][j]);
        if (in_rows(r2, K.s0, K.sn)) src_row<VEC>(src, 2, r2, C.x, [&](int j, float s, int) __attribute__((always_inline)) { v[j] = fmaf(qd[a0][j], s, v[j]); });
        if constexpr (T == 3)
#pragma unroll
            for (int j = 0; j < VEC; ++j) q3[a0][j] = v[j];
        if (in_rows(r2, C.z0, C.zn) && C.own) st_once<VEC, NT>(at(at(T == 3 ? K.wa : K.wb, o1 - 4 * (int64_t)C.pitch4), here(C.cx)), v);
    }
    if constexpr (T == 3 && (PH > 1 || (PH == 1 && S >= 7))) {
        exchange_row0<VEC>(q3[a5], ext);
        lap_at<VEC, a5>(q3, ext, lap);
#pragma unroll
        for (int j = 0; j < VEC; ++j) v[j] = fmaf(qd[a5][j], lap[j], (q3[a5][j] + q3[a5][j]) - q2[a5][j]);
        if (in_rows(r3, K.s0, K.sn)) src_row<VEC>(src, 3, r3, C.x, [&](int j, float s, int) __attribute__((always_inline)) { v[j] = fmaf(qd[a5][j], s, v[j]); });
        if (r3 < C.z1 && C.own) st_once<VEC, NT>(at(at(K.wb, o1 - 8 * (int64_t)C.pitch4), here(C.cx)), v);
    }
    o1 += C.pitch4;
}

// ROW(phase, S, s) for nine march steps.
#define RTM_NINE(ROW, PH, s)                                                                    \
    ROW(PH, 0, s); ROW(PH, 1, s + 1); ROW(PH, 2, s + 2); ROW(PH, 3, s + 3); ROW(PH, 4, s + 4);   \
    ROW(PH, 5, s + 5); ROW(PH, 6, s + 6); ROW(PH, 7, s + 7); ROW(PH, 8, s + 8);

// ---------------------------------------------------------------------------
// Reverse
// ---------------------------------------------------------------------------

// Receiver nodes of one step, in LDS: a chunk of the tile's list (sorted by
// row) with the signal sums, loaded before the march, so that a row with
// receivers waits for no load.  next: first list entry not yet in a chunk.
template <int VEC>
struct RecLds {
    int z[64 * VEC + 1], col[64 * VEC];  // z[64 VEC]: past the last row
    float val[64 * VEC];
};

struct RecList {
    int next, end, cur, row;  // uniform; row: of the first node not yet added
};

template <int VEC>
__device__ __forceinline__ void rec_chunk(RecLds<VEC> &L, RecList &R, const InjEnt *__restrict__ ents,
                                          const Contrib *__restrict__ cont, const float *sig, int xs, int lane)
{
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        const int i = R.next + 64 * j + lane;
        int z = 1 << 30;
        if (i < R.end) {
            const InjEnt E = ents[i];
            z = E.z;
            L.col[64 * j + lane] = E.x - xs;
            L.val[64 * j + lane] = inj_sum(E, cont, sig);
        }
        L.z[64 * j + lane] = z;
    }
    R.next = min(R.next + 64 * VEC, R.end);
    R.cur = 0;
    __syncthreads();
    R.row = __builtin_amdgcn_readfirstlane(L.z[0]);
}

// Adds D' times the receiver sums of row r into v.  The workgroup is this
// wavefront; r, R and the branches are uniform.  sv, has: one slot per
// column, has zero on entry.
template <int VEC>
__device__ __forceinline__ void rec_row(RecLds<VEC> &L, RecList &R, const InjEnt *__restrict__ ents,
                                        const Contrib *__restrict__ cont, const float *sig, int xs, int lane, int r,
                                        const float (&d)[VEC], float (&v)[VEC], float *sv, int *has)
{
    do {
        int n = 0;
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            const int i = 64 * j + lane;
            const bool mine = i >= R.cur && L.z[i] == r;
            if (mine) {
                sv[L.col[i]] = L.val[i];
                has[L.col[i]] = 1;
            }
            n += __popcll(__ballot(mine));
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            const int c = lane * VEC + j;
            if (has[c]) {
                v[j] = fmaf(d[j], sv[c], v[j]);
                has[c] = 0;
            }
        }
        __syncthreads();
        R.cur += n;
        if (R.cur == 64 * VEC && R.next < R.end)
            rec_chunk<VEC>(L, R, ents, cont, sig, xs, lane);
        else
            R.row = __builtin_amdgcn_readfirstlane(L.z[R.cur]);
    } while (R.row == r);
}

template <int VEC, int T, bool GRAD>
struct RevMulti {
    const gfloat *P0, *P1, *M0, *M1, *Dp;
    gfloat *WPa, *WPb, *WMa, *WMb;  // p^{k-T+1}, p^{k-T}; mu^{k-T+2}, mu^{k-T+1}
    gfloat *A0, *A1;                // num, den | G
    float *wadj;
    const InjEnt *ents;
    const Contrib *cont;
    const float *sig;               // receiver signal at time k
    RecLds<VEC> *rl;                // LDS, one per step
    float *sv;
    int *has;
    int nrec, k, s0, alo;
    unsigned sn, an;
    bool alane, reinject;
    Strip C;
};

template <int VEC, bool GRAD>
struct RevIn {
    float p0[VEC], m0[VEC], p1[VEC], m1[VEC], d[VEC], g[GRAD ? VEC : 1];
    f4v hp, hm;
};

template <int VEC, int T, bool GRAD>
__device__ __forceinline__ void rev_ends(const RevMulti<VEC, T, GRAD> &K, const RowAt &ra, RevIn<VEC, GRAD> &in)
{
    if (K.C.ends) {
        in.hp = *(const gf4v *)at(at(K.P0, ra.off) - 4, here(K.C.hx));
        in.hm = *(const gf4v *)at(at(K.M0, ra.off) - 4, here(K.C.hx));
    }
}

template <int VEC, int T, bool GRAD, bool AHEAD>
__device__ __forceinline__ void rev_fetch(const RevMulti<VEC, T, GRAD> &K, RowAt &ra, RowAt &rq, RevIn<VEC, GRAD> &in)
{
    const unsigned lx = here(K.C.lx);
    ldv<VEC>(at(at(K.P0, rq.off), lx), in.p0);
    ldv<VEC>(at(at(K.M0, rq.off), lx), in.m0);
    ldv<VEC>(at(at(K.P1, ra.off), lx), in.p1);
    ldv<VEC>(at(at(K.M1, ra.off), lx), in.m1);
    ldv<VEC>(at(at(K.Dp, ra.off), lx), in.d);
    if constexpr (GRAD) ldv<VEC>(at(at(K.A0, ra.off), lx), in.g);
    if constexpr (AHEAD) rev_ends<VEC, T, GRAD>(K, ra, in);
    ra.next(K.C.pitch4, K.C.NZr);
    rq.next(K.C.pitch4, K.C.NZr);
    if constexpr (!AHEAD) rev_ends<VEC, T, GRAD>(K, ra, in);
}

// Source terms of step s at row r of the reconstruction (into v) and, in the
// gradient pass, of the gradient sum g and the wavelet adjoint (mu: the
// receiver field the row's gradient term took).
template <int VEC, int T, bool GRAD>
__device__ __forceinline__ void rev_src(const RevMulti<VEC, T, GRAD> &K, const SrcLane &src, int s, int r,
                                        const float (&d)[VEC], const float (&mu)[VEC], float (&v)[VEC], float *g)
{
    if (!in_rows(r, K.s0, K.sn)) return;
    const bool mine = K.C.own && in_rows(r, K.C.z0, K.C.zn);
    src_row<VEC>(src, s, r, K.C.x, [&](int j, float val, int l) __attribute__((always_inline)) {
        if constexpr (GRAD) {
            if (mine) {
                g[j] = fmaf(mu[j], d[j] * val, g[j]);
                if (K.wadj) {
                    const float wsum = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(src.wsum), l));
                    const int slot = __builtin_amdgcn_readlane(src.slot, l);
                    K.wadj[(int64_t)(K.k - s + 1) * kMaxNodes + slot] = wsum * mu[j];
                }
            }
        }
        if (K.reinject) v[j] = fmaf(d[j], val, v[j]);
    });
}

// March step s = 9 i + S (PH = min(i, 2)), rows as in the forward march.
// Imaging: all terms of a row are added at step two's row r2, where p^k,
// mu^{k+1} (step two's previous levels), p^{k-1}, mu^k (its centre) and, with
// three steps, the new p^{k-2}, mu^{k-1} are in registers.  Gradient: the
// row's sum travels through the queue qg, taking each step's term where
// that step is computed.
template <int VEC, int T, int P, bool NT, bool GRAD, int PH, int S>
__device__ __forceinline__ void rev_row(const RevMulti<VEC, T, GRAD> &K, float (&q1p)[9][VEC], float (&q1m)[9][VEC],
                                           float (&q2p)[9][VEC], float (&q2m)[9][VEC], float (&q3p)[9][VEC],
                                           float (&q3m)[9][VEC], float (&qd)[9][VEC], float (&qg)[9][VEC],
                                           RevIn<VEC, GRAD> (&in)[P > 0 ? P : 1], float (&ia)[VEC], float (&ib)[VEC],
                                           const SrcLane &src, RecList (&R)[T], RowAt &ra, RowAt &rq, int64_t &o1,
                                           int r1)
{
    constexpr int a0 = S % 9, a4 = (S + 4) % 9, a5 = (S + 5) % 9, a8 = (S + 8) % 9;
    const Strip &C = K.C;
    const int r2 = r1 - 4, r3 = r1 - 8;
    RevIn<VEC, GRAD> &I = in[P > 0 ? S % (P > 0 ? P : 1) : 0];
    const f4v tp = I.hp, tm = I.hm;
    if constexpr (P == 0) rev_fetch<VEC, T, GRAD, false>(K, ra, rq, I);
    float hl[4], hr[4], ext[VEC + 8], lap[VEC], vp[VEC], vm[VEC], d[VEC], p1[VEC], m1[VEC], g[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        q1p[a8][j] = I.p0[j];
        q1m[a8][j] = I.m0[j];
        d[j] = I.d[j];
        p1[j] = I.p1[j];
        m1[j] = I.m1[j];
        if constexpr (GRAD) g[j] = I.g[j];
    }
    if constexpr (!GRAD && P == 0) {
        if (in_rows(r2, K.alo, K.an) && K.alane) {
            ld_once<VEC, NT>(at(at(K.A0, o1 - 4 * (int64_t)C.pitch4), here(C.cx)), ia);
            ld_once<VEC, NT>(at(at(K.A1, o1 - 4 * (int64_t)C.pitch4), here(C.cx)), ib);
        }
    }
    if constexpr (P > 0) rev_fetch<VEC, T, GRAD, true>(K, ra, rq, I);
    halo_split(tp, C.lane, hl, hr);
    exchange_row<VEC>(q1p[a4], hl, hr, ext);
    lap_at<VEC, a4>(q1p, ext, lap);
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        if constexpr (GRAD) g[j] = fmaf(q1m[a4][j], d[j] * lap[j], g[j]);
        vp[j] = fmaf(d[j], lap[j], (q1p[a4][j] + q1p[a4][j]) - p1[j]);
    }
    halo_split(tm, C.lane, hl, hr);
    exchange_row<VEC>(q1m[a4], hl, hr, ext);
    lap_at<VEC, a4>(q1m, ext, lap);
#pragma unroll
    for (int j = 0; j < VEC; ++j) vm[j] = fmaf(d[j], lap[j], (q1m[a4][j] + q1m[a4][j]) - m1[j]);
    rev_src<VEC, T, GRAD>(K, src, 1, r1, d, q1m[a4], vp, g);
    if (R[0].row == r1)
        rec_row<VEC>(K.rl[0], R[0], K.ents, K.cont, K.sig, C.xs, C.lane, r1, d, vm, K.sv, K.has);
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        q2p[a4][j] = vp[j];
        q2m[a4][j] = vm[j];
        qd[a4][j] = d[j];
        if constexpr (GRAD) qg[a4][j] = g[j];
    }
    if constexpr (T == 2)
        if (in_rows(r1, C.z0, C.zn) && C.own) {
            st_once<VEC, NT>(at(at(K.WPa, o1), here(C.cx)), vp);
            st_once<VEC, NT>(at(at(K.WMa, o1), here(C.cx)), vm);
        }
    if constexpr (PH > 0 || S == 8) {
        exchange_row0<VEC>(q2p[a0], ext);
        lap_at<VEC, a0>(q2p, ext, lap);
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            if constexpr (GRAD) qg[a0][j] = fmaf(q2m[a0][j], qd[a0][j] * lap[j], qg[a0][j]);
            vp[j] = fmaf(qd[a0][j], lap[j], (q2p[a0][j] + q2p[a0][j]) - q1p[a0][j]);
        }
        exchange_row0<VEC>(q2m[a0], ext);
        lap_at<VEC, a0>(q2m, ext, lap);
#pragma unroll
        for (int j = 0; j < VEC; ++j) vm[j] = fmaf(qd[a0][j], lap[j], (q2m[a0][j] + q2m[a0][j]) - q1m[a0][j]);
        rev_src<VEC, T, GRAD>(K, src, 2, r2, qd[a0], q2m[a0], vp, qg[a0]);
        if (R[1].row == r2)
            rec_row<VEC>(K.rl[1], R[1], K.ents, K.cont, K.sig - K.nrec, C.xs, C.lane, r2, qd[a0], vm, K.sv, K.has);
        const bool mine = in_rows(r2, C.z0, C.zn);
        if (mine && C.own) {
            const int64_t o2 = o1 - 4 * (int64_t)C.pitch4;
            st_once<VEC, NT>(at(at(T == 3 ? K.WPa : K.WPb, o2), here(C.cx)), vp);
            st_once<VEC, NT>(at(at(T == 3 ? K.WMa : K.WMb, o2), here(C.cx)), vm);
            if constexpr (GRAD && T == 2) st_once<VEC, NT>(at(at(K.A0, o2), here(C.cx)), qg[a0]);
        }
        if constexpr (!GRAD) {
            if (in_rows(r2, K.alo, K.an) && K.alane) {
                float sa[VEC], sb[VEC];
#pragma unroll
                for (int j = 0; j < VEC; ++j) {  // levels k, k - 1 (and k - 2) in turn
                    sa[j] = fmaf(q2p[a0][j], q2m[a0][j], fmaf(q1p[a0][j], q1m[a0][j], ia[j]));
                    sb[j] = fmaf(q2p[a0][j], q2p[a0][j], fmaf(q1p[a0][j], q1p[a0][j], ib[j]));
                    if constexpr (T == 3) {
                        sa[j] = fmaf(vp[j], vm[j], sa[j]);
                        sb[j] = fmaf(vp[j], vp[j], sb[j]);
                    }
                }
                st_once<VEC, NT>(at(at(K.A0, o1 - 4 * (int64_t)C.pitch4), here(C.cx)), sa);
                st_once<VEC, NT>(at(at(K.A1, o1 - 4 * (int64_t)C.pitch4), here(C.cx)), sb);
            }
        }
        if constexpr (T == 3)
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                q3p[a0][j] = vp[j];
                q3m[a0][j] = vm[j];
            }
    }
    if constexpr (!GRAD && P > 0) {
        // the next row's sums
        if (in_rows(r2 + 1, K.alo, K.an) && K.alane) {
            ld_once<VEC, NT>(at(at(K.A0, o1 - 3 * (int64_t)C.pitch4), here(C.cx)), ia);
            ld_once<VEC, NT>(at(at(K.A1, o1 - 3 * (int64_t)C.pitch4), here(C.cx)), ib);
        }
    }
    if constexpr (T == 3 && (PH > 1 || (PH == 1 && S >= 7))) {
        exchange_row0<VEC>(q3p[a5], ext);
        lap_at<VEC, a5>(q3p, ext, lap);
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            if constexpr (GRAD) qg[a5][j] = fmaf(q3m[a5][j], qd[a5][j] * lap[j], qg[a5][j]);
            vp[j] = fmaf(qd[a5][j], lap[j], (q3p[a5][j] + q3p[a5][j]) - q2p[a5][j]);
        }
        exchange_row0<VEC>(q3m[a5], ext);
        lap_at<VEC, a5>(q3m, ext, lap);
#pragma unroll
        for (int j = 0; j < VEC; ++j) vm[j] = fmaf(qd[a5][j], lap[j], (q3m[a5][j] + q3m[a5][j]) - q2m[a5][j]);
        rev_src<VEC, T, GRAD>(K, src, 3, r3, qd[a5], q3m[a5], vp, qg[a5]);
        if (R[T - 1].row == r3)
            rec_row<VEC>(K.rl[T - 1], R[T - 1], K.ents, K.cont, K.sig - 2 * K.nrec, C.xs, C.lane, r3, qd[a5], vm, K.sv,
                         K.has);
        if (r3 < C.z1 && C.own) {
            const int64_t o3 = o1 - 8 * (int64_t)C.pitch4;
            st_once<VEC, NT>(at(at(K.WPb, o3), here(C.cx)), vp);
            st_once<VEC, NT>(at(at(K.WMb, o3), here(C.cx)), vm);
            if constexpr (GRAD) st_once<VEC, NT>(at(at(K.A0, o3), here(C.cx)), qg[a5]);
        }
    }
    o1 += C.pitch4;
}

}  // namespace

// Steps n .. n + T - 1 of every tile; workgroups past the stencil slots
// record receivers from the read set.
template <int VEC, int T, int P, bool NT>
__global__ __launch_bounds__(64) void fwd2d_multi_kernel(const ShotDev *__restrict__ shots,
                                                      const Tile2D *__restrict__ tiles, int ntiles, int nslots,
                                                      const InjEnt *__restrict__ ents,
                                                      const Contrib *__restrict__ cont,
                                                      const SampleTask *__restrict__ stasks, int nsample, int n)
{
    const int b = blockIdx.x;
    const int lane = threadIdx.x;
    if (b >= nslots) {
        const int t = b - nslots, g = t / nsample, level = n - (T - 1) + g;
        if (T == 3 && g == 0) {
            if (n >= 3) sample_body(shots, stasks[t], level, 6, lane);
        } else if (level >= 0) {
            sample_body(shots, stasks[t - g * nsample], level, level & 1, lane);
        }
        return;
    }
    const int t = xcd_tile(b, nslots);
    if (t >= ntiles) return;
    TileEntry &tile = *(TileEntry *)(uintptr_t)(tiles + t);
    ShotEntry &S = *(ShotEntry *)(uintptr_t)(shots + tile.shot);
    FwdMulti<VEC, T> K;
    K.C = make_strip<VEC, T>(S, tile);
    const int64_t org = S.L.org + tile.x0;
    K.pc = gp(S.fld[n & 1] + org);
    K.pm = gp(S.fld[(n + 1) & 1] + org);
    K.wa = gp(S.fld[4 + ((n + T - 1) & 1)] + org);
    K.wb = gp(S.fld[4 + ((n + T) & 1)] + org);
    K.Dp = gp(S.Dp + org);
    const bool mid = T == 3 && nsample > 0;
    K.mid = mid ? gp(S.fld[2] + org) : nullptr;
    K.m0 = mid ? max(tile.z0, S.sz0) : 0;
    K.mn = mid ? (unsigned)max(min(tile.z1, S.sz1) - K.m0, 0) : 0u;

    float q1[9][VEC], q2[9][VEC], q3[9][VEC], qd[9][VEC];
    FwdIn<VEC> in[P > 0 ? P : 1];
    strip_fill<VEC>(K.C, K.pc, K.C.r0 - 4, q1);
    RowAt ra, rq;
    ra.start(K.C.r0, K.C.pitch4, K.C.NZr);
    rq.start(K.C.r0 + 4, K.C.pitch4, K.C.NZr);
#pragma unroll
    for (int i = 0; i < (P > 0 ? P : 1); ++i) {
        in[i].h = f4v{0.f, 0.f, 0.f, 0.f};
        if constexpr (P > 0) fwd_fetch<VEC, T, true>(K, ra, rq, in[i]);
        else if (K.C.ends) in[i].h = *(const gf4v *)at(at(K.pc, ra.off) - 4, here(K.C.hx));
    }
    SrcLane src{-(1 << 30), 0, 0, 0.f, 0.f};
    K.s0 = 0;
    K.sn = 0;
    if (tile.s1end > tile.s1beg) {
        src = src_load<T>(tile, ents, cont, S.wav + n, 1, lane, false);
        // the first step's list holds every node of the others; sorted by row
        K.s0 = __builtin_amdgcn_readlane(src.z, 0);
        K.sn = (unsigned)(__builtin_amdgcn_readlane(src.z, tile.s1end - tile.s1beg - 1) + 1 - K.s0);
    }
#pragma unroll
    for (int i = 0; i < 9; ++i)
#pragma unroll
        for (int j = 0; j < VEC; ++j) q2[i][j] = q3[i][j] = qd[i][j] = 0.f;
    int64_t o1 = (int64_t)K.C.r0 * (int64_t)K.C.pitch4;
    const int nstep = tile.z1 - tile.z0 + (T - 1) * kZUnroll;
#define RTM_ROW(PH, SS, ZZ) fwd_row<VEC, T, P, NT, PH, SS>(K, q1, q2, q3, qd, in, src, ra, rq, o1, K.C.r0 + (ZZ))
    RTM_NINE(RTM_ROW, 0, 0)
    if constexpr (T == 3) {
        RTM_NINE(RTM_ROW, 1, 9)
    }
    for (int s = 9 * (T - 1); s < nstep; s += 9) {
        RTM_NINE(RTM_ROW, 2, s)
    }
#undef RTM_ROW
}

template <int VEC, int T, int P, bool NT, bool GRAD>
__global__ __launch_bounds__(64) void rev2d_multi_kernel(const ShotDev *__restrict__ shots, const Tile2D *__restrict__ tiles,
                                                      int ntiles, int nslots, const InjEnt *__restrict__ ents,
                                                      const Contrib *__restrict__ cont, int k, int reinject,
                                                      float *__restrict__ wadj)
{
    const int t = xcd_tile(blockIdx.x, nslots);
    if (t >= ntiles) return;
    TileEntry &tile = *(TileEntry *)(uintptr_t)(tiles + t);
    ShotEntry &S = *(ShotEntry *)(uintptr_t)(shots + tile.shot);
    const int lane = threadIdx.x;
    __shared__ RecLds<VEC> rl[T];
    __shared__ float sv[64 * VEC];
    __shared__ int has[64 * VEC];
    RevMulti<VEC, T, GRAD> K;
    K.C = make_strip<VEC, T>(S, tile);
    const int64_t org = S.L.org + tile.x0;
    K.P0 = gp(S.fld[k & 1] + org);
    K.P1 = gp(S.fld[(k + 1) & 1] + org);
    K.M0 = gp(S.fld[2 + ((k + 1) & 1)] + org);
    K.M1 = gp(S.fld[2 + (k & 1)] + org);
    K.WPa = gp(S.fld[4 + ((k - T + 1) & 1)] + org);
    K.WPb = gp(S.fld[4 + ((k - T) & 1)] + org);
    K.WMa = gp(S.fld[6 + ((k - T + 2) & 1)] + org);
    K.WMb = gp(S.fld[6 + ((k - T + 1) & 1)] + org);
    K.Dp = gp(S.Dp + org);
    K.A0 = gp(S.acc0 + org);
    K.A1 = GRAD ? nullptr : gp(S.acc1 + org);
    K.wadj = wadj;
    K.ents = ents;
    K.cont = cont;
    K.sig = S.sig + (int64_t)k * S.nrec;
    K.nrec = S.nrec;
    K.rl = rl;
    K.sv = sv;
    K.has = has;
    K.k = k;
    K.alo = max(tile.z0, S.iz0);
    K.an = (unsigned)max(min(tile.z1, S.iz1) - K.alo, 0);
    K.alane = K.C.own && K.C.x + VEC > S.ix0 && K.C.x < S.ix1;
    K.reinject = reinject != 0;

    float q1p[9][VEC], q1m[9][VEC], q2p[9][VEC], q2m[9][VEC], q3p[9][VEC], q3m[9][VEC], qd[9][VEC], qg[9][VEC];
    float ia[VEC], ib[VEC];
    RevIn<VEC, GRAD> in[P > 0 ? P : 1];
    strip_fill<VEC>(K.C, K.P0, K.C.r0 - 4, q1p);
    strip_fill<VEC>(K.C, K.M0, K.C.r0 - 4, q1m);
    RowAt ra, rq;
    ra.start(K.C.r0, K.C.pitch4, K.C.NZr);
    rq.start(K.C.r0 + 4, K.C.pitch4, K.C.NZr);
#pragma unroll
    for (int i = 0; i < (P > 0 ? P : 1); ++i) {
        in[i].hp = in[i].hm = f4v{0.f, 0.f, 0.f, 0.f};
        if constexpr (P > 0) rev_fetch<VEC, T, GRAD, true>(K, ra, rq, in[i]);
        else rev_ends<VEC, T, GRAD>(K, ra, in[i]);
    }
    SrcLane src{-(1 << 30), 0, 0, 0.f, 0.f};
    K.s0 = 0;
    K.sn = 0;
    if (tile.s1end > tile.s1beg) {
        src = src_load<T>(tile, ents, cont, S.wav + k, -1, lane, GRAD && wadj);
        // the first step's list holds every node of the others; sorted by row
        K.s0 = __builtin_amdgcn_readlane(src.z, 0);
        K.sn = (unsigned)(__builtin_amdgcn_readlane(src.z, tile.s1end - tile.s1beg - 1) + 1 - K.s0);
    }
    RecList R[T];
#pragma unroll
    for (int s = 1; s <= T; ++s) {
        int beg, end;
        rec_range<T>(tile, s, beg, end);
        R[s - 1] = RecList{beg, end, 0, 1 << 30};
    }
    if (tile.r1end > tile.r1beg) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) has[lane * VEC + j] = 0;
#pragma unroll
        for (int s = 1; s <= T; ++s) {
            if (lane == 0) rl[s - 1].z[64 * VEC] = 1 << 30;
            rec_chunk<VEC>(rl[s - 1], R[s - 1], ents, cont, K.sig - (s - 1) * S.nrec, tile.x0, lane);
        }
    }
#pragma unroll
    for (int i = 0; i < 9; ++i)
#pragma unroll
        for (int j = 0; j < VEC; ++j) q2p[i][j] = q2m[i][j] = q3p[i][j] = q3m[i][j] = qd[i][j] = qg[i][j] = 0.f;
#pragma unroll
    for (int j = 0; j < VEC; ++j) ia[j] = ib[j] = 0.f;
    int64_t o1 = (int64_t)K.C.r0 * (int64_t)K.C.pitch4;
    const int nstep = tile.z1 - tile.z0 + (T - 1) * kZUnroll;
#define RTM_ROW(PH, SS, ZZ) \
    rev_row<VEC, T, P, NT, GRAD, PH, SS>(K, q1p, q1m, q2p, q2m, q3p, q3m, qd, qg, in, ia, ib, src, R, ra, rq, o1, K.C.r0 + (ZZ))
    RTM_NINE(RTM_ROW, 0, 0)
    if constexpr (T == 3) {
        RTM_NINE(RTM_ROW, 1, 9)
    }
    for (int s = 9 * (T - 1); s < nstep; s += 9) {
        RTM_NINE(RTM_ROW, 2, s)
    }
#undef RTM_ROW
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------

namespace {

// Tiles from which on the other wavefronts of a SIMD hide a row's loads: four
// per SIMD, what the ring's 126 registers leave room for.  Forward (us per
// step), 16 shots (3168 tiles): 52.7 with the ring, 55.3 without; 24 shots
// (4752): 83.0 and 80.9; 48 shots (9504): 152.8 and 149.9.
constexpr int kAheadTiles = 4 * 1024;

template <int V, int T, bool N>
void fwd_launch(const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots, const InjEnt *ents,
                const Contrib *cont, const SampleTask *stasks, int nsample, int n, hipStream_t st)
{
    const dim3 grid(nslots + T * nsample), block(64);
    if constexpr (V < 4)  // four floats per lane leave no registers for the ring
        if (ntiles < kAheadTiles) {
            hipLaunchKernelGGL((fwd2d_multi_kernel<V, T, 3, N>), grid, block, 0, st, shots, tiles, ntiles, nslots,
                               ents, cont, stasks, nsample, n);
            return;
        }
    hipLaunchKernelGGL((fwd2d_multi_kernel<V, T, 0, N>), grid, block, 0, st, shots, tiles, ntiles, nslots, ents, cont,
                       stasks, nsample, n);
}

// The reverse triple holds six field queues (167 registers at two floats per
// lane): the ring would cost it a wavefront per SIMD (4 shots: 39.5 us per
// step without, 44.7 with it).
template <int V, int T, bool N, bool G>
void rev_launch(const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots, const InjEnt *ents,
                const Contrib *cont, int k, int reinject, float *wadj, hipStream_t st)
{
    if constexpr (V < 4 && T == 2)
        if (ntiles < kAheadTiles) {
            hipLaunchKernelGGL((rev2d_multi_kernel<V, T, 3, N, G>), dim3(nslots), dim3(64), 0, st, shots, tiles, ntiles,
                               nslots, ents, cont, k, reinject, wadj);
            return;
        }
    hipLaunchKernelGGL((rev2d_multi_kernel<V, T, 0, N, G>), dim3(nslots), dim3(64), 0, st, shots, tiles, ntiles, nslots,
                       ents, cont, k, reinject, wadj);
}

}  // namespace

// `code`: floats per lane | block shape << 8 | kOnce (strips of up to two
// floats per lane).
#define RTM_VECS(CALL)                          \
    switch (code) {                             \
    case 1: CALL(1, false); break;              \
    case 2: CALL(2, false); break;              \
    case 4: CALL(4, false); break;              \
    case 1 | kOnce: CALL(1, true); break;       \
    case 2 | kOnce: CALL(2, true); break;       \
    default: return hipErrorInvalidValue;       \
    }                                           \
    return hipGetLastError();

hipError_t launch_fwd2d_t2(int code, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                           const InjEnt *ents, const Contrib *cont, const SampleTask *stasks, int nsample, int n,
                           hipStream_t st)
{
    if (const int shape = code >> 8 & 0xff)
        return launch_fwd2d_block(shape, 2, shots, tiles, ntiles, nslots, ents, cont, stasks, nsample, n, st);
#define RTM_CALL(V, N) fwd_launch<V, 2, N>(shots, tiles, ntiles, nslots, ents, cont, stasks, nsample, n, st)
    RTM_VECS(RTM_CALL)
#undef RTM_CALL
}

hipError_t launch_fwd2d_t3(int code, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                           const InjEnt *ents, const Contrib *cont, const SampleTask *stasks, int nsample, int n,
                           hipStream_t st)
{
    if (const int shape = code >> 8 & 0xff)
        return launch_fwd2d_block(shape, 3, shots, tiles, ntiles, nslots, ents, cont, stasks, nsample, n, st);
#define RTM_CALL(V, N) fwd_launch<V, 3, N>(shots, tiles, ntiles, nslots, ents, cont, stasks, nsample, n, st)
    RTM_VECS(RTM_CALL)
#undef RTM_CALL
}

hipError_t launch_rev2d_t2(int code, bool grad, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                           const InjEnt *ents, const Contrib *cont, int k, int reinject, float *wadj, hipStream_t st)
{
    if (const int shape = code >> 8 & 0xff)
        return launch_rev2d_block(shape, 2, grad, shots, tiles, ntiles, nslots, ents, cont, k, reinject, wadj, st);
#define RTM_CALL(V, N)                                                                                          \
    if (grad)                                                                                                \
        rev_launch<V, 2, N, true>(shots, tiles, ntiles, nslots, ents, cont, k, reinject, wadj, st);              \
    else                                                                                                     \
        rev_launch<V, 2, N, false>(shots, tiles, ntiles, nslots, ents, cont, k, reinject, wadj, st)
    RTM_VECS(RTM_CALL)
#undef RTM_CALL
}

hipError_t launch_rev2d_t3(int code, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                           const InjEnt *ents, const Contrib *cont, int k, int reinject, hipStream_t st)
{
    if (const int shape = code >> 8 & 0xff)
        return launch_rev2d_block(shape, 3, false, shots, tiles, ntiles, nslots, ents, cont, k, reinject, nullptr, st);
#define RTM_CALL(V, N) rev_launch<V, 3, N, false>(shots, tiles, ntiles, nslots, ents, cont, k, reinject, nullptr, st)
    RTM_VECS(RTM_CALL)
#undef RTM_CALL
}

hipError_t launch_rev2d_t3_grad(int code, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                                const InjEnt *ents, const Contrib *cont, int k, int reinject, float *wadj,
                                hipStream_t st)
{
    if (const int shape = code >> 8 & 0xff)
        return launch_rev2d_block(shape, 3, true, shots, tiles, ntiles, nslots, ents, cont, k, reinject, wadj, st);
#define RTM_CALL(V, N) rev_launch<V, 3, N, true>(shots, tiles, ntiles, nslots, ents, cont, k, reinject, wadj, st)
    RTM_VECS(RTM_CALL)
#undef RTM_CALL
}

}  // namespace rtm
