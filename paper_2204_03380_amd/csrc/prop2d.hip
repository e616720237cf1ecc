// 2-D propagation kernels for gfx950.
//
// One wavefront (64 lanes) owns a strip of 64 * VEC consecutive x cells and
// marches down the rows [z0, z1) of its tile.  Each lane keeps the nine rows
// z-4 .. z+4 of its VEC cells in registers (a register queue), so every
// stored value of the input field is read from memory once per tile plus the
// 8-row overlap with the tiles above and below.  The march is unrolled by
// nine so that the queue rotates by register renaming, not by moves.  The
// x-neighbours of the centre row come from the adjacent lanes through DPP
// wave shifts; lanes 0 and 63 supply the 4-cell halo at the strip ends with
// one extra load.
//
// The stencil is evaluated as
//   L p_i = sum_axis sum_{m=1..4} c_m ((p_{i+m} + p_{i-m}) - 2 p_i),
// algebraically the 8th-order Laplacian of Sec. 3, but exactly zero on a
// constant field in FP32: the rounded weights then cannot add a spurious
// mass term, which would otherwise accumulate into a phase error of ~1e-3
// after a few thousand steps.
//
// Fields are stored with a zero halo and the scaled velocity term
// D' = (v dt / h)^2 is zero there, so updating a halo cell reproduces zero;
// lanes past the grid edge only have to skip their loads and stores.
#include <atomic>

#include "stencil.h"

namespace rtm {
namespace {

// --------------------------------------------------------------------------
// Forward step
// --------------------------------------------------------------------------

template <int VEC>
struct FwdCtx {
    const gfloat *pc;  // p^n
    gfloat *po;        // p^{n-1}, overwritten by p^{n+1}
    const gfloat *Dp;
    int64_t pitch;
    int x, x0, NX, lane, w;  // x0: first cell of this wave's strip; w: wave in the workgroup
    bool live, own;
};

// Row z of the march.  Queue slot (S + i) % 9 holds row z - 4 + i; the slot
// of row z + 4 is refilled here.  With TX strips per workgroup the inner
// strip ends come from the edge ring (slot S holds row z); the workgroup
// meets at a barrier every third row, which orders each ring write (row
// z + 4, end of this step) before its read four steps later and each read
// before the slot is rewritten five steps later.
// The one-step forward row (forward and receiver-only kernels) with one
// strip per workgroup fetches each row's strip-end halo one march step early
// (hc: the halo of row z, fetched at row z - 1), as the two-step kernels do:
// 326 -> 339 us without it for 48 shots at vec 1.  The one-step reverse
// kernel keeps the in-step load (no consistent gain: 854 -> 874 us at vec 1,
// 868 -> 849 at vec 4).
template <int VEC, int TX>
constexpr bool ahead1() { return TX == 1 && VEC != 2; }

// Strip-end halo of row z into hl / hr: the early-fetched one (then fetch
// row z + 1's, always a stored row as z < NZr) or a load now.
template <int VEC, int TX, bool AHEAD>
__device__ __forceinline__ void row_halo(const gfloat *f, int64_t pitch, int z, int x0, int NX, int lane, int w,
                                         f4v &hc, float (&hl)[4], float (&hr)[4])
{
    if constexpr (AHEAD) {
        const f4v t = hc;
        hc = halo_fetch<VEC>(f + (int64_t)(z + 1) * pitch, x0, NX, lane, true);
        halo_split(t, lane, hl, hr);
    } else {
        load_halo_outer<VEC>(f + (int64_t)z * pitch, x0, NX, lane, w == 0, w == TX - 1, hl, hr);
    }
}

template <int VEC, int TX, int S>
__device__ __forceinline__ void fwd_row(const FwdCtx<VEC> &C, float (&q)[9][VEC], int z, EdgeRing<TX> &R, f4v &hc)
{
    constexpr int r0 = (S + 0) % 9, r1 = (S + 1) % 9, r2 = (S + 2) % 9, r3 = (S + 3) % 9, r4 = (S + 4) % 9,
                  r5 = (S + 5) % 9, r6 = (S + 6) % 9, r7 = (S + 7) % 9, r8 = (S + 8) % 9;
    if constexpr (TX > 1 && S % 3 == 0) __syncthreads();
    const int64_t o = (int64_t)z * C.pitch + C.x;
    float old[VEC], d[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) q[r8][j] = old[j] = d[j] = 0.f;
    if (C.live) {
        ldv<VEC>(C.pc + o + 4 * C.pitch, q[r8]);
        ldv<VEC>(C.po + o, old);
        ldv<VEC>(C.Dp + o, d);
    }
    float hl[4], hr[4], ext[VEC + 8];
    row_halo<VEC, TX, ahead1<VEC, TX>()>(C.pc, C.pitch, z, C.x0, C.NX, C.lane, C.w, hc, hl, hr);
    ring_get<TX>(R, S, C.w, C.lane, hl, hr);
    exchange_row<VEC>(q[r4], hl, hr, ext);
    float out[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        const float c = q[r4][j], c2 = c + c;
        float lap = d2(c2, ext[3 + j], ext[5 + j], ext[2 + j], ext[6 + j], ext[1 + j], ext[7 + j], ext[j], ext[8 + j]);
        lap += d2(c2, q[r3][j], q[r5][j], q[r2][j], q[r6][j], q[r1][j], q[r7][j], q[r0][j], q[r8][j]);
        out[j] = fmaf(d[j], lap, c2 - old[j]);
    }
    if (C.own) stv<VEC>(C.po + o, out);
    if constexpr (TX > 1) ring_put<VEC, TX>(R, (S + 4) % 9, C.w, C.lane, q[r8]);
}

// --------------------------------------------------------------------------
// Reverse step
// --------------------------------------------------------------------------

template <int VEC>
struct RevCtx {
    const gfloat *P0;  // p^k
    gfloat *P1;        // p^{k+1} -> p^{k-1}
    const gfloat *M0;  // mu^{k+1}
    gfloat *M1;        // mu^{k+2} -> mu^k
    const gfloat *Dp;
    gfloat *A0, *A1;   // num, den | G
    int64_t pitch;
    int x, x0, NX, lane, w, iz0, iz1;
    bool live, own, own_img, reinject;
};

template <int VEC, bool GRAD, int TX, int S>
__device__ __forceinline__ void rev_row(const RevCtx<VEC> &C, float (&qp)[9][VEC], float (&qm)[9][VEC], int z,
                                        EdgeRing<TX> &RP, EdgeRing<TX> &RM, f4v &hp, f4v &hm)
{
    constexpr int r0 = (S + 0) % 9, r1 = (S + 1) % 9, r2 = (S + 2) % 9, r3 = (S + 3) % 9, r4 = (S + 4) % 9,
                  r5 = (S + 5) % 9, r6 = (S + 6) % 9, r7 = (S + 7) % 9, r8 = (S + 8) % 9;
    if constexpr (TX > 1 && S % 3 == 0) __syncthreads();
    const int64_t o = (int64_t)z * C.pitch + C.x;
    float p1[VEC], m1[VEC], d[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) qp[r8][j] = qm[r8][j] = p1[j] = m1[j] = d[j] = 0.f;
    if (C.live) {
        ldv<VEC>(C.P0 + o + 4 * C.pitch, qp[r8]);
        ldv<VEC>(C.M0 + o + 4 * C.pitch, qm[r8]);
        ldv_s<VEC>(C.P1 + o, p1);
        ldv_s<VEC>(C.M1 + o, m1);
        ldv_s<VEC>(C.Dp + o, d);
    }
    float hl[4], hr[4], ext[VEC + 8];
    float np[VEC], nm[VEC], inc[VEC];
    row_halo<VEC, TX, false>(C.P0, C.pitch, z, C.x0, C.NX, C.lane, C.w, hp, hl, hr);
    ring_get<TX>(RP, S, C.w, C.lane, hl, hr);
    exchange_row<VEC>(qp[r4], hl, hr, ext);
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        const float c = qp[r4][j], c2 = c + c;
        float lap = d2(c2, ext[3 + j], ext[5 + j], ext[2 + j], ext[6 + j], ext[1 + j], ext[7 + j], ext[j], ext[8 + j]);
        lap += d2(c2, qp[r3][j], qp[r5][j], qp[r2][j], qp[r6][j], qp[r1][j], qp[r7][j], qp[r0][j], qp[r8][j]);
        inc[j] = d[j] * lap;                 // gradient term (GRAD)
        np[j] = fmaf(d[j], lap, c2 - p1[j]);  // same rounding as the two-step kernel
    }
    if (C.own) stv<VEC>(C.P1 + o, np);
    row_halo<VEC, TX, false>(C.M0, C.pitch, z, C.x0, C.NX, C.lane, C.w, hm, hl, hr);
    ring_get<TX>(RM, S, C.w, C.lane, hl, hr);
    exchange_row<VEC>(qm[r4], hl, hr, ext);
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        const float c = qm[r4][j], c2 = c + c;
        float lap = d2(c2, ext[3 + j], ext[5 + j], ext[2 + j], ext[6 + j], ext[1 + j], ext[7 + j], ext[j], ext[8 + j]);
        lap += d2(c2, qm[r3][j], qm[r5][j], qm[r2][j], qm[r6][j], qm[r1][j], qm[r7][j], qm[r0][j], qm[r8][j]);
        nm[j] = fmaf(d[j], lap, c2 - m1[j]);
    }
    if (C.own) stv<VEC>(C.M1 + o, nm);
    if constexpr (GRAD) {
        if (C.own) {
            float g[VEC];
            ldv<VEC>(C.A0 + o, g);
#pragma unroll
            for (int j = 0; j < VEC; ++j) g[j] = fmaf(qm[r4][j], inc[j], g[j]);
            stv<VEC>(C.A0 + o, g);
        }
    } else {
        if (z >= C.iz0 && z < C.iz1 && C.own_img) {
            float a[VEC], b[VEC];
            ldv_s<VEC>(C.A0 + o, a);
            ldv_s<VEC>(C.A1 + o, b);
#pragma unroll
            for (int j = 0; j < VEC; ++j) {
                a[j] = fmaf(qp[r4][j], qm[r4][j], a[j]);
                b[j] = fmaf(qp[r4][j], qp[r4][j], b[j]);
            }
            stv_s<VEC>(C.A0 + o, a);
            stv_s<VEC>(C.A1 + o, b);
        }
    }
    if constexpr (TX > 1) {
        ring_put<VEC, TX>(RP, (S + 4) % 9, C.w, C.lane, qp[r8]);
        ring_put<VEC, TX>(RM, (S + 4) % 9, C.w, C.lane, qm[r8]);
    }
}

// Runs ROWCALL(S, z) over the tile's rows, nine per trip (z1 - z0 is a
// multiple of nine), so that S = (z - z0) mod 9 is a compile-time constant.
#define RTM_MARCH(ROWCALL)                                                                     \
    for (int z = T.z0; z < T.z1; z += kZUnroll) {                                              \
        ROWCALL(0, z); ROWCALL(1, z + 1); ROWCALL(2, z + 2); ROWCALL(3, z + 3);                \
        ROWCALL(4, z + 4); ROWCALL(5, z + 5); ROWCALL(6, z + 6); ROWCALL(7, z + 7);            \
        ROWCALL(8, z + 8);                                                                     \
    }

}  // namespace

// Forward step n of every tile:  p^{n+1} = 2 p^n - p^{n-1} + D' (L p^n + s^n),
// written over p^{n-1}; workgroups past the stencil slots record d^n = R p^n.
// The source term is added to the stored value after the march by the lane
// that stored it (same thread, so program order makes the value visible).
// A workgroup of TX wavefronts covers TX adjacent strips of one tile.
template <int VEC, int TX>
__device__ __forceinline__ void fwd2d_tile(const ShotDev *__restrict__ shots, const Tile2D *__restrict__ tiles, int t,
                                           const InjEnt *__restrict__ ents, const Contrib *__restrict__ cont, int n,
                                           int w, int lane, EdgeRing<TX> &ring)
{
    const Tile2D T = tiles[t];
    const ShotDev &S = shots[T.shot];
    FwdCtx<VEC> C;
    C.pitch = S.L.pitch;
    C.NX = S.L.NX;
    C.pc = gp(S.fld[n & 1] + S.L.org);
    C.po = gp(S.fld[(n + 1) & 1] + S.L.org);
    C.Dp = gp(S.Dp + S.L.org);
    C.lane = lane;
    C.w = w;
    C.x0 = T.x0 + w * 64 * VEC;
    C.x = C.x0 + lane * VEC;
    C.live = C.x < C.NX + kRadius;
    C.own = C.x < C.NX;

    float q[9][VEC];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) q[i][j] = 0.f;
        if (C.live) ldv<VEC>(C.pc + (int64_t)(T.z0 - 4 + i) * C.pitch + C.x, q[i]);
        // rows z0 .. z0 + 3 (queue slots 4..7, ring slots 0..3); the first
        // march step opens with a barrier
        if constexpr (TX > 1)
            if (i >= 4) ring_put<VEC, TX>(ring, i - 4, w, lane, q[i]);
    }
    f4v hc = halo_fetch<VEC>(C.pc + (int64_t)T.z0 * C.pitch, C.x0, C.NX, lane, ahead1<VEC, TX>());
#define RTM_FWD_ROW(SS, ZZ) fwd_row<VEC, TX, SS>(C, q, ZZ, ring, hc)
    RTM_MARCH(RTM_FWD_ROW)
#undef RTM_FWD_ROW
    // Source injection: p^{n+1} += D' s^n at the source nodes of this tile.
    const float *wav = S.wav + n;
    for (int e = T.sbeg; e < T.send; ++e) {
        const InjEnt E = ents[e];
        if (owns<VEC>(E.x, C.x0, C.lane)) {
            const int64_t o = (int64_t)E.z * C.pitch + E.x;
            C.po[o] = fmaf(C.Dp[o], inj_sum(E, cont, wav), C.po[o]);
        }
    }
}

template <int VEC, int TX>
__global__ __launch_bounds__(64 * TX) void fwd2d_kernel(const ShotDev *__restrict__ shots,
                                                        const Tile2D *__restrict__ tiles, int ntiles, int nslots,
                                                        const InjEnt *__restrict__ ents,
                                                        const Contrib *__restrict__ cont,
                                                        const SampleTask *__restrict__ stasks, int nsample, int n)
{
    const int b = blockIdx.x;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (b >= nslots) {
        const int task = (b - nslots) * TX + w;
        if (task < nsample) sample_body(shots, stasks[task], n, n & 1, lane);
        return;
    }
    const int t = xcd_tile(b, nslots);
    if (t >= ntiles) return;  // whole workgroup
    __shared__ EdgeRing<TX> ring;
    fwd2d_tile<VEC, TX>(shots, tiles, t, ents, cont, n, w, lane, ring);
}

// Reverse step k of every tile, Eqs. (2), (3) and (6) in one pass:
//   p^{k-1} = 2 p^k - p^{k+1} + D' (L p^k + s^k)         (reconstruction)
//   mu^k    = 2 mu^{k+1} - mu^{k+2} + D' (L mu^{k+1} + r^k)  (receiver field)
// and either the imaging sums num += p^k mu^{k+1}, den += (p^k)^2 on the
// interior (GRAD = false) or the gradient sum G += mu^{k+1} D' (L p^k + s^k)
// on the whole padded grid (GRAD = true).  With reinject = 0 the source term
// is left out of the reconstruction (Eq. (6) as written).  The source and
// receiver terms are added after the march by the lanes that stored the
// cells.  When wadj is non-null, those lanes also write each source node's
// coefficient times mu^{k+1} to wadj[k * kMaxNodes + node].
// With one float per lane the reverse kernel fits in 64 registers; asking
// for 8 waves per SIMD then hides more latency (measured: 4.5 vs 4.2 TB/s
// on 16 shots of the 2301 x 751 grid).  Wider lanes would spill.
// rev2d_kernel's tile body as a function, for the persistent pass.  The
// kernel keeps its own copy of the body: compiled through this function,
// its one-float-per-lane instance (held to 64 registers for 8 waves per
// SIMD) spills 156 bytes per lane, while the copy fits.
template <int VEC, bool GRAD, int TX>
__device__ __forceinline__ void rev2d_tile(const ShotDev *__restrict__ shots, const Tile2D *__restrict__ tiles, int t,
                                           const InjEnt *__restrict__ ents, const Contrib *__restrict__ cont, int k,
                                           int reinject, float *__restrict__ wadj, int w, int lane,
                                           EdgeRing<TX> &ring_p, EdgeRing<TX> &ring_m)
{
    const Tile2D T = tiles[t];
    const ShotDev &S = shots[T.shot];
    RevCtx<VEC> C;
    C.pitch = S.L.pitch;
    C.NX = S.L.NX;
    C.P0 = gp(S.fld[k & 1] + S.L.org);
    C.P1 = gp(S.fld[(k + 1) & 1] + S.L.org);
    C.M0 = gp(S.fld[2 + ((k + 1) & 1)] + S.L.org);
    C.M1 = gp(S.fld[2 + (k & 1)] + S.L.org);
    C.Dp = gp(S.Dp + S.L.org);
    C.A0 = gp(S.acc0 + S.L.org);
    C.A1 = GRAD ? nullptr : gp(S.acc1 + S.L.org);
    C.lane = lane;
    C.w = w;
    C.x0 = T.x0 + w * 64 * VEC;
    C.x = C.x0 + lane * VEC;
    C.live = C.x < C.NX + kRadius;
    C.own = C.x < C.NX;
    // Lanes whose cells overlap the interior accumulate the image sums (their
    // other cells lie in the band or halo, whose sums are never read).
    C.own_img = C.own && C.x + VEC > S.ix0 && C.x < S.ix1;
    C.iz0 = S.iz0;
    C.iz1 = S.iz1;
    C.reinject = reinject != 0;

    float qp[9][VEC], qm[9][VEC];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) qp[i][j] = qm[i][j] = 0.f;
        if (C.live) {
            ldv<VEC>(C.P0 + (int64_t)(T.z0 - 4 + i) * C.pitch + C.x, qp[i]);
            ldv<VEC>(C.M0 + (int64_t)(T.z0 - 4 + i) * C.pitch + C.x, qm[i]);
        }
        if constexpr (TX > 1)
            if (i >= 4) {
                ring_put<VEC, TX>(ring_p, i - 4, w, lane, qp[i]);
                ring_put<VEC, TX>(ring_m, i - 4, w, lane, qm[i]);
            }
    }
    f4v hp = f4v{0.f, 0.f, 0.f, 0.f}, hm = hp;  // (the reverse rows load their halo in-step)
#define RTM_REV_ROW(SS, ZZ) rev_row<VEC, GRAD, TX, SS>(C, qp, qm, ZZ, ring_p, ring_m, hp, hm)
    RTM_MARCH(RTM_REV_ROW)
#undef RTM_REV_ROW
    // Source term at step k: reconstruction (re-injection), gradient, wavelet adjoint.
    const float *wav = S.wav + k;
    for (int e = T.sbeg; e < T.send; ++e) {
        const InjEnt E = ents[e];
        if (owns<VEC>(E.x, C.x0, C.lane)) {
            const int64_t o = (int64_t)E.z * C.pitch + E.x;
            const float sv = inj_sum(E, cont, wav);
            if (C.reinject) C.P1[o] = fmaf(C.Dp[o], sv, C.P1[o]);
            if (GRAD) C.A0[o] = fmaf(C.M0[o], C.Dp[o] * sv, C.A0[o]);
            if (wadj) {
                float wsum = 0.f;
                for (int c = E.cbeg; c < E.cend; ++c) wsum += cont[c].w;
                wadj[(int64_t)k * kMaxNodes + E.slot] = wsum * C.M0[o];
            }
        }
    }
    // Receiver term: mu^k += D' R^T g^k.
    inject_nodes(C.M1, C.Dp, ents, T.rbeg, T.rend, cont, S.sig + (int64_t)k * S.nrec, C.pitch, C.pitch);
}

template <int VEC, bool GRAD, int TX>
__global__ __launch_bounds__(64 * TX) __attribute__((amdgpu_waves_per_eu(VEC == 1 ? 8 : 1, 8)))
void rev2d_kernel(const ShotDev *__restrict__ shots, const Tile2D *__restrict__ tiles, int ntiles, int nslots,
                  const InjEnt *__restrict__ ents, const Contrib *__restrict__ cont, int k, int reinject,
                  float *__restrict__ wadj)
{
    const int t = xcd_tile(blockIdx.x, nslots);
    if (t >= ntiles) return;  // whole workgroup
    const Tile2D T = tiles[t];
    const ShotDev &S = shots[T.shot];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __shared__ EdgeRing<TX> ring_p, ring_m;
    RevCtx<VEC> C;
    C.pitch = S.L.pitch;
    C.NX = S.L.NX;
    C.P0 = gp(S.fld[k & 1] + S.L.org);
    C.P1 = gp(S.fld[(k + 1) & 1] + S.L.org);
    C.M0 = gp(S.fld[2 + ((k + 1) & 1)] + S.L.org);
    C.M1 = gp(S.fld[2 + (k & 1)] + S.L.org);
    C.Dp = gp(S.Dp + S.L.org);
    C.A0 = gp(S.acc0 + S.L.org);
    C.A1 = GRAD ? nullptr : gp(S.acc1 + S.L.org);
    C.lane = lane;
    C.w = w;
    C.x0 = T.x0 + w * 64 * VEC;
    C.x = C.x0 + lane * VEC;
    C.live = C.x < C.NX + kRadius;
    C.own = C.x < C.NX;
    // Lanes whose cells overlap the interior accumulate the image sums (their
    // other cells lie in the band or halo, whose sums are never read).
    C.own_img = C.own && C.x + VEC > S.ix0 && C.x < S.ix1;
    C.iz0 = S.iz0;
    C.iz1 = S.iz1;
    C.reinject = reinject != 0;

    float qp[9][VEC], qm[9][VEC];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) qp[i][j] = qm[i][j] = 0.f;
        if (C.live) {
            ldv<VEC>(C.P0 + (int64_t)(T.z0 - 4 + i) * C.pitch + C.x, qp[i]);
            ldv<VEC>(C.M0 + (int64_t)(T.z0 - 4 + i) * C.pitch + C.x, qm[i]);
        }
        if constexpr (TX > 1)
            if (i >= 4) {
                ring_put<VEC, TX>(ring_p, i - 4, w, lane, qp[i]);
                ring_put<VEC, TX>(ring_m, i - 4, w, lane, qm[i]);
            }
    }
    f4v hp = f4v{0.f, 0.f, 0.f, 0.f}, hm = hp;  // (the reverse rows load their halo in-step)
#define RTM_REV_ROW(SS, ZZ) rev_row<VEC, GRAD, TX, SS>(C, qp, qm, ZZ, ring_p, ring_m, hp, hm)
    RTM_MARCH(RTM_REV_ROW)
#undef RTM_REV_ROW
    // Source term at step k: reconstruction (re-injection), gradient, wavelet adjoint.
    const float *wav = S.wav + k;
    for (int e = T.sbeg; e < T.send; ++e) {
        const InjEnt E = ents[e];
        if (owns<VEC>(E.x, C.x0, C.lane)) {
            const int64_t o = (int64_t)E.z * C.pitch + E.x;
            const float sv = inj_sum(E, cont, wav);
            if (C.reinject) C.P1[o] = fmaf(C.Dp[o], sv, C.P1[o]);
            if (GRAD) C.A0[o] = fmaf(C.M0[o], C.Dp[o] * sv, C.A0[o]);
            if (wadj) {
                float wsum = 0.f;
                for (int c = E.cbeg; c < E.cend; ++c) wsum += cont[c].w;
                wadj[(int64_t)k * kMaxNodes + E.slot] = wsum * C.M0[o];
            }
        }
    }
    // Receiver term: mu^k += D' R^T g^k.
    inject_nodes(C.M1, C.Dp, ents, T.rbeg, T.rend, cont, S.sig + (int64_t)k * S.nrec, C.pitch, C.pitch);
}

// Receiver wavefield alone, for migration with a stored source wavefield
// (Algorithm 2): mu^k = 2 mu^{k+1} - mu^{k+2} + D' (L mu^{k+1} + r^k), the
// forward row update applied to mu (same operations as the mu half of the
// fused reverse kernel), with the receiver term added after the march.  At
// a stored level (snap non-null: the dense interior p^k) the imaging sums
// num += p^k mu^{k+1}, den += (p^k)^2 take mu^{k+1} from the register queue.
// IMG selects the imaging variant at compile time, so that the other steps
// run the plain forward code.
template <int VEC, int TX, bool IMG>
__global__ __launch_bounds__(64 * TX) void recv2d_kernel(const ShotDev *__restrict__ shots,
                                                         const Tile2D *__restrict__ tiles, int ntiles, int nslots,
                                                         const InjEnt *__restrict__ ents,
                                                         const Contrib *__restrict__ cont, int k,
                                                         const float *__restrict__ snap)
{
    const int t = xcd_tile(blockIdx.x, nslots);
    if (t >= ntiles) return;  // whole workgroup
    const Tile2D T = tiles[t];
    const ShotDev &S = shots[T.shot];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __shared__ EdgeRing<TX> ring;
    FwdCtx<VEC> C;
    C.pitch = S.L.pitch;
    C.NX = S.L.NX;
    C.pc = gp(S.fld[2 + ((k + 1) & 1)] + S.L.org);  // mu^{k+1}
    C.po = gp(S.fld[2 + (k & 1)] + S.L.org);        // mu^{k+2} -> mu^k
    C.Dp = gp(S.Dp + S.L.org);
    C.lane = lane;
    C.w = w;
    C.x0 = T.x0 + w * 64 * VEC;
    C.x = C.x0 + lane * VEC;
    C.live = C.x < C.NX + kRadius;
    C.own = C.x < C.NX;
    const bool img = IMG && C.own && C.x + VEC > S.ix0 && C.x < S.ix1;
    const SnapImg I{snap, S.ix1 - S.ix0, 1, S.ix0, S.ix1, 0, S.iz0};
    gfloat *A0 = gp(S.acc0 + S.L.org), *A1 = gp(S.acc1 + S.L.org);

    float q[9][VEC];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
        for (int j = 0; j < VEC; ++j) q[i][j] = 0.f;
        if (C.live) ldv<VEC>(C.pc + (int64_t)(T.z0 - 4 + i) * C.pitch + C.x, q[i]);
        if constexpr (TX > 1)
            if (i >= 4) ring_put<VEC, TX>(ring, i - 4, w, lane, q[i]);
    }
    f4v hc = halo_fetch<VEC>(C.pc + (int64_t)T.z0 * C.pitch, C.x0, C.NX, lane, ahead1<VEC, TX>());
#define RTM_RECV_ROW(SS, ZZ)                                                                        \
    fwd_row<VEC, TX, SS>(C, q, ZZ, ring, hc);                                                      \
    if constexpr (IMG)                                                                             \
        if (img && (ZZ) >= S.iz0 && (ZZ) < S.iz1)                                                  \
            snap_image<VEC>(I, A0, A1, (int64_t)(ZZ) * C.pitch + C.x, ZZ, 0, C.x, q[((SS) + 4) % 9]);
    RTM_MARCH(RTM_RECV_ROW)
#undef RTM_RECV_ROW
    // Receiver term: mu^k += D' R^T g^k.
    inject_nodes(C.po, C.Dp, ents, T.rbeg, T.rend, cont, S.sig + (int64_t)k * S.nrec, C.pitch, C.pitch);
}

// ---------------------------------------------------------------------------
// Persistent passes: one launch for all time steps of a pass
// ---------------------------------------------------------------------------
//
// A grid small enough to be resident as a whole (sized from the occupancy
// of the kernel) walks the pass's work items (tiles, and in modeling the
// receiver sampling tasks) step after step: workgroup b takes items b,
// b + G, b + 2G, ... of every step.  The steps of different shots are not
// tied to each other: an item of shot s at step r waits only until the
// counter of shot s shows all of that shot's items of step r - 1 done
// (r * items(s) completions), so a shot with little work runs ahead of a
// larger one.  One wave per workgroup: after an item the wave makes its
// stores visible to the whole GPU (agent-scope release fence, which also
// writes them back from this XCD's L2) and lane 0 increments the counter;
// a waiting wave's lane 0 reads the counter, and once it suffices the wave
// takes an agent-scope acquire fence (dropping stale L1/L2 lines) before
// touching the fields.  Every wait is bounded: after `limit` ticks of the
// constant 100 MHz clock, or as soon as another workgroup has given up, the
// waiting workgroup sets *status and returns, so a grid that cannot make
// progress (not all workgroups resident) still ends.

// Waits until *cnt >= target (lane 0 polls); false if the pass was abandoned.
__device__ __forceinline__ bool persist_wait(unsigned *cnt, unsigned target, unsigned *status, uint64_t limit,
                                             int lane)
{
    int ok = 1;
    if (lane == 0) {
        const uint64_t t0 = wall_clock64();
        while (__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            if (__hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u ||
                wall_clock64() - t0 > limit) {
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        if (!ok) __hip_atomic_store(status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    ok = __builtin_amdgcn_readfirstlane(ok);
    if (ok) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return ok != 0;
}

// Publishes the item just done: this wave's stores, then the count.
__device__ __forceinline__ void persist_done(unsigned *cnt, int lane)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if (lane == 0) __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Forward steps n0 .. n0 + nsteps - 1 (fwd2d_kernel's step, one strip per
// workgroup), with the sampling tasks of each step when stasks != nullptr.
template <int VEC>
__global__ __launch_bounds__(64) void fwd2d_persist_kernel(const ShotDev *__restrict__ shots,
                                                           const Tile2D *__restrict__ tiles,
                                                           const PItem *__restrict__ items, int nitems,
                                                           const int *__restrict__ shot_items,
                                                           const InjEnt *__restrict__ ents,
                                                           const Contrib *__restrict__ cont,
                                                           const SampleTask *__restrict__ stasks, int n0, int nsteps,
                                                           unsigned *cnt, unsigned *status, uint64_t limit)
{
    const int lane = threadIdx.x & 63;
    __shared__ EdgeRing<1> ring;
    for (int r = 0; r < nsteps; ++r) {
        const int n = n0 + r;
        for (int i = blockIdx.x; i < nitems; i += gridDim.x) {
            const PItem it = items[i];
            if (!persist_wait(cnt + it.shot, (unsigned)r * (unsigned)shot_items[it.shot], status, limit, lane)) return;
            if (it.idx >= 0) {
                fwd2d_tile<VEC, 1>(shots, tiles, it.idx, ents, cont, n, 0, lane, ring);
            } else {
                sample_body(shots, stasks[-1 - it.idx], n, n & 1, lane);
            }
            persist_done(cnt + it.shot, lane);
        }
    }
}

// Reverse steps k0, k0 - 1, ..., k0 - nsteps + 1 (rev2d_kernel's step).
template <int VEC, bool GRAD>
__global__ __launch_bounds__(64) void rev2d_persist_kernel(const ShotDev *__restrict__ shots, const Tile2D *__restrict__ tiles,
                          const PItem *__restrict__ items, int nitems, const int *__restrict__ shot_items,
                          const InjEnt *__restrict__ ents, const Contrib *__restrict__ cont, int k0, int nsteps,
                          int reinject, float *__restrict__ wadj, unsigned *cnt, unsigned *status, uint64_t limit)
{
    const int lane = threadIdx.x & 63;
    __shared__ EdgeRing<1> ring_p, ring_m;
    for (int r = 0; r < nsteps; ++r) {
        const int k = k0 - r;
        for (int i = blockIdx.x; i < nitems; i += gridDim.x) {
            const PItem it = items[i];
            if (!persist_wait(cnt + it.shot, (unsigned)r * (unsigned)shot_items[it.shot], status, limit, lane)) return;
            rev2d_tile<VEC, GRAD, 1>(shots, tiles, it.idx, ents, cont, k, reinject, wadj, 0, lane, ring_p, ring_m);
            persist_done(cnt + it.shot, lane);
        }
    }
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------

// Workgroups of a persistent launch: at most what the GPU holds resident at
// once (occupancy of the kernel times the compute units), at most nitems;
// and the bounded wait in ticks of the constant clock.
template <class K>
hipError_t persist_grid(K kernel, int nitems, double wait_ms, int *grid, uint64_t *limit)
{
    int dev = 0, cus = 0, per_cu = 0, khz = 0;
    hipError_t e;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev)) != hipSuccess) return e;
    if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 64, 0)) != hipSuccess) return e;
    if (per_cu < 1 || cus < 1) return hipErrorInvalidConfiguration;
    const int64_t g = std::min<int64_t>((int64_t)per_cu * cus, nitems);
    *grid = (int)std::max<int64_t>(g, 1);
    *limit = (uint64_t)((double)(khz > 0 ? khz : 100000) * wait_ms);
    return hipSuccess;
}

template <int V>
hipError_t fwd2d_persist_launch(const ShotDev *shots, const Tile2D *tiles, const PItem *items, int nitems,
                                const int *shot_items, const InjEnt *ents, const Contrib *cont,
                                const SampleTask *stasks, int n0, int nsteps, unsigned *cnt, unsigned *status,
                                double wait_ms, hipStream_t st)
{
    int grid = 0;
    uint64_t limit = 0;
    hipError_t e = persist_grid(fwd2d_persist_kernel<V>, nitems, wait_ms, &grid, &limit);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((fwd2d_persist_kernel<V>), dim3(grid), dim3(64), 0, st, shots, tiles, items, nitems,
                       shot_items, ents, cont, stasks, n0, nsteps, cnt, status, limit);
    return hipGetLastError();
}

template <int V, bool G>
hipError_t rev2d_persist_launch(const ShotDev *shots, const Tile2D *tiles, const PItem *items, int nitems,
                                const int *shot_items, const InjEnt *ents, const Contrib *cont, int k0, int nsteps,
                                int reinject, float *wadj, unsigned *cnt, unsigned *status, double wait_ms,
                                hipStream_t st)
{
    int grid = 0;
    uint64_t limit = 0;
    hipError_t e = persist_grid(rev2d_persist_kernel<V, G>, nitems, wait_ms, &grid, &limit);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((rev2d_persist_kernel<V, G>), dim3(grid), dim3(64), 0, st, shots, tiles, items, nitems,
                       shot_items, ents, cont, k0, nsteps, reinject, wadj, cnt, status, limit);
    return hipGetLastError();
}

hipError_t launch_fwd2d_persist(int vec, const ShotDev *shots, const Tile2D *tiles, const PItem *items, int nitems,
                                const int *shot_items, const InjEnt *ents, const Contrib *cont,
                                const SampleTask *stasks, int n0, int nsteps, unsigned *cnt, unsigned *status,
                                double wait_ms, hipStream_t st)
{
    if (nitems < 1 || nsteps < 1) return hipSuccess;
    switch (vec) {
    case 1: return fwd2d_persist_launch<1>(shots, tiles, items, nitems, shot_items, ents, cont, stasks, n0, nsteps, cnt,
                                           status, wait_ms, st);
    case 2: return fwd2d_persist_launch<2>(shots, tiles, items, nitems, shot_items, ents, cont, stasks, n0, nsteps, cnt,
                                           status, wait_ms, st);
    case 4: return fwd2d_persist_launch<4>(shots, tiles, items, nitems, shot_items, ents, cont, stasks, n0, nsteps, cnt,
                                           status, wait_ms, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_rev2d_persist(int vec, bool grad, const ShotDev *shots, const Tile2D *tiles, const PItem *items,
                                int nitems, const int *shot_items, const InjEnt *ents, const Contrib *cont, int k0,
                                int nsteps, int reinject, float *wadj, unsigned *cnt, unsigned *status,
                                double wait_ms, hipStream_t st)
{
    if (nitems < 1 || nsteps < 1) return hipSuccess;
#define RTM_REVP(V, G) \
    rev2d_persist_launch<V, G>(shots, tiles, items, nitems, shot_items, ents, cont, k0, nsteps, reinject, wadj, cnt, \
                               status, wait_ms, st)
    switch (vec * 2 + (grad ? 1 : 0)) {
    case 2: return RTM_REVP(1, false);
    case 3: return RTM_REVP(1, true);
    case 4: return RTM_REVP(2, false);
    case 5: return RTM_REVP(2, true);
    case 8: return RTM_REVP(4, false);
    case 9: return RTM_REVP(4, true);
    default: return hipErrorInvalidValue;
    }
#undef RTM_REVP
}

hipError_t launch_fwd2d(int vec, int tx, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                        const InjEnt *ents, const Contrib *cont, const SampleTask *stasks, int nsample, int n,
                        hipStream_t st)
{
    dim3 grid(nslots + (nsample + tx - 1) / tx), block(64 * tx);
#define RTM_FWD2D(V, X) \
    hipLaunchKernelGGL((fwd2d_kernel<V, X>), grid, block, 0, st, shots, tiles, ntiles, nslots, ents, cont, stasks, nsample, n)
#define RTM_FWD2D_X(V)                              \
    switch (tx) {                                   \
    case 1: RTM_FWD2D(V, 1); break;                 \
    case 2: RTM_FWD2D(V, 2); break;                 \
    case 4: RTM_FWD2D(V, 4); break;                 \
    default: return hipErrorInvalidValue;           \
    }
    switch (vec) {
    case 1: RTM_FWD2D_X(1); break;
    case 2: RTM_FWD2D_X(2); break;
    case 4: RTM_FWD2D_X(4); break;
    default: return hipErrorInvalidValue;
    }
#undef RTM_FWD2D_X
#undef RTM_FWD2D
    return hipGetLastError();
}

hipError_t launch_rev2d(int vec, int tx, bool grad, const ShotDev *shots, const Tile2D *tiles, int ntiles,
                        int nslots, const InjEnt *ents, const Contrib *cont, int k, int reinject, float *wadj,
                        hipStream_t st)
{
    dim3 grid(nslots), block(64 * tx);
#define RTM_REV2D(V, G, X) \
    hipLaunchKernelGGL((rev2d_kernel<V, G, X>), grid, block, 0, st, shots, tiles, ntiles, nslots, ents, cont, k, reinject, wadj)
#define RTM_REV2D_X(V, G)                           \
    switch (tx) {                                   \
    case 1: RTM_REV2D(V, G, 1); break;              \
    case 2: RTM_REV2D(V, G, 2); break;              \
    case 4: RTM_REV2D(V, G, 4); break;              \
    default: return hipErrorInvalidValue;           \
    }
    if (grad) {
        switch (vec) {
        case 1: RTM_REV2D_X(1, true); break;
        case 2: RTM_REV2D_X(2, true); break;
        case 4: RTM_REV2D_X(4, true); break;
        default: return hipErrorInvalidValue;
        }
    } else {
        switch (vec) {
        case 1: RTM_REV2D_X(1, false); break;
        case 2: RTM_REV2D_X(2, false); break;
        case 4: RTM_REV2D_X(4, false); break;
        default: return hipErrorInvalidValue;
        }
    }
#undef RTM_REV2D_X
#undef RTM_REV2D
    return hipGetLastError();
}

hipError_t launch_recv2d(int vec, int tx, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                         const InjEnt *ents, const Contrib *cont, int k, const float *snap, hipStream_t st)
{
    dim3 grid(nslots), block(64 * tx);
#define RTM_RECV2D(V, X)                                                                                             \
    if (snap)                                                                                                        \
        hipLaunchKernelGGL((recv2d_kernel<V, X, true>), grid, block, 0, st, shots, tiles, ntiles, nslots, ents, cont, k, \
                           snap);                                                                                    \
    else                                                                                                             \
        hipLaunchKernelGGL((recv2d_kernel<V, X, false>), grid, block, 0, st, shots, tiles, ntiles, nslots, ents, cont, \
                           k, snap)
#define RTM_RECV2D_X(V)                             \
    switch (tx) {                                   \
    case 1: RTM_RECV2D(V, 1); break;                \
    case 2: RTM_RECV2D(V, 2); break;                \
    case 4: RTM_RECV2D(V, 4); break;                \
    default: return hipErrorInvalidValue;           \
    }
    switch (vec) {
    case 1: RTM_RECV2D_X(1); break;
    case 2: RTM_RECV2D_X(2); break;
    case 4: RTM_RECV2D_X(4); break;
    default: return hipErrorInvalidValue;
    }
#undef RTM_RECV2D_X
#undef RTM_RECV2D
    return hipGetLastError();
}

}  // namespace rtm
