// 3-D propagation kernels for gfx950.
//
// A workgroup of TY wavefronts owns a tile of 64 * VEC x cells by TY * RW rows
// in y and marches down z over [z0, z1) (a multiple of the 9-plane register
// queue).  Wavefront w holds the RW rows from y0 + w RW on:
//  - z-neighbours come from its register queues of planes z-4 .. z+4;
//  - x-neighbours from the adjacent lanes through DPP, with the 4 + 4 cells
//    beyond the strip ends of all RW rows loaded by one instruction (8 RW
//    lanes) and handed to lanes 0 and 63 through LDS;
//  - y-neighbours from its own rows and, beyond them, from an LDS copy of the
//    centre plane z: every wavefront writes its rows there and the tile's
//    4 + 4 halo rows.  The copy is double-buffered, so one barrier per plane
//    suffices.
// Everything a plane needs from memory (queue rows of plane z + 4, older
// level, D', halos, imaging sums) is loaded one plane ahead in one batch:
// loads return in order, so a load issued and awaited inside the plane would
// also wait for the whole batch behind it.
//
// An access takes a scalar pointer to its plane, which advances in place, and
// one 32-bit vector offset per row.  The pointers are opaque to the compiler:
// it would form every address of nine unrolled planes ahead, and had up to
// 378 scalar registers in vector lanes then, moved back for every access (with
// the rows' offsets scalar as well; on grids in the memory-side cache, where
// instructions count, that took as long as one row of tiles: 144^3 in 1 x 4 x 9
// tiles 17.5 -> 11.2 us, reverse 64^3 17.0 -> 12.1, 300^3 forward 96 -> 91).
//
// Bound: memory traffic.  A forward step must move four arrays, a reverse one
// seven and the imaging sums twice; 612 x 612 x 356 cells (533 MB an array)
// took 581 us (5.6 TB/s with 4.9 arrays read for 3) and 1365 us, of which the
// x-innermost tile order (whole rows of tiles on one XCD) took 25 and 103 us,
// non-temporal access to what a step touches once 22 and 85, and wider and
// taller tiles the rest: now 418 and 1096 us at 5.7 and 5.8 TB/s, with 3.5 arrays
// read for 3 and 9.0 for 6.  501 x 501 x 235: forward 255 -> 165, reverse 596 ->
// 473, receiver 270 -> 178; 188^3, in the memory-side cache: forward 24.7 -> 20.4,
// reverse 65.0 -> 54.3 us.  Two rows per
// wavefront share y-neighbours and halo loads in the reverse kernel, which is
// short of registers for more wavefronts (188^3: 8 rows as 4 x 2 49.6, as
// 8 x 1 57.6 us).
// Stencil, update and injection follow the 2-D kernels (difference form that
// is exactly zero on constant fields; source and receiver terms added after
// the march by the lanes that stored the cells).
#include "multi2d.h"

namespace rtm {
namespace {

typedef __attribute__((address_space(4))) const Tile3D Tile3Entry;

// Number of y-halo rows a wave loads per plane (8 halo rows over TY waves).
template <int TY>
constexpr int halo_per_wave() { return (8 + TY - 1) / TY; }

template <int VEC, int TY, int RW>
struct Lds {
    float row[2][TY * RW + 8][64 * VEC];
    __attribute__((aligned(16))) float ends[2][TY][RW * 8];  // strip-end cells of each row: 4 left, 4 right
};

// Per lane: bit i set where `lane_in` and row y + i lies in [lo, hi).  Kept in
// a vector register: the compiler would otherwise copy the whole march for
// either value of each (uniform) row test.
template <int RW>
__device__ __forceinline__ unsigned row_mask(int y, int lo, int hi, bool lane_in)
{
    unsigned m = 0;
#pragma unroll
    for (int i = 0; i < RW; ++i) m |= lane_in && y + i >= lo && y + i < hi ? 1u << i : 0u;
    return here(m);
}

// What every march knows of its tile.  Field pointers point at row -4, column
// x0 of a plane; rows and columns outside the stored ones are read from the
// zero halo instead, so that no load needs a guard.
template <int VEC, int TY, int RW>
struct Ctx3 {
    int64_t plane4;            // bytes per plane
    // per lane, byte offsets inside a plane (of rows and columns that are stored):
    unsigned row[RW];                    // its columns of each own row
    unsigned hrow[halo_per_wave<TY>()];  // of this wave's y-halo rows
    unsigned erow;                       // its strip-end cell, from x0 - 4
    unsigned own;                        // bit i: this lane stores cells of own row i
    int pitch4, x, x0, y, y0, NX, NY, lane, w;
};

template <int VEC, int TY, int RW>
__device__ __forceinline__ Ctx3<VEC, TY, RW> make_ctx3(ShotEntry &S, Tile3Entry &T)
{
    Ctx3<VEC, TY, RW> C;
    C.pitch4 = (int)S.L.pitch * 4;
    C.plane4 = S.L.plane * 4;
    C.NX = S.L.NX;
    C.NY = S.L.NY;
    C.lane = threadIdx.x & 63;
    C.w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    C.x0 = T.x0;
    C.y0 = T.y0;
    C.x = T.x0 + C.lane * VEC;
    C.y = T.y0 + C.w * RW;
    const unsigned lx = (unsigned)(min(C.x, (C.NX + VEC - 1) / VEC * VEC) - T.x0) * 4u;
    C.own = row_mask<RW>(C.y, 0, C.NY, C.x < C.NX);
    // rows from -4 on, so that the offsets are not negative
#pragma unroll
    for (int i = 0; i < RW; ++i) C.row[i] = (unsigned)(min(C.y + i, C.NY + kRadius - 1) + kRadius) * (unsigned)C.pitch4 + lx;
#pragma unroll
    for (int i = 0; i < halo_per_wave<TY>(); ++i) {
        const int h = C.w + i * TY;
        const int yh = h < 4 ? C.y0 - 4 + h : C.y0 + TY * RW + (h - 4);
        C.hrow[i] = (unsigned)(min(yh, C.NY + kRadius - 1) + kRadius) * (unsigned)C.pitch4 + lx;
    }
    // lane 8 i + e: cell e of row i's 4 left and 4 right strip-end cells
    const int e = C.lane & 7, ye = min(C.y + min(C.lane >> 3, RW - 1), C.NY + kRadius - 1) + kRadius;
    const int xe = e < 4 ? e : min(64 * VEC, C.NX + kRadius - C.x0) + e;  // from x0 - 4; past the grid: zero halo
    C.erow = (unsigned)ye * (unsigned)C.pitch4 + (unsigned)xe * 4u;
    return C;
}

// Everything one field needs from memory for one plane of the wave's rows.
template <int VEC, int TY, int RW>
struct FieldNext {
    float q[RW][VEC];                      // queue rows of plane z + 4
    float halo[halo_per_wave<TY>()][VEC];  // this wave's y-halo rows of plane z
    float end;                             // this lane's strip-end cell of plane z
};

// Advances a pointer by a plane, in place (see the head of the file).
template <class P>
__device__ __forceinline__ void next_plane(P &p, int64_t plane4)
{
    p = at(p, plane4);
    asm("" : "+s"(p));
}

// A field read at planes z (strip ends and y-halo) and z + 4 (queue rows).
struct Field3 {
    const gfloat *z, *z4;
    __device__ __forceinline__ void start(const gfloat *f, int64_t plane4)
    {
        z = f;
        z4 = at(f, 4 * plane4);
    }
    __device__ __forceinline__ void next(int64_t plane4)
    {
        next_plane(z, plane4);
        next_plane(z4, plane4);
    }
};

// Issues the loads of field f for its plane.
template <int VEC, int TY, int RW>
__device__ __forceinline__ void field_prefetch(const Ctx3<VEC, TY, RW> &C, const Field3 &f, FieldNext<VEC, TY, RW> &nx)
{
#pragma unroll
    for (int i = 0; i < RW; ++i) ldv<VEC>(at(f.z4, here(C.row[i])), nx.q[i]);
#pragma unroll
    for (int i = 0; i < halo_per_wave<TY>(); ++i)
        if (TY <= 8 || C.w + i * TY < 8) ldv<VEC>(at(f.z, here(C.hrow[i])), nx.halo[i]);
    if (C.lane < 8 * RW) nx.end = *at(f.z - 4, here(C.erow));
}

// Writes the centre rows (queue slot of plane z), the y-halo rows and the
// strip-end cells into LDS buffer `buf`.
template <int VEC, int TY, int RW>
__device__ __forceinline__ void field_publish(const Ctx3<VEC, TY, RW> &C, Lds<VEC, TY, RW> &L, int buf,
                                              const float (&c)[RW][VEC], const FieldNext<VEC, TY, RW> &nx)
{
#pragma unroll
    for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int j = 0; j < VEC; ++j) L.row[buf][4 + C.w * RW + i][C.lane * VEC + j] = c[i][j];
#pragma unroll
    for (int i = 0; i < halo_per_wave<TY>(); ++i) {
        const int h = C.w + i * TY;
        if (TY <= 8 || h < 8) {
            const int slot = h < 4 ? h : TY * RW + 4 + (h - 4);
#pragma unroll
            for (int j = 0; j < VEC; ++j) L.row[buf][slot][C.lane * VEC + j] = nx.halo[i][j];
        }
    }
    if (C.lane < 8 * RW) L.ends[buf][C.w][C.lane] = nx.end;
}

// Unscaled 3-D Laplacian of the wave's centre cells; q[k]: planes z - 4 + k
// (rotated by S).
template <int VEC, int TY, int RW, int S>
__device__ __forceinline__ void lap3(const Ctx3<VEC, TY, RW> &C, const Lds<VEC, TY, RW> &L, int buf,
                                     const float (&q)[9][RW][VEC], float (&lap)[RW][VEC])
{
    constexpr int r0 = (S + 0) % 9, r1 = (S + 1) % 9, r2 = (S + 2) % 9, r3 = (S + 3) % 9, r4 = (S + 4) % 9,
                  r5 = (S + 5) % 9, r6 = (S + 6) % 9, r7 = (S + 7) % 9, r8 = (S + 8) % 9;
    float yn[RW + 8][VEC];  // rows y - 4 .. y + RW + 3 of plane z
#pragma unroll
    for (int i = 0; i < RW + 8; ++i)
#pragma unroll
        for (int j = 0; j < VEC; ++j)
            yn[i][j] = i >= 4 && i < RW + 4 ? q[r4][i - 4 < 0 ? 0 : (i - 4 >= RW ? 0 : i - 4)][j]
                                            : L.row[buf][C.w * RW + i][C.lane * VEC + j];
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        float hl[4], hr[4], ext[VEC + 8];
        halo_split(*(const f4v *)&L.ends[buf][C.w][8 * i + (C.lane < 32 ? 0 : 4)], C.lane, hl, hr);
        exchange_row<VEC>(q[r4][i], hl, hr, ext);
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            const float c = q[r4][i][j], c2 = c + c;
            float l = d2(c2, ext[3 + j], ext[5 + j], ext[2 + j], ext[6 + j], ext[1 + j], ext[7 + j], ext[j], ext[8 + j]);
            l += d2(c2, yn[i + 3][j], yn[i + 5][j], yn[i + 2][j], yn[i + 6][j], yn[i + 1][j], yn[i + 7][j], yn[i][j],
                    yn[i + 8][j]);
            l += d2(c2, q[r3][i][j], q[r5][i][j], q[r2][i][j], q[r6][i][j], q[r1][i][j], q[r7][i][j], q[r0][i][j],
                    q[r8][i][j]);
            lap[i][j] = l;
        }
    }
}

// The wave's rows of the plane that f points at.
template <int VEC, int TY, int RW, bool NT>
__device__ __forceinline__ void plane_load(const Ctx3<VEC, TY, RW> &C, const gfloat *f, float (&v)[RW][VEC])
{
#pragma unroll
    for (int i = 0; i < RW; ++i) ld_once<VEC, NT>(at(f, here(C.row[i])), v[i]);
}

template <int VEC, int TY, int RW, bool NT>
__device__ __forceinline__ void plane_store(const Ctx3<VEC, TY, RW> &C, gfloat *f, const float (&v)[RW][VEC])
{
#pragma unroll
    for (int i = 0; i < RW; ++i)
        if (C.own >> i & 1) st_once<VEC, NT>(at(f, here(C.row[i])), v[i]);
}

// One field's update (forward pass, receiver field of storage RTM).  IMG: at
// a stored level, the imaging sums take p^k from the dense snapshot.
template <int VEC, int TY, int RW, bool IMG>
struct StepIn {
    FieldNext<VEC, TY, RW> f;
    float old[RW][VEC], d[RW][VEC];
    float s[IMG ? RW : 1][VEC], a[IMG ? RW : 1][VEC], b[IMG ? RW : 1][VEC];
};

template <int VEC, int TY, int RW, bool IMG>
struct Step3 {
    Field3 pc;              // all at the plane to load next ...
    const gfloat *old, *Dp, *A0, *A1;
    gfloat *po, *S0, *S1;   // ... and at the plane to store
    SnapImg I;
    int z1;
    unsigned izn;   // interior planes from I.iz0
    unsigned mask;  // per lane: the own rows that hold interior cells
};

template <int VEC, int TY, int RW, bool IMG, bool NT>
__device__ __forceinline__ void step_fetch(const Ctx3<VEC, TY, RW> &C, Step3<VEC, TY, RW, IMG> &K, int z,
                                           StepIn<VEC, TY, RW, IMG> &in)
{
    field_prefetch<VEC, TY, RW>(C, K.pc, in.f);
    plane_load<VEC, TY, RW, NT>(C, K.old, in.old);
    plane_load<VEC, TY, RW, NT>(C, K.Dp, in.d);
    if constexpr (IMG)
        if (in_rows(z, K.I.iz0, K.izn)) {
#pragma unroll
            for (int i = 0; i < RW; ++i)
                if (K.mask >> i & 1) {
                    const int64_t row = ((int64_t)(z - K.I.iz0) * K.I.nyi + (C.y + i - K.I.iy0)) * K.I.nxi - K.I.ix0;
#pragma unroll
                    for (int j = 0; j < VEC; ++j)
                        in.s[i][j] = C.x + j >= K.I.ix0 && C.x + j < K.I.ix1 ? K.I.snap[row + C.x + j] : 0.f;
                    ld_once<VEC, NT>(at(K.A0, here(C.row[i])), in.a[i]);
                    ld_once<VEC, NT>(at(K.A1, here(C.row[i])), in.b[i]);
                }
        }
    K.pc.next(C.plane4);
    next_plane(K.old, C.plane4);
    next_plane(K.Dp, C.plane4);
    if constexpr (IMG) {
        next_plane(K.A0, C.plane4);
        next_plane(K.A1, C.plane4);
    }
}

template <int VEC, int TY, int RW, bool NT, bool IMG, int S>
__device__ __forceinline__ void step_plane(const Ctx3<VEC, TY, RW> &C, Step3<VEC, TY, RW, IMG> &K, Lds<VEC, TY, RW> &L,
                                           float (&q)[9][RW][VEC], StepIn<VEC, TY, RW, IMG> &in, int z)
{
    constexpr int r4 = (S + 4) % 9, r8 = (S + 8) % 9;
    const int buf = z & 1;
    float old[RW][VEC], d[RW][VEC], sn[RW][VEC], sa[RW][VEC], sb[RW][VEC];
#pragma unroll
    for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            q[r8][i][j] = in.f.q[i][j];
            old[i][j] = in.old[i][j];
            d[i][j] = in.d[i][j];
            if constexpr (IMG) {
                sn[i][j] = in.s[i][j];
                sa[i][j] = in.a[i][j];
                sb[i][j] = in.b[i][j];
            }
        }
    field_publish<VEC, TY, RW>(C, L, buf, q[r4], in.f);
    if (z + 1 < K.z1) step_fetch<VEC, TY, RW, IMG, NT>(C, K, z + 1, in);
    __syncthreads();
    float lap[RW][VEC];
    lap3<VEC, TY, RW, S>(C, L, buf, q, lap);
#pragma unroll
    for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int j = 0; j < VEC; ++j) lap[i][j] = fmaf(d[i][j], lap[i][j], (q[r4][i][j] + q[r4][i][j]) - old[i][j]);
    plane_store<VEC, TY, RW, NT>(C, K.po, lap);
    if constexpr (IMG)
        if (in_rows(z, K.I.iz0, K.izn)) {
#pragma unroll
            for (int i = 0; i < RW; ++i)
                if (K.mask >> i & 1) {
#pragma unroll
                    for (int j = 0; j < VEC; ++j) {
                        sa[i][j] = fmaf(sn[i][j], q[r4][i][j], sa[i][j]);
                        sb[i][j] = fmaf(sn[i][j], sn[i][j], sb[i][j]);
                    }
                    st_once<VEC, NT>(at(K.S0, here(C.row[i])), sa[i]);
                    st_once<VEC, NT>(at(K.S1, here(C.row[i])), sb[i]);
                }
        }
    next_plane(K.po, C.plane4);
    if constexpr (IMG) {
        next_plane(K.S0, C.plane4);
        next_plane(K.S1, C.plane4);
    }
}

// Runs ROWCALL(S, z) over the tile's planes, nine per trip (z1 - z0 is a
// multiple of nine), so that S = (z - z0) mod 9 is a compile-time constant.
#define RTM_MARCH3(ROWCALL)                                                                    \
    for (int z = T.z0; z < T.z1; z += kZUnroll) {                                              \
        ROWCALL(0, z); ROWCALL(1, z + 1); ROWCALL(2, z + 2); ROWCALL(3, z + 3);                \
        ROWCALL(4, z + 4); ROWCALL(5, z + 5); ROWCALL(6, z + 6); ROWCALL(7, z + 7);            \
        ROWCALL(8, z + 8);                                                                     \
    }

template <int VEC, int TY, int RW, bool NT, bool IMG>
__device__ __forceinline__ void step_march(const Ctx3<VEC, TY, RW> &C, Step3<VEC, TY, RW, IMG> &K, Lds<VEC, TY, RW> &L,
                                           Tile3Entry &T)
{
    float q[9][RW][VEC];
    StepIn<VEC, TY, RW, IMG> in;
#pragma unroll
    for (int i = 0; i < 8; ++i) plane_load<VEC, TY, RW, false>(C, at(K.pc.z, (i - 4) * C.plane4), q[i]);
    step_fetch<VEC, TY, RW, IMG, NT>(C, K, T.z0, in);
#define RTM_STEP3(SS, ZZ) step_plane<VEC, TY, RW, NT, IMG, SS>(C, K, L, q, in, ZZ)
    RTM_MARCH3(RTM_STEP3)
#undef RTM_STEP3
}

// Does this wave-lane own padded cell (y, x) of the tile?
template <int VEC, int TY, int RW>
__device__ __forceinline__ bool owns3(const Ctx3<VEC, TY, RW> &C, int y, int x)
{
    return y >= C.y && y < C.y + RW && x >= C.x && x < C.x + VEC;
}

// The fused reverse pair of fields.
template <int VEC, int TY, int RW, bool GRAD>
struct RevIn3 {
    FieldNext<VEC, TY, RW> p, m;
    float p1[RW][VEC], m1[RW][VEC], d[RW][VEC], a[RW][VEC], b[GRAD ? 1 : RW][VEC];
};

template <int VEC, int TY, int RW, bool GRAD>
struct Rev3 {
    Field3 P0, M0;                             // all at the plane to load next ...
    const gfloat *P1, *M1, *Dp, *A0, *A1;
    gfloat *WP, *WM, *S0, *S1;                 // ... and at the plane to store
    int z1, alo;    // the sums cover planes [alo, alo + an) ...
    unsigned an;
    unsigned mask;  // ... and, per lane, these of the own rows
};

template <int VEC, int TY, int RW, bool GRAD, bool NT>
__device__ __forceinline__ void rev_fetch3(const Ctx3<VEC, TY, RW> &C, Rev3<VEC, TY, RW, GRAD> &K, int z,
                                           RevIn3<VEC, TY, RW, GRAD> &in)
{
    field_prefetch<VEC, TY, RW>(C, K.P0, in.p);
    field_prefetch<VEC, TY, RW>(C, K.M0, in.m);
    plane_load<VEC, TY, RW, NT>(C, K.P1, in.p1);
    plane_load<VEC, TY, RW, NT>(C, K.M1, in.m1);
    plane_load<VEC, TY, RW, NT>(C, K.Dp, in.d);
    if (in_rows(z, K.alo, K.an)) {
#pragma unroll
        for (int i = 0; i < RW; ++i)
            if (K.mask >> i & 1) {
                ld_once<VEC, NT>(at(K.A0, here(C.row[i])), in.a[i]);
                if constexpr (!GRAD) ld_once<VEC, NT>(at(K.A1, here(C.row[i])), in.b[i]);
            }
    }
    K.P0.next(C.plane4);
    K.M0.next(C.plane4);
    next_plane(K.P1, C.plane4);
    next_plane(K.M1, C.plane4);
    next_plane(K.Dp, C.plane4);
    next_plane(K.A0, C.plane4);
    if constexpr (!GRAD) next_plane(K.A1, C.plane4);
}

template <int VEC, int TY, int RW, bool NT, bool GRAD, int S>
__device__ __forceinline__ void rev_plane3(const Ctx3<VEC, TY, RW> &C, Rev3<VEC, TY, RW, GRAD> &K,
                                           Lds<VEC, TY, RW> &LP, Lds<VEC, TY, RW> &LM, float (&qp)[9][RW][VEC],
                                           float (&qm)[9][RW][VEC], RevIn3<VEC, TY, RW, GRAD> &in, int z)
{
    constexpr int r4 = (S + 4) % 9, r8 = (S + 8) % 9;
    const int buf = z & 1;
    float p1[RW][VEC], m1[RW][VEC], d[RW][VEC], a[RW][VEC], b[RW][VEC];
#pragma unroll
    for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            qp[r8][i][j] = in.p.q[i][j];
            qm[r8][i][j] = in.m.q[i][j];
            p1[i][j] = in.p1[i][j];
            m1[i][j] = in.m1[i][j];
            d[i][j] = in.d[i][j];
            a[i][j] = in.a[i][j];
            if constexpr (!GRAD) b[i][j] = in.b[i][j];
        }
    field_publish<VEC, TY, RW>(C, LP, buf, qp[r4], in.p);
    field_publish<VEC, TY, RW>(C, LM, buf, qm[r4], in.m);
    if (z + 1 < K.z1) rev_fetch3<VEC, TY, RW, GRAD, NT>(C, K, z + 1, in);
    __syncthreads();
    float lp[RW][VEC], lm[RW][VEC];
    lap3<VEC, TY, RW, S>(C, LP, buf, qp, lp);
#pragma unroll
    for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int j = 0; j < VEC; ++j) {
            const float cp = qp[r4][i][j], inc = d[i][j] * lp[i][j];
            if constexpr (GRAD) {
                a[i][j] = fmaf(qm[r4][i][j], inc, a[i][j]);
            } else {
                a[i][j] = fmaf(cp, qm[r4][i][j], a[i][j]);
                b[i][j] = fmaf(cp, cp, b[i][j]);
            }
            lp[i][j] = inc + ((cp + cp) - p1[i][j]);
        }
    plane_store<VEC, TY, RW, NT>(C, K.WP, lp);
    lap3<VEC, TY, RW, S>(C, LM, buf, qm, lm);
#pragma unroll
    for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int j = 0; j < VEC; ++j) lm[i][j] = fmaf(d[i][j], lm[i][j], (qm[r4][i][j] + qm[r4][i][j]) - m1[i][j]);
    plane_store<VEC, TY, RW, NT>(C, K.WM, lm);
    if (in_rows(z, K.alo, K.an)) {
#pragma unroll
        for (int i = 0; i < RW; ++i)
            if (K.mask >> i & 1) {
                st_once<VEC, NT>(at(K.S0, here(C.row[i])), a[i]);
                if constexpr (!GRAD) st_once<VEC, NT>(at(K.S1, here(C.row[i])), b[i]);
            }
    }
    next_plane(K.WP, C.plane4);
    next_plane(K.WM, C.plane4);
    next_plane(K.S0, C.plane4);
    if constexpr (!GRAD) next_plane(K.S1, C.plane4);
}

}  // namespace

// Field pointer at (y = -4, x = x0) of plane z0, as Ctx3's row offsets count.
#define RTM_AT3(f) at(gp(f) + S.L.org - kRadius * S.L.pitch + T.x0, (int64_t)T.z0 * C.plane4)

// Forward step n (see the 2-D kernel): tiles of 64*VEC x TY*RW x (z1 - z0).
// Workgroups past the stencil slots record d^n = R p^n, one receiver task
// of 64 per wavefront.
template <int VEC, int TY, int RW, bool NT>
__global__ __launch_bounds__(64 * TY) void fwd3d_kernel(const ShotDev *__restrict__ shots,
                                                        const Tile3D *__restrict__ tiles, int ntiles, int nslots,
                                                        const InjEnt *__restrict__ ents,
                                                        const Contrib *__restrict__ cont,
                                                        const SampleTask *__restrict__ stasks, int nsample, int n)
{
    __shared__ Lds<VEC, TY, RW> L;
    const int b = blockIdx.x;
    if (b >= nslots) {
        const int task = (b - nslots) * TY + (int)(threadIdx.x >> 6);
        if (task < nsample) sample_body(shots, stasks[task], n, n & 1, (int)(threadIdx.x & 63));
        return;
    }
    const int t = xcd_tile(b, nslots);
    if (t >= ntiles) return;
    Tile3Entry &T = *(Tile3Entry *)(uintptr_t)(tiles + t);
    ShotEntry &S = *(ShotEntry *)(uintptr_t)(shots + T.shot);
    const Ctx3<VEC, TY, RW> C = make_ctx3<VEC, TY, RW>(S, T);
    Step3<VEC, TY, RW, false> K{};
    K.pc.start(RTM_AT3(S.fld[n & 1]), C.plane4);
    K.old = K.po = RTM_AT3(S.fld[(n + 1) & 1]);
    K.Dp = RTM_AT3(S.Dp);
    K.z1 = T.z1;
    step_march<VEC, TY, RW, NT, false>(C, K, L, T);
    const float *wav = S.wav + n;
    for (int e = T.sbeg; e < T.send; ++e) {
        const InjEnt E = ents[e];
        if (owns3(C, E.y, E.x)) {
            const int64_t o = (int64_t)E.z * S.L.plane + (int64_t)E.y * S.L.pitch + E.x;
            gfloat *po = gp(S.fld[(n + 1) & 1]) + S.L.org;
            po[o] = fmaf((gp(S.Dp) + S.L.org)[o], inj_sum(E, cont, wav), po[o]);
        }
    }
}

// Reverse step k (see the 2-D kernel), with LDS copies of both fields.
template <int VEC, int TY, int RW, bool NT, bool GRAD>
__global__ __launch_bounds__(64 * TY) void rev3d_kernel(const ShotDev *__restrict__ shots,
                                                        const Tile3D *__restrict__ tiles, int ntiles, int nslots,
                                                        const InjEnt *__restrict__ ents,
                                                        const Contrib *__restrict__ cont, int k, int reinject,
                                                        float *__restrict__ wadj)
{
    __shared__ Lds<VEC, TY, RW> LP, LM;
    const int t = xcd_tile(blockIdx.x, nslots);
    if (t >= ntiles) return;
    Tile3Entry &T = *(Tile3Entry *)(uintptr_t)(tiles + t);
    ShotEntry &S = *(ShotEntry *)(uintptr_t)(shots + T.shot);
    const Ctx3<VEC, TY, RW> C = make_ctx3<VEC, TY, RW>(S, T);
    Rev3<VEC, TY, RW, GRAD> K;
    K.P0.start(RTM_AT3(S.fld[k & 1]), C.plane4);
    K.M0.start(RTM_AT3(S.fld[2 + ((k + 1) & 1)]), C.plane4);
    K.P1 = K.WP = RTM_AT3(S.fld[(k + 1) & 1]);
    K.M1 = K.WM = RTM_AT3(S.fld[2 + (k & 1)]);
    K.Dp = RTM_AT3(S.Dp);
    K.A0 = K.S0 = RTM_AT3(S.acc0);
    K.A1 = K.S1 = GRAD ? nullptr : RTM_AT3(S.acc1);
    K.z1 = T.z1;
    // the gradient sum covers the whole padded grid, the imaging sums the interior
    K.alo = GRAD ? T.z0 : max(T.z0, S.iz0);
    K.an = (unsigned)max((GRAD ? T.z1 : min(T.z1, S.iz1)) - K.alo, 0);
    K.mask = GRAD ? C.own : row_mask<RW>(C.y, S.iy0, S.iy1, C.x + VEC > S.ix0 && C.x < S.ix1);
    float qp[9][RW][VEC], qm[9][RW][VEC];
    RevIn3<VEC, TY, RW, GRAD> in;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        plane_load<VEC, TY, RW, false>(C, at(K.P0.z, (i - 4) * C.plane4), qp[i]);
        plane_load<VEC, TY, RW, false>(C, at(K.M0.z, (i - 4) * C.plane4), qm[i]);
    }
    rev_fetch3<VEC, TY, RW, GRAD, NT>(C, K, T.z0, in);
#define RTM_REV3(SS, ZZ) rev_plane3<VEC, TY, RW, NT, GRAD, SS>(C, K, LP, LM, qp, qm, in, ZZ)
    RTM_MARCH3(RTM_REV3)
#undef RTM_REV3
    const gfloat *Dp = gp(S.Dp) + S.L.org, *M0 = gp(S.fld[2 + ((k + 1) & 1)]) + S.L.org;
    gfloat *P1 = gp(S.fld[(k + 1) & 1]) + S.L.org, *A0 = gp(S.acc0) + S.L.org;
    const float *wav = S.wav + k;
    for (int e = T.sbeg; e < T.send; ++e) {
        const InjEnt E = ents[e];
        if (owns3(C, E.y, E.x)) {
            const int64_t o = (int64_t)E.z * S.L.plane + (int64_t)E.y * S.L.pitch + E.x;
            const float ds = Dp[o] * inj_sum(E, cont, wav);
            if (reinject) P1[o] = P1[o] + ds;
            if (GRAD) A0[o] = fmaf(M0[o], ds, A0[o]);
            if (wadj) {
                float wsum = 0.f;
                for (int c = E.cbeg; c < E.cend; ++c) wsum += cont[c].w;
                wadj[(int64_t)k * kMaxNodes + E.slot] = wsum * M0[o];
            }
        }
    }
    inject_nodes(gp(S.fld[2 + (k & 1)]) + S.L.org, Dp, ents, T.rbeg, T.rend, cont, S.sig + (int64_t)k * S.nrec, S.L.plane,
                 S.L.pitch);
}

// Receiver wavefield alone, for migration with a stored source wavefield
// (see the 2-D kernel): the forward plane update applied to mu, with the
// imaging sums at a stored level taking p^k from the dense snapshot (IMG).
template <int VEC, int TY, int RW, bool NT, bool IMG>
__global__ __launch_bounds__(64 * TY) void recv3d_kernel(const ShotDev *__restrict__ shots,
                                                         const Tile3D *__restrict__ tiles, int ntiles, int nslots,
                                                         const InjEnt *__restrict__ ents,
                                                         const Contrib *__restrict__ cont, int k,
                                                         const float *__restrict__ snap)
{
    __shared__ Lds<VEC, TY, RW> L;
    const int t = xcd_tile(blockIdx.x, nslots);
    if (t >= ntiles) return;
    Tile3Entry &T = *(Tile3Entry *)(uintptr_t)(tiles + t);
    ShotEntry &S = *(ShotEntry *)(uintptr_t)(shots + T.shot);
    const Ctx3<VEC, TY, RW> C = make_ctx3<VEC, TY, RW>(S, T);
    Step3<VEC, TY, RW, IMG> K{};
    K.pc.start(RTM_AT3(S.fld[2 + ((k + 1) & 1)]), C.plane4);  // mu^{k+1}
    K.old = K.po = RTM_AT3(S.fld[2 + (k & 1)]);               // mu^{k+2} -> mu^k
    K.Dp = RTM_AT3(S.Dp);
    K.z1 = T.z1;
    if constexpr (IMG) {
        K.A0 = K.S0 = RTM_AT3(S.acc0);
        K.A1 = K.S1 = RTM_AT3(S.acc1);
        K.I = SnapImg{snap, S.ix1 - S.ix0, S.iy1 - S.iy0, S.ix0, S.ix1, S.iy0, S.iz0};
        K.izn = (unsigned)(S.iz1 - S.iz0);
        K.mask = row_mask<RW>(C.y, S.iy0, S.iy1, C.x + VEC > S.ix0 && C.x < S.ix1);
    }
    step_march<VEC, TY, RW, NT, IMG>(C, K, L, T);
    inject_nodes(gp(S.fld[2 + (k & 1)]) + S.L.org, gp(S.Dp) + S.L.org, ents, T.rbeg, T.rend, cont,
                 S.sig + (int64_t)k * S.nrec, S.L.plane, S.L.pitch);
}

// `code` is floats per lane | kOnce where the arrays of a step exceed the
// memory-side cache; `ty` rows per tile.  CALL takes floats per lane,
// wavefronts and rows per wavefront: one row each, but two of 16 rows at one
// float per lane and, in the reverse kernels (two fields, twice the
// registers), of eight rows at one and two floats.
#define RTM_ONCE3(CALL, V, Y, R) do { if (once) CALL(V, Y, R, true); else CALL(V, Y, R, false); } while (0)
#define RTM_FWD_SHAPES(CALL)                        \
    switch (vec << 8 | ty) {                        \
    case 0x104: RTM_ONCE3(CALL, 1, 4, 1); break;    \
    case 0x108: RTM_ONCE3(CALL, 1, 8, 1); break;    \
    case 0x110: RTM_ONCE3(CALL, 1, 8, 2); break;    \
    case 0x204: RTM_ONCE3(CALL, 2, 4, 1); break;    \
    case 0x208: RTM_ONCE3(CALL, 2, 8, 1); break;    \
    case 0x210: RTM_ONCE3(CALL, 2, 16, 1); break;   \
    case 0x404: RTM_ONCE3(CALL, 4, 4, 1); break;    \
    case 0x408: RTM_ONCE3(CALL, 4, 8, 1); break;    \
    default: return hipErrorInvalidValue;           \
    }
#define RTM_REV_SHAPES(CALL)                        \
    switch (vec << 8 | ty) {                        \
    case 0x104: RTM_ONCE3(CALL, 1, 4, 1); break;    \
    case 0x108: RTM_ONCE3(CALL, 1, 4, 2); break;    \
    case 0x110: RTM_ONCE3(CALL, 1, 8, 2); break;    \
    case 0x204: RTM_ONCE3(CALL, 2, 4, 1); break;    \
    case 0x208: RTM_ONCE3(CALL, 2, 4, 2); break;    \
    case 0x404: RTM_ONCE3(CALL, 4, 4, 1); break;    \
    case 0x408: RTM_ONCE3(CALL, 4, 8, 1); break;    \
    default: return hipErrorInvalidValue;           \
    }

hipError_t launch_fwd3d(int code, int ty, const ShotDev *shots, const Tile3D *tiles, int ntiles, int nslots,
                        const InjEnt *ents, const Contrib *cont, const SampleTask *stasks, int nsample, int n,
                        hipStream_t st)
{
    const int vec = code & 0xff;
    const bool once = code & kOnce;
    if (!stasks) nsample = 0;
#define RTM_F3(V, Y, R, N)                                                                                          \
    hipLaunchKernelGGL((fwd3d_kernel<V, Y, R, N>), dim3(nslots + (nsample + Y - 1) / Y), dim3(64 * Y), 0, st, shots, \
                       tiles, ntiles, nslots, ents, cont, stasks, nsample, n)
    RTM_FWD_SHAPES(RTM_F3)
#undef RTM_F3
    return hipGetLastError();
}

hipError_t launch_rev3d(int code, int ty, bool grad, const ShotDev *shots, const Tile3D *tiles, int ntiles, int nslots,
                        const InjEnt *ents, const Contrib *cont, int k, int reinject, float *wadj, hipStream_t st)
{
    const int vec = code & 0xff;
    const bool once = code & kOnce;
#define RTM_R3(V, Y, R, N)                                                                                         \
    do {                                                                                                           \
        if (grad)                                                                                                  \
            hipLaunchKernelGGL((rev3d_kernel<V, Y, R, N, true>), dim3(nslots), dim3(64 * Y), 0, st, shots, tiles,  \
                               ntiles, nslots, ents, cont, k, reinject, wadj);                                     \
        else                                                                                                       \
            hipLaunchKernelGGL((rev3d_kernel<V, Y, R, N, false>), dim3(nslots), dim3(64 * Y), 0, st, shots, tiles, \
                               ntiles, nslots, ents, cont, k, reinject, wadj);                                     \
    } while (0)
    RTM_REV_SHAPES(RTM_R3)
#undef RTM_R3
    return hipGetLastError();
}

hipError_t launch_recv3d(int code, int ty, const ShotDev *shots, const Tile3D *tiles, int ntiles, int nslots,
                         const InjEnt *ents, const Contrib *cont, int k, const float *snap, hipStream_t st)
{
    const int vec = code & 0xff;
    const bool once = code & kOnce;
#define RTM_RC3(V, Y, R, N)                                                                                         \
    do {                                                                                                            \
        if (snap)                                                                                                   \
            hipLaunchKernelGGL((recv3d_kernel<V, Y, R, N, true>), dim3(nslots), dim3(64 * Y), 0, st, shots, tiles,  \
                               ntiles, nslots, ents, cont, k, snap);                                                \
        else                                                                                                        \
            hipLaunchKernelGGL((recv3d_kernel<V, Y, R, N, false>), dim3(nslots), dim3(64 * Y), 0, st, shots, tiles, \
                               ntiles, nslots, ents, cont, k, snap);                                                \
    } while (0)
    RTM_FWD_SHAPES(RTM_RC3)
#undef RTM_RC3
    return hipGetLastError();
}

}  // namespace rtm
