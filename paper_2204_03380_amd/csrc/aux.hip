// Auxiliary kernels of librtm: random boundary padding and its adjoint,
// preparation of the scaled velocity term, trace transposes, receiver-field
// start, last-sample recording, image and gradient finalisation, and field
// unpacking.  All run once per call (not per time step).
#include <algorithm>

#include "common.h"

namespace rtm {
namespace {

constexpr int kBlock = 256;

__device__ __forceinline__ int64_t gstride() { return (int64_t)gridDim.x * blockDim.x; }
__device__ __forceinline__ int64_t gid() { return (int64_t)blockIdx.x * blockDim.x + threadIdx.x; }

inline unsigned grid_for(int64_t n)
{
    int64_t b = (n + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    if (b > 65536) b = 65536;
    return (unsigned)b;
}

// Grid for reductions: kPer elements per thread and round, at most four
// blocks per CU.  Each block ends in one atomic on the same word, which cost
// more than the reading on small arrays (1.2 MB: 13 us with one element per
// thread and up to 1024 blocks, 4.7 with sixteen).
constexpr int kPer = 8;

inline unsigned grid_reduce(int64_t n)
{
    const int64_t b = (n + 2 * kPer * kBlock - 1) / (2 * kPer * kBlock);
    return (unsigned)std::min<int64_t>(std::max<int64_t>(b, 1), 1024);
}

// Wavefronts over rows (612 x 612 x 356 cells, us: image 232 -> 140, den_max 212
// -> 91, build_dp 416 -> 297; 401 x 401 x 135 snapshot 82 -> 47, with one cell
// per thread and its divisions before): wavefront w of the grid takes chunks of 256 columns,
// F(row, x0) with x0 the chunk's first column, four columns per lane at x0 +
// lane + 64 u.  Row and chunk are uniform, so their divisions cost nothing
// per cell.  rows * chunks fits 32 bits (grids hold fewer than 2^31 cells).
constexpr int kChunk = 256;

template <class F>
__device__ __forceinline__ void chunks_do(unsigned rows, unsigned len, F f)
{
    const unsigned per = (len + kChunk - 1) / kChunk, n = rows * per;
    const unsigned w = __builtin_amdgcn_readfirstlane(blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6));
    for (unsigned i = w; i < n; i += gridDim.x * (kBlock / 64)) {
        const unsigned row = i / per;
        f(row, (i - row * per) * kChunk + (threadIdx.x & 63));
    }
}

inline unsigned grid_chunks(int64_t rows, int64_t len)
{
    const int64_t n = (rows * ((len + kChunk - 1) / kChunk) + kBlock / 64 - 1) / (kBlock / 64);
    return (unsigned)std::min<int64_t>(std::max<int64_t>(n, 1), 16384);
}

// SplitMix64 (Steele, Lea & Flood 2014): output number k + 1 of the stream
// seeded with `seed` (state advanced by the golden-ratio increment, then the
// 64-bit finaliser).
__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t k)
{
    uint64_t z = seed + (k + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Random factor of band cell j, uniform in [0.7, 1.3): one FP32 fma of the
// exact 24-bit fraction.
__device__ __forceinline__ float rbc_factor(uint64_t seed, uint64_t j)
{
    const float u = (float)(splitmix64_at(seed, j) >> 40) * (1.0f / 16777216.0f);
    return __builtin_fmaf(0.6f, u, 0.7f);
}

struct PadDims {
    int ndim;
    int nb;
    int64_t nx, ny, nz;
    int64_t NX, NY, NZ;
};

__device__ __forceinline__ int64_t clampi(int64_t v, int64_t lo, int64_t hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Distance of a padded coordinate from the interior [0, n) along one axis.
__device__ __forceinline__ int64_t band_depth(int64_t a, int64_t n) { return a < 0 ? -a : (a >= n ? a - n + 1 : 0); }

// Depth of a band cell: the largest per-axis distance from the interior.
__device__ __forceinline__ int64_t cell_depth(const PadDims &d, int64_t ix, int64_t iy, int64_t iz)
{
    int64_t m = band_depth(ix, d.nx);
    m = max(m, band_depth(iz, d.nz));
    if (d.ndim == 3) m = max(m, band_depth(iy, d.ny));
    return m;
}

// Block-wide max / min of unsigned values (kBlock threads), then one
// atomic per block.
template <bool MAX>
__device__ __forceinline__ void block_reduce_atomic(unsigned m, unsigned *out)
{
    __shared__ unsigned part[kBlock / 64];
    for (int off = 32; off > 0; off >>= 1) {
        unsigned o = (unsigned)__shfl_xor((int)m, off);
        m = MAX ? max(m, o) : min(m, o);
    }
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) m = MAX ? max(m, part[w]) : min(m, part[w]);
        if (MAX) atomicMax(out, m);
        else atomicMin(out, m);
    }
}

// Largest and (MIN) smallest IEEE bit pattern into out[0], out[1]: for positive
// finite data these are the maximum and the minimum; a NaN, infinity or
// negative value compares above +inf's pattern.  One pass over the data, eight
// loads in flight per thread (1.2 MB: 4.7 us, two passes with one took 27; 533 MB:
// 121 and 458).
template <bool MIN>
__global__ __launch_bounds__(kBlock) void vrange_kernel(const float *__restrict__ v, int64_t n,
                                                        unsigned *__restrict__ out)
{
    unsigned hi = 0u, lo = 0xffffffffu;
    for (int64_t i = gid(); i < n; i += kPer * gstride()) {
        unsigned x[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u) x[u] = __float_as_uint(v[min(i + u * gstride(), n - 1)]);
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            hi = max(hi, x[u]);
            lo = min(lo, x[u]);
        }
    }
    block_reduce_atomic<true>(hi, out);
    if (MIN) block_reduce_atomic<false>(lo, out + 1);
}

// out[i] = i odd ? odd : even.
__global__ void set_u32_kernel(unsigned *__restrict__ p, int n, unsigned even, unsigned odd)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = i & 1 ? odd : even;
}

// Band cell value: min(f_j v_edge, cap); with the taper min(c_i (f_j v_edge),
// cap) at depth i; 0 above the interior with the free surface.
__global__ void rbc_pad_kernel(PadDims d, const float *__restrict__ v_int, uint64_t seed, float v_cap,
                               const unsigned *__restrict__ cap_bits, BandOpts o, float *__restrict__ v_pad)
{
    const float cap = cap_bits ? __uint_as_float(*cap_bits) : v_cap;
    const int64_t n = d.NX * d.NY * d.NZ;
    for (int64_t j = gid(); j < n; j += gstride()) {
        const int64_t x = j % d.NX;
        const int64_t y = (j / d.NX) % d.NY;
        const int64_t z = j / (d.NX * d.NY);
        const int64_t ix = x - d.nb, iz = z - d.nb, iy = (d.ndim == 3) ? y - d.nb : 0;
        const bool inside = ix >= 0 && ix < d.nx && iy >= 0 && iy < d.ny && iz >= 0 && iz < d.nz;
        const int64_t e = (clampi(iz, 0, d.nz - 1) * d.ny + clampi(iy, 0, d.ny - 1)) * d.nx + clampi(ix, 0, d.nx - 1);
        const float ve = v_int[e];
        if (inside) {
            v_pad[j] = ve;
        } else if ((o.flags & kBandFreeSurface) && iz < 0) {
            v_pad[j] = 0.f;
        } else {
            const float f = rbc_factor(seed, (uint64_t)j);
            float v = __fmul_rn(f, ve);
            if (o.flags & kBandTaper) v = __fmul_rn(o.c[cell_depth(d, ix, iy, iz) - 1], v);
            v_pad[j] = fminf(v, cap);
        }
    }
}

// Gather form of the padding adjoint: each interior cell collects its own
// gradient and (c_i) f_j times the gradient of every uncapped band cell j
// whose clamped coordinates are this cell (free-surface cells are constant).
// An interior cell has one such term, one on a face nb + 1, on an edge (nb +
// 1)^2, at a corner (2-D: (nb + 1)^2, 3-D: (nb + 1)^3): a thread that walked a
// corner by itself, one gather and one factor after the other, set the whole
// launch's time (401 .. 1201 x 300 cells, nb 40: 371 us; now 27).  A thread
// still walks its own cell, four gathers ahead, but cells of many terms that
// stand alone in their wavefront, or of very many, are shared by its lanes:
// partial sums over every 64th term, added up in a fixed order.
struct AdjCell {
    float ve;
    int64_t x0, y0, z0, cx, cy, cz;  // first padded cell of the box; the cell itself
    int mx, my;                      // box extents
    int m;                           // cells in the box
};

__device__ __forceinline__ AdjCell adj_cell(const PadDims &d, const float *__restrict__ v_int, int64_t i)
{
    AdjCell c;
    const int64_t ix = i % d.nx;
    const int64_t iy = (i / d.nx) % d.ny;
    const int64_t iz = i / (d.nx * d.ny);
    c.ve = v_int[i];
    c.cx = ix + d.nb;
    c.cz = iz + d.nb;
    c.cy = d.ndim == 3 ? iy + d.nb : 0;
    // Padded coordinate ranges that clamp onto (iz, iy, ix).
    c.x0 = ix == 0 ? 0 : c.cx;
    c.z0 = iz == 0 ? 0 : c.cz;
    c.y0 = iy == 0 ? 0 : c.cy;
    c.mx = (int)((ix == d.nx - 1 ? d.NX - 1 : c.cx) - c.x0) + 1;
    c.my = (int)((iy == d.ny - 1 ? d.NY - 1 : c.cy) - c.y0) + 1;
    c.m = c.mx * c.my * ((int)((iz == d.nz - 1 ? d.NZ - 1 : c.cz) - c.z0) + 1);
    return c;
}

// Adds terms beg, beg + step, ... of a cell, in that order.  LINE: the box is
// one cell wide along all axes but one, so that a term's cell takes no
// division (the 2-D case above: 27 us, 40 without).
template <bool LINE>
__device__ __forceinline__ float adj_sum(const PadDims &d, const AdjCell &c, uint64_t seed, float cap,
                                         const BandOpts &o, const float *__restrict__ g_pad, int beg, int step)
{
    constexpr int U = 4;
    const int lx = c.mx > 1, ly = !lx && c.my > 1, lz = !lx && !ly;
    auto cell = [&](int t, int64_t &x, int64_t &y, int64_t &z) {
        if (LINE) {
            x = c.x0 + (lx ? t : 0);
            y = c.y0 + (ly ? t : 0);
            z = c.z0 + (lz ? t : 0);
        } else {
            const int yz = t / c.mx, zz = yz / c.my;
            x = c.x0 + (t - yz * c.mx);
            y = c.y0 + (yz - zz * c.my);
            z = c.z0 + zz;
        }
    };
    float acc = 0.f;
    for (int t0 = beg; t0 < c.m; t0 += U * step) {
        float g[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int64_t x, y, z;
            cell(min(t0 + u * step, c.m - 1), x, y, z);
            g[u] = g_pad[(z * d.NY + y) * d.NX + x];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = t0 + u * step;
            if (t >= c.m) break;
            int64_t x, y, z;
            cell(t, x, y, z);
            if (z == c.cz && y == c.cy && x == c.cx) {
                acc += g[u];
            } else if (!((o.flags & kBandFreeSurface) && z < d.nb)) {
                float f = rbc_factor(seed, (uint64_t)((z * d.NY + y) * d.NX + x));
                float v = __fmul_rn(f, c.ve);
                if (o.flags & kBandTaper) {
                    const float k = o.c[cell_depth(d, x - d.nb, (d.ndim == 3) ? y - d.nb : 0, z - d.nb) - 1];
                    v = __fmul_rn(k, v);
                    f = __fmul_rn(k, f);
                }
                if (v < cap) acc = fmaf(f, g[u], acc);
            }
        }
    }
    return acc;
}

constexpr int kAdjLong = 16, kAdjShare = 1024;  // terms; a wavefront with at most 8 long cells shares them too

__global__ __launch_bounds__(kBlock) void pad_adjoint_kernel(PadDims d, const float *__restrict__ v_int, uint64_t seed,
                                                             float v_cap, const unsigned *__restrict__ cap_bits,
                                                             BandOpts o, const float *__restrict__ g_pad,
                                                             float *__restrict__ g_int)
{
    const float cap = cap_bits ? __uint_as_float(*cap_bits) : v_cap;
    const int64_t n = d.nx * d.ny * d.nz;
    const int lane = threadIdx.x & 63;
    // whole wavefronts: lanes past the end hold no cell but help with the shared ones
    for (int64_t i = gid(); i - lane < n; i += gstride()) {
        const bool in = i < n;
        AdjCell c = adj_cell(d, v_int, min(i, n - 1));
        if (!in) c.m = 0;
        const bool few = __popcll(__ballot(c.m >= kAdjLong)) <= 8;
        const bool share = c.m >= kAdjShare || (few && c.m >= kAdjLong);
        if (in && !share) {
            const int mz = c.m / (c.mx * c.my);
            if (__all((c.mx > 1) + (c.my > 1) + (mz > 1) <= 1)) g_int[i] = adj_sum<true>(d, c, seed, cap, o, g_pad, 0, 1);
            else g_int[i] = adj_sum<false>(d, c, seed, cap, o, g_pad, 0, 1);
        }
        for (uint64_t todo = __ballot(share); todo != 0; todo &= todo - 1) {
            const int64_t j = i - lane + (__ffsll((unsigned long long)todo) - 1);
            float s = adj_sum<false>(d, adj_cell(d, v_int, j), seed, cap, o, g_pad, lane, 64);
            for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
            if (lane == 0) g_int[j] = s;
        }
    }
}

__global__ void fill_kernel(float *__restrict__ p, int64_t n, float v)
{
    for (int64_t i = gid(); i < n; i += gstride()) p[i] = v;
}

typedef float fill4 __attribute__((ext_vector_type(4)));

// Zeros n 16-byte units; NT: past the caches.
template <bool NT>
__global__ __launch_bounds__(kBlock) void zero_kernel(fill4 *__restrict__ p, int64_t n)
{
    const fill4 z = {0.f, 0.f, 0.f, 0.f};
    for (int64_t i = gid(); i < n; i += gstride()) {
        if (NT) __builtin_nontemporal_store(z, p + i);
        else p[i] = z;
    }
}

// D'[cell] = (v dt / h)^2 on the padded grid, zero in the halo.
__global__ __launch_bounds__(kBlock) void build_dp_kernel(Layout L, const float *__restrict__ v_pad, float dt_over_h,
                                                          float *__restrict__ Dp)
{
    const unsigned py = (unsigned)(L.plane / L.pitch), rows = (unsigned)(L.total / L.pitch);
    chunks_do(rows, (unsigned)L.pitch, [&](unsigned row, unsigned x0) {
        const int zz = (int)(row / py) - kRadius, yy = L.ndim == 3 ? (int)(row % py) - kRadius : 0;
        const bool in = zz >= 0 && zz < L.NZ && yy >= 0 && yy < L.NY;
        const float *v = v_pad + ((int64_t)min(max(zz, 0), L.NZ - 1) * L.NY + min(max(yy, 0), L.NY - 1)) * L.NX;
        float c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = in ? v[min(max((int)(x0 + 64 * u) - kXOff, 0), L.NX - 1)] * dt_over_h : 0.f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int x = (int)(x0 + 64 * u), xx = x - kXOff;
            if (x < L.pitch) Dp[(int64_t)row * L.pitch + x] = xx >= 0 && xx < L.NX ? c[u] * c[u] : 0.f;
        }
    });
}

// Dense [NZ][NY][NX] copy of a halo-layout field.
__global__ void unpack_kernel(Layout L, const float *__restrict__ f, float *__restrict__ out)
{
    const int64_t n = (int64_t)L.NX * L.NY * L.NZ;
    for (int64_t j = gid(); j < n; j += gstride()) {
        const int64_t x = j % L.NX;
        const int64_t y = (j / L.NX) % L.NY;
        const int64_t z = j / ((int64_t)L.NX * L.NY);
        out[j] = f[L.org + z * L.plane + y * L.pitch + x];
    }
}

// Traces of every shot between the caller's [nrec][nt1] and the [nt1][nrec]
// that the passes read (IN) or write, through a 32 x 33 LDS tile; blockIdx.x:
// 32 receivers, y: 32 samples, z: shot.
template <bool IN>
__global__ __launch_bounds__(256) void traces_kernel(const ShotDev *__restrict__ shots, int nsh, int64_t nt1)
{
    __shared__ float tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8 threads
    const int64_t r0 = (int64_t)blockIdx.x * 32;
    for (int s = blockIdx.z; s < nsh; s += gridDim.z) {
        const int64_t R = shots[s].nrec;
        if (r0 >= R) continue;
        // in: R x nt1 -> nt1 x R; out: nt1 x R -> R x nt1
        const float *from = IN ? shots[s].traces_in : shots[s].rec_out;
        float *to = IN ? const_cast<float *>(shots[s].sig) : shots[s].traces_out;
        for (int64_t t0 = (int64_t)blockIdx.y * 32; t0 < nt1; t0 += (int64_t)gridDim.y * 32) {
            for (int i = ty; i < 32; i += 8) {
                const int64_t r = r0 + (IN ? i : tx), t = t0 + (IN ? tx : i);
                if (r < R && t < nt1) tile[i][tx] = from[IN ? r * nt1 + t : t * R + r];
            }
            __syncthreads();
            for (int i = ty; i < 32; i += 8) {
                const int64_t r = r0 + (IN ? tx : i), t = t0 + (IN ? i : tx);
                if (r < R && t < nt1) to[IN ? t * R + r : r * nt1 + t] = tile[tx][i];
            }
            __syncthreads();
        }
    }
}

// mu^N = D' (R^T g^N): one thread per receiver injection node, any shot.
__global__ void inj_set_kernel(const ShotDev *__restrict__ shots, const InjEnt *__restrict__ ents, int ebeg, int eend,
                               const Contrib *__restrict__ cont, int step)
{
    const int e = ebeg + (int)gid();
    if (e >= eend) return;
    const InjEnt E = ents[e];
    const ShotDev &S = shots[E.shot];
    const float *sig = S.sig + (int64_t)step * S.nrec;
    float s = 0.f;
    for (int c = E.cbeg; c < E.cend; ++c) s = fmaf(cont[c].w, sig[cont[c].idx], s);
    const int64_t off = S.L.org + (int64_t)E.z * S.L.plane + (int64_t)E.y * S.L.pitch + E.x;
    float *mu = S.fld[2 + (step & 1)];
    mu[off] = S.Dp[off] * s;
}

// d^n = R p^n for all receivers of every shot (used for the last sample).
__global__ void sample_kernel(const ShotDev *__restrict__ shots, const SampleTask *__restrict__ stasks, int n,
                              int slot)
{
    const SampleTask task = stasks[blockIdx.x];
    const ShotDev &S = shots[task.shot];
    const int r = task.r0 + (int)threadIdx.x;
    if (r >= S.nrec) return;
    const float *p = S.fld[slot] + S.L.org;
    float s = 0.f;
    for (int q = 0; q < kMaxNodes; ++q) s = fmaf(S.rw[r * kMaxNodes + q], p[S.rnode[r * kMaxNodes + q]], s);
    S.rec_out[(int64_t)n * S.nrec + r] = s;
}

// Index of interior row `row` (z ny + y) of a shot, x = 0.
__device__ __forceinline__ int64_t interior_row(const ShotDev &S, unsigned row)
{
    const unsigned ny = (unsigned)(S.iy1 - S.iy0), z = row / ny;
    return S.L.org + (int64_t)(z + S.iz0) * S.L.plane + (int64_t)(row - z * ny + S.iy0) * S.L.pitch + S.ix0;
}

__device__ __forceinline__ unsigned interior_rows(const ShotDev &S)
{
    return (unsigned)(S.iy1 - S.iy0) * (unsigned)(S.iz1 - S.iz0);
}

// max of den over the interior box of each shot, as float bits (den >= 0), to
// out[shot]; blockIdx.y: shot.
__global__ __launch_bounds__(kBlock) void den_max_kernel(const ShotDev *__restrict__ shots, int nsh,
                                                         unsigned *__restrict__ out)
{
    for (int s = blockIdx.y; s < nsh; s += gridDim.y) {
        const ShotDev &S = shots[s];
        const unsigned nx = (unsigned)(S.ix1 - S.ix0);
        unsigned m = 0u;
        chunks_do(interior_rows(S), nx, [&](unsigned row, unsigned x0) {
            const float *b = S.acc1 + interior_row(S, row);
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = b[min(x0 + 64 * u, nx - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) m = max(m, __float_as_uint(fmaxf(v[u], 0.f)));
        });
        block_reduce_atomic<true>(m, out + s);
        __syncthreads();
    }
}

// image = num / (den + eps max(den)) on the interior crop (Eq. (3)) of shots
// [first, first + count), which share the image buffer and its extents: the
// shots' values are added (accumulate) or replace each other in their order.
__global__ __launch_bounds__(kBlock) void image_kernel(const ShotDev *__restrict__ shots, int first, int count,
                                                       const unsigned *__restrict__ dmax_bits, float eps_rel,
                                                       float *__restrict__ image, int accumulate,
                                                       float *__restrict__ num_out, float *__restrict__ den_out)
{
    const ShotDev &F = shots[first];
    const unsigned nx = (unsigned)(F.ix1 - F.ix0);
    chunks_do(interior_rows(F), nx, [&](unsigned row, unsigned x0) {
        const int64_t o = (int64_t)row * nx;
        float v[4] = {};
        if (image && accumulate)
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = image[o + min(x0 + 64 * u, nx - 1)];
        for (int s = accumulate ? 0 : count - 1; s < count; ++s) {
#pragma clang fp contract(off)
            const ShotDev &S = shots[first + s];
            const float stab = eps_rel * __uint_as_float(dmax_bits[first + s]);
            const int64_t r = interior_row(S, row);
            float a[4], b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a[u] = S.acc0[r + min(x0 + 64 * u, nx - 1)];
                b[u] = S.acc1[r + min(x0 + 64 * u, nx - 1)];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float w = a[u] / (b[u] + stab);
                v[u] = accumulate ? v[u] + w : w;
                if (x0 + 64 * u < nx) {
                    if (num_out) num_out[o + x0 + 64 * u] = a[u];
                    if (den_out) den_out[o + x0 + 64 * u] = b[u];
                }
            }
        }
        if (image)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (x0 + 64 * u < nx) image[o + x0 + 64 * u] = v[u];
    });
}

// Dense interior copy of p^m (field fld[lev] of the shot table) for the
// migration with a stored source wavefield: out[(z ny + y) nx + x] = p at
// interior cell (x, y, z).
__global__ __launch_bounds__(kBlock) void snap_store_kernel(const ShotDev *__restrict__ shots, int shot, int lev,
                                                            float *__restrict__ out)
{
    const ShotDev &S = shots[shot];
    const float *f = S.fld[lev];
    const unsigned nx = (unsigned)(S.ix1 - S.ix0);
    chunks_do(interior_rows(S), nx, [&](unsigned row, unsigned x0) {
        const int64_t r = interior_row(S, row);
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = f[r + min(x0 + 64 * u, nx - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (x0 + 64 * u < nx) __builtin_nontemporal_store(v[u], out + (int64_t)row * nx + x0 + 64 * u);
    });
}

// flag |= 1 if any of x[0 .. n) is NaN or infinite (one atomic per block).
__global__ __launch_bounds__(kBlock) void nonfinite_kernel(const float *__restrict__ x, int64_t n,
                                                           unsigned *__restrict__ flag)
{
    unsigned m = 0u;
    for (int64_t i = gid(); i < n; i += gstride()) m = max(m, __float_as_uint(x[i]) & 0x7fffffffu);
    block_reduce_atomic<true>(m >= 0x7f800000u ? 1u : 0u, flag);
}

// grad_v = 2 G / (v^3 dt^2) on the dense padded grid.
__global__ void grad_kernel(const ShotDev *__restrict__ shots, int shot, const float *__restrict__ v_pad, float dt,
                            float *__restrict__ grad)
{
    const ShotDev &S = shots[shot];
    const Layout L = S.L;
    const int64_t n = (int64_t)L.NX * L.NY * L.NZ;
    const float two_over_dt2 = 2.0f / (dt * dt);
    for (int64_t j = gid(); j < n; j += gstride()) {
        const int64_t x = j % L.NX, y = (j / L.NX) % L.NY, z = j / ((int64_t)L.NX * L.NY);
        const float G = S.acc0[L.org + z * L.plane + y * L.pitch + x];
        const float v = v_pad[j];
        grad[j] = v > 0.f ? two_over_dt2 * G / (v * v * v) : 0.f;  // dJ/dv = 2 v dt^2 dJ/dD
    }
}

// dJ/dw^n = h^-2 sum over source nodes of the recorded coefficient * mu^{n+1}.
__global__ void wadj_kernel(const float *__restrict__ parts, int nt, float scale, float *__restrict__ out)
{
    const int n = (int)gid();
    if (n >= nt) return;
    float s = 0.f;
    for (int q = 0; q < kMaxNodes; ++q) s += parts[(int64_t)n * kMaxNodes + q];
    out[n] = s * scale;
}

// Columns [x0, x0 + w) of a [nz][nxg] array into (mode 0) or added from
// (mode 1) a dense [nz][w] window.
__global__ void window_kernel(float *__restrict__ global, const float *__restrict__ win_in,
                              float *__restrict__ win_out, int64_t nz, int64_t nxg, int64_t x0, int64_t w, int mode)
{
    const int64_t n = nz * w;
    for (int64_t i = gid(); i < n; i += gstride()) {
        const int64_t z = i / w, x = i % w;
        const int64_t g = z * nxg + x0 + x;
        if (mode == 0) win_out[i] = global[g];
        else global[g] += win_in[i];
    }
}

// Residual r = d - d_obs and per-block partial sums of r^2 (fixed order
// within a block); a second single-block pass adds the partials in order,
// so J = 0.5 sum r^2 is deterministic.
constexpr int kMisfitBlocks = 1024;

__global__ __launch_bounds__(kBlock) void misfit_partial_kernel(const float *__restrict__ d,
                                                                const float *__restrict__ dobs,
                                                                float *__restrict__ r, int64_t n,
                                                                double *__restrict__ part)
{
    __shared__ double sh[kBlock];
    double acc = 0.0;
    for (int64_t i = gid(); i < n; i += gstride()) {
        const float v = d[i] - dobs[i];
        if (r) r[i] = v;
        acc += (double)v * (double)v;
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(kBlock) void misfit_final_kernel(const double *__restrict__ part, int nparts,
                                                              double *__restrict__ out)
{
    __shared__ double sh[kBlock];
    double acc = 0.0;
    for (int i = threadIdx.x; i < nparts; i += kBlock) acc += part[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = 0.5 * sh[0];
}

}  // namespace

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------

static PadDims pad_dims(int ndim, int nb, int64_t nx, int64_t ny, int64_t nz)
{
    PadDims d;
    d.ndim = ndim;
    d.nb = nb;
    d.nx = nx;
    d.ny = (ndim == 3) ? ny : 1;
    d.nz = nz;
    d.NX = nx + 2 * nb;
    d.NZ = nz + 2 * nb;
    d.NY = (ndim == 3) ? ny + 2 * nb : 1;
    return d;
}

// Streaming copy of n 16-byte units: the bandwidth reference of the
// measurements (a plain read-once, write-once kernel of known size).  Each
// thread keeps kCopyUnroll independent 16-byte loads in flight; a block's
// loads of one round are contiguous (kBlock x 16 B per unrolled slot), and
// blocks stride over the buffer in whole rounds.
constexpr int kCopyUnroll = 4;
typedef float copy4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kBlock) void stream_copy_kernel(const copy4 *__restrict__ src,
                                                             copy4 *__restrict__ dst, int64_t n)
{
    const int64_t round = (int64_t)kBlock * kCopyUnroll;
    for (int64_t base = (int64_t)blockIdx.x * round; base < n; base += (int64_t)gridDim.x * round) {
        copy4 v[kCopyUnroll];
#pragma unroll
        for (int u = 0; u < kCopyUnroll; ++u) {
            const int64_t i = base + (int64_t)u * kBlock + threadIdx.x;
            if (i < n) v[u] = __builtin_nontemporal_load(src + i);
        }
#pragma unroll
        for (int u = 0; u < kCopyUnroll; ++u) {
            const int64_t i = base + (int64_t)u * kBlock + threadIdx.x;
            if (i < n) __builtin_nontemporal_store(v[u], dst + i);
        }
    }
}

hipError_t launch_vrange(const float *v, int64_t n, unsigned *maxmin2, hipStream_t st)
{
    hipLaunchKernelGGL(set_u32_kernel, dim3(1), dim3(64), 0, st, maxmin2, 2, 0u, 0xffffffffu);
    hipLaunchKernelGGL((vrange_kernel<true>), dim3(grid_reduce(n)), dim3(kBlock), 0, st, v, n, maxmin2);
    return hipGetLastError();
}

hipError_t launch_stream_copy(const void *src, void *dst, int64_t units, int blocks_per_cu, hipStream_t st)
{
    if (units <= 0) return hipSuccess;
    const int64_t round = (int64_t)kBlock * kCopyUnroll;
    int64_t b = (units + round - 1) / round;
    const int64_t cap = (int64_t)256 * blocks_per_cu;
    if (b > cap) b = cap;
    hipLaunchKernelGGL(stream_copy_kernel, dim3((unsigned)b), dim3(kBlock), 0, st, (const copy4 *)src, (copy4 *)dst,
                       units);
    return hipGetLastError();
}

hipError_t launch_vmax(const float *v, int64_t n, unsigned *out, hipStream_t st)
{
    hipLaunchKernelGGL(set_u32_kernel, dim3(1), dim3(64), 0, st, out, 1, 0u, 0u);
    hipLaunchKernelGGL((vrange_kernel<false>), dim3(grid_reduce(n)), dim3(kBlock), 0, st, v, n, out);
    return hipGetLastError();
}

hipError_t launch_rbc_pad(int ndim, int nb, int64_t nx, int64_t ny, int64_t nz, const float *v_int, uint64_t seed,
                          float v_cap, const unsigned *cap_bits, const BandOpts &o, float *v_pad, hipStream_t st)
{
    PadDims d = pad_dims(ndim, nb, nx, ny, nz);
    hipLaunchKernelGGL(rbc_pad_kernel, dim3(grid_for(d.NX * d.NY * d.NZ)), dim3(kBlock), 0, st, d, v_int, seed,
                       v_cap, cap_bits, o, v_pad);
    return hipGetLastError();
}

hipError_t launch_pad_adjoint(int ndim, int nb, int64_t nx, int64_t ny, int64_t nz, const float *v_int,
                              uint64_t seed, float v_cap, const unsigned *cap_bits, const BandOpts &o,
                              const float *g_pad, float *g_int, hipStream_t st)
{
    PadDims d = pad_dims(ndim, nb, nx, ny, nz);
    hipLaunchKernelGGL(pad_adjoint_kernel, dim3(grid_for(d.nx * d.ny * d.nz)), dim3(kBlock), 0, st, d, v_int, seed,
                       v_cap, cap_bits, o, g_pad, g_int);
    return hipGetLastError();
}

hipError_t launch_fill(float *p, int64_t n, float v, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n)), dim3(kBlock), 0, st, p, n, v);
    return hipGetLastError();
}

// Zeros `bytes` (a multiple of 16) from a 16-byte-aligned address; beyond the
// memory-side cache, past the caches.
hipError_t launch_zero(void *p, size_t bytes, hipStream_t st)
{
    const int64_t n = (int64_t)(bytes / 16);
    if (n <= 0) return hipSuccess;
    if (bytes > ((size_t)256 << 20))
        hipLaunchKernelGGL((zero_kernel<true>), dim3(grid_for(n)), dim3(kBlock), 0, st, (fill4 *)p, n);
    else
        hipLaunchKernelGGL((zero_kernel<false>), dim3(grid_for(n)), dim3(kBlock), 0, st, (fill4 *)p, n);
    return hipGetLastError();
}

hipError_t launch_build_dp(const Layout &L, const float *v_pad, float dt_over_h, float *Dp, hipStream_t st)
{
    hipLaunchKernelGGL(build_dp_kernel, dim3(grid_chunks(L.total / L.pitch, L.pitch)), dim3(kBlock), 0, st, L, v_pad, dt_over_h, Dp);
    return hipGetLastError();
}

hipError_t launch_unpack(const Layout &L, const float *f, float *out, hipStream_t st)
{
    hipLaunchKernelGGL(unpack_kernel, dim3(grid_for((int64_t)L.NX * L.NY * L.NZ)), dim3(kBlock), 0, st, L, f, out);
    return hipGetLastError();
}

// Traces of every shot into (in) or out of the workspace.
hipError_t launch_traces(const ShotDev *shots, int nsh, int maxrec, int64_t nt1, bool in, hipStream_t st)
{
    const dim3 grid((unsigned)((maxrec + 31) / 32), (unsigned)std::min<int64_t>((nt1 + 31) / 32, 65535),
                    (unsigned)std::min(nsh, 65535));
    if (in)
        hipLaunchKernelGGL((traces_kernel<true>), grid, dim3(256), 0, st, shots, nsh, nt1);
    else
        hipLaunchKernelGGL((traces_kernel<false>), grid, dim3(256), 0, st, shots, nsh, nt1);
    return hipGetLastError();
}

hipError_t launch_inj_set(const ShotDev *shots, const InjEnt *ents, int ebeg, int eend, const Contrib *cont, int step,
                          hipStream_t st)
{
    int n = eend - ebeg;
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(inj_set_kernel, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, st, shots, ents, ebeg, eend,
                       cont, step);
    return hipGetLastError();
}

hipError_t launch_sample(const ShotDev *shots, const SampleTask *stasks, int ntask, int n, int slot, hipStream_t st)
{
    if (ntask <= 0) return hipSuccess;
    hipLaunchKernelGGL(sample_kernel, dim3(ntask), dim3(64), 0, st, shots, stasks, n, slot);
    return hipGetLastError();
}

// max(den) of every shot to dmax_bits[shot].
hipError_t launch_den_max(const ShotDev *shots, int nsh, int64_t rows, int64_t len, unsigned *dmax_bits, hipStream_t st)
{
    hipLaunchKernelGGL(set_u32_kernel, dim3((nsh + kBlock - 1) / kBlock), dim3(kBlock), 0, st, dmax_bits, nsh, 0u, 0u);
    // one atomic per block: at most 512 of them on a shot's word
    const unsigned bx = std::min(grid_chunks((rows + 3) / 4, len), 512u);
    hipLaunchKernelGGL(den_max_kernel, dim3(bx, (unsigned)std::min(nsh, 65535)), dim3(kBlock), 0, st, shots, nsh,
                       dmax_bits);
    return hipGetLastError();
}

hipError_t launch_image(const ShotDev *shots, int first, int count, int64_t rows, int64_t len,
                        const unsigned *dmax_bits, float eps_rel, float *image, int accumulate, float *num, float *den,
                        hipStream_t st)
{
    hipLaunchKernelGGL(image_kernel, dim3(grid_chunks(rows, len)), dim3(kBlock), 0, st, shots, first, count, dmax_bits,
                       eps_rel, image, accumulate, num, den);
    return hipGetLastError();
}

hipError_t launch_snap_store(const ShotDev *shots, int shot, int lev, int64_t ninterior, float *out, hipStream_t st)
{
    // blocks of four chunks; the kernel strides over what is left
    hipLaunchKernelGGL(snap_store_kernel, dim3(grid_chunks((ninterior + kChunk - 1) / kChunk, kChunk)), dim3(kBlock), 0,
                       st, shots, shot, lev, out);
    return hipGetLastError();
}

hipError_t launch_nonfinite(const float *x, int64_t n, unsigned *flag, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(nonfinite_kernel, dim3(grid_reduce(n)), dim3(kBlock), 0, st, x, n, flag);
    return hipGetLastError();
}

hipError_t launch_grad(const ShotDev *shots, int shot, int64_t npad, const float *v_pad, float dt, float *grad,
                       hipStream_t st)
{
    hipLaunchKernelGGL(grad_kernel, dim3(grid_for(npad)), dim3(kBlock), 0, st, shots, shot, v_pad, dt, grad);
    return hipGetLastError();
}

hipError_t launch_window(float *global, const float *win_in, float *win_out, int64_t nz, int64_t nxg, int64_t x0,
                         int64_t w, int mode, hipStream_t st)
{
    hipLaunchKernelGGL(window_kernel, dim3(grid_for(nz * w)), dim3(kBlock), 0, st, global, win_in, win_out, nz, nxg, x0,
                       w, mode);
    return hipGetLastError();
}

size_t misfit_ws_bytes() { return sizeof(double) * (kMisfitBlocks + 1); }

hipError_t launch_misfit(const float *d, const float *dobs, float *r, int64_t n, void *ws, double *J, hipStream_t st)
{
    double *part = (double *)ws;
    const unsigned nb = std::min<int64_t>(kMisfitBlocks, std::max<int64_t>(1, (n + kBlock - 1) / kBlock));
    hipLaunchKernelGGL(misfit_partial_kernel, dim3(nb), dim3(kBlock), 0, st, d, dobs, r, n, part);
    hipLaunchKernelGGL(misfit_final_kernel, dim3(1), dim3(kBlock), 0, st, (const double *)part, (int)nb, J);
    return hipGetLastError();
}

hipError_t launch_wadj(const float *parts, int nt, float scale, float *out, hipStream_t st)
{
    hipLaunchKernelGGL(wadj_kernel, dim3((nt + kBlock - 1) / kBlock), dim3(kBlock), 0, st, parts, nt, scale, out);
    return hipGetLastError();
}

}  // namespace rtm
