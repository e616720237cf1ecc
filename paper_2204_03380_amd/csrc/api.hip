// Host runtime of librtm: argument validation, acquisition tables,
// workspace carving and the launch sequences behind the C ABI of
// include/rtm.h.  Every device buffer comes from the caller.
#include <algorithm>
#include <array>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <tuple>
#include <vector>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "common.h"
#include "rtm.h"

namespace rtm {
// prop2d.hip (one step per launch, persistent passes)
hipError_t launch_fwd2d(int vec, int tx, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                        const InjEnt *ents, const Contrib *cont, const SampleTask *stasks, int nsample, int n,
                        hipStream_t st);
hipError_t launch_rev2d(int vec, int tx, bool grad, const ShotDev *shots, const Tile2D *tiles, int ntiles,
                        int nslots, const InjEnt *ents, const Contrib *cont, int k, int reinject, float *wadj,
                        hipStream_t st);
// prop2d_multi.hip
hipError_t launch_fwd2d_t2(int vec, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                           const InjEnt *ents, const Contrib *cont, const SampleTask *stasks, int nsample, int n,
                           hipStream_t st);
hipError_t launch_rev2d_t2(int vec, bool grad, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                           const InjEnt *ents, const Contrib *cont, int k, int reinject, float *wadj, hipStream_t st);
hipError_t launch_fwd2d_t3(int vec, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                           const InjEnt *ents, const Contrib *cont, const SampleTask *stasks, int nsample, int n,
                           hipStream_t st);
hipError_t launch_rev2d_t3(int vec, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                           const InjEnt *ents, const Contrib *cont, int k, int reinject, hipStream_t st);
hipError_t launch_rev2d_t3_grad(int vec, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                                const InjEnt *ents, const Contrib *cont, int k, int reinject, float *wadj,
                                hipStream_t st);
// prop2d.hip
hipError_t launch_fwd2d_persist(int vec, const ShotDev *shots, const Tile2D *tiles, const PItem *items, int nitems,
                                const int *shot_items, const InjEnt *ents, const Contrib *cont,
                                const SampleTask *stasks, int n0, int nsteps, unsigned *cnt, unsigned *status,
                                double wait_ms, hipStream_t st);
hipError_t launch_rev2d_persist(int vec, bool grad, const ShotDev *shots, const Tile2D *tiles, const PItem *items,
                                int nitems, const int *shot_items, const InjEnt *ents, const Contrib *cont, int k0,
                                int nsteps, int reinject, float *wadj, unsigned *cnt, unsigned *status,
                                double wait_ms, hipStream_t st);
hipError_t launch_recv2d(int vec, int tx, const ShotDev *shots, const Tile2D *tiles, int ntiles, int nslots,
                         const InjEnt *ents, const Contrib *cont, int k, const float *snap, hipStream_t st);
// prop3d.hip
hipError_t launch_fwd3d(int vec, int ty, const ShotDev *shots, const Tile3D *tiles, int ntiles, int nslots,
                        const InjEnt *ents, const Contrib *cont, const SampleTask *stasks, int nsample, int n,
                        hipStream_t st);
hipError_t launch_rev3d(int vec, int ty, bool grad, const ShotDev *shots, const Tile3D *tiles, int ntiles, int nslots,
                        const InjEnt *ents, const Contrib *cont, int k, int reinject, float *wadj, hipStream_t st);
hipError_t launch_recv3d(int vec, int ty, const ShotDev *shots, const Tile3D *tiles, int ntiles, int nslots,
                         const InjEnt *ents, const Contrib *cont, int k, const float *snap, hipStream_t st);
// aux.hip
hipError_t launch_vrange(const float *v, int64_t n, unsigned *maxmin2, hipStream_t st);
hipError_t launch_vmax(const float *v, int64_t n, unsigned *out, hipStream_t st);
hipError_t launch_stream_copy(const void *src, void *dst, int64_t units, int blocks_per_cu, hipStream_t st);
hipError_t launch_rbc_pad(int ndim, int nb, int64_t nx, int64_t ny, int64_t nz, const float *v_int, uint64_t seed,
                          float v_cap, const unsigned *cap_bits, const BandOpts &o, float *v_pad, hipStream_t st);
hipError_t launch_pad_adjoint(int ndim, int nb, int64_t nx, int64_t ny, int64_t nz, const float *v_int,
                              uint64_t seed, float v_cap, const unsigned *cap_bits, const BandOpts &o,
                              const float *g_pad, float *g_int, hipStream_t st);
hipError_t launch_fill(float *p, int64_t n, float v, hipStream_t st);
hipError_t launch_zero(void *p, size_t bytes, hipStream_t st);
hipError_t launch_build_dp(const Layout &L, const float *v_pad, float dt_over_h, float *Dp, hipStream_t st);
hipError_t launch_unpack(const Layout &L, const float *f, float *out, hipStream_t st);
hipError_t launch_traces(const ShotDev *shots, int nsh, int maxrec, int64_t nt1, bool in, hipStream_t st);
hipError_t launch_inj_set(const ShotDev *shots, const InjEnt *ents, int ebeg, int eend, const Contrib *cont, int step,
                          hipStream_t st);
hipError_t launch_sample(const ShotDev *shots, const SampleTask *stasks, int ntask, int n, int slot, hipStream_t st);
hipError_t launch_den_max(const ShotDev *shots, int nsh, int64_t rows, int64_t len, unsigned *dmax_bits, hipStream_t st);
hipError_t launch_image(const ShotDev *shots, int first, int count, int64_t rows, int64_t len,
                        const unsigned *dmax_bits, float eps_rel, float *image, int accumulate, float *num, float *den,
                        hipStream_t st);
hipError_t launch_grad(const ShotDev *shots, int shot, int64_t npad, const float *v_pad, float dt, float *grad,
                       hipStream_t st);
hipError_t launch_snap_store(const ShotDev *shots, int shot, int lev, int64_t ninterior, float *out, hipStream_t st);
hipError_t launch_nonfinite(const float *x, int64_t n, unsigned *flag, hipStream_t st);
hipError_t launch_wadj(const float *parts, int nt, float scale, float *out, hipStream_t st);
size_t misfit_ws_bytes();
hipError_t launch_misfit(const float *d, const float *dobs, float *r, int64_t n, void *ws, double *J, hipStream_t st);
hipError_t launch_window(float *global, const float *win_in, float *win_out, int64_t nz, int64_t nxg, int64_t x0,
                         int64_t w, int mode, hipStream_t st);
}  // namespace rtm

using namespace rtm;

namespace {

// ---------------------------------------------------------------------------
// Errors
// ---------------------------------------------------------------------------

thread_local std::string t_err;

int fail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    t_err = buf;
    return code;
}

}  // namespace

// Error state shared with the other sources of the library.
namespace rtm {
int set_error(int code, const char *msg) { return fail(code, "%s", msg); }
void clear_error() { t_err.clear(); }
}  // namespace rtm

namespace {

#define RTM_HIP(call)                                                                         \
    do {                                                                                      \
        hipError_t e_ = (call);                                                               \
        if (e_ != hipSuccess) return fail(RTM_EHIP, "%s: %s", #call, hipGetErrorString(e_)); \
    } while (0)

// ---------------------------------------------------------------------------
// Tuning: strip width (VEC floats per lane) and rows per tile.
// ---------------------------------------------------------------------------

struct Tune {
    int vec;
    int zseg;
    int ty;  // 3-D: y rows per workgroup
    int tx;  // 2-D: wavefronts (adjacent strips) per workgroup
    int steps = 1;  // 2-D: time steps per launch (1, 2 or 3)
    int zin = 0;    // 3-D: tiles numbered with z innermost (else x innermost)
    int block = 0;  // 2-D multi-step: index of kBlockShapes (0: marching strips)
    int once = 0;   // 3-D, 2-D multi-step: kOnce, or 0
    int code() const { return vec | block << 8 | once; }  // as the multi-step and 3-D launchers take it
};

// 2-D shapes: ((steps - 1) << 28) | (tx << 24) | (vec << 16) | zseg;
// defaults from sweeps over 48 shots of the 2301 x 751 folded grid: three
// steps per launch at vec 2, 108-row tiles (reverse 412 us per step, RTM
// forward 153; two steps at vec 4 took 584 and 212, three at vec 4 545 and
// 201).  Modeling, which takes two steps per launch, then runs at vec 2
// (232 us per step against 213 at vec 4).
std::atomic<int> g_tune2d_fwd{(2 << 28) | (1 << 24) | (2 << 16) | 108};
std::atomic<int> g_tune2d_rev{(2 << 28) | (1 << 24) | (2 << 16) | 108};
std::atomic<int> g_tune_exact{0};  // 1: take the configured shapes as they are
std::atomic<double> g_persist_wait_ms{4000.0};  // bounded wait of persistent passes

// 3-D shapes: (vec << 24) | (ty << 16) | (z_inner << 15) | zseg: the largest
// tiles that fit_tune3 chooses from; defaults from sweeps over 64^3 to 512 x
// 512 x 256 grids (612 x 612 x 356 padded, us per step: forward, 2 floats x
// 16 rows 418, 2 x 8 446, 1 x 8 456; reverse, 1 x 8 1096, 1 x 16 1101, 2 x 8
// 1101, 1 x 4 1108).
std::atomic<int> g_tune3d_fwd{(2 << 24) | (16 << 16) | 126};
std::atomic<int> g_tune3d_rev{(1 << 24) | (8 << 16) | 54};

Tune get_tune(int which, int ndim)
{
    if (ndim == 3) {
        int v = (which == 0 ? g_tune3d_fwd : g_tune3d_rev).load();
        Tune t{v >> 24, v & 0x7fff, (v >> 16) & 0xff, 1};
        t.zin = (v >> 15) & 1;
        return t;
    }
    int v = (which == 0 ? g_tune2d_fwd : g_tune2d_rev).load();
    return Tune{(v >> 16) & 0xff, v & 0xffff, 1, (v >> 24) & 0xf, ((v >> 28) & 0x3) + 1};
}

constexpr int kMinZseg = kZUnroll;

// ---------------------------------------------------------------------------
// Optional event timing of the time loops (measurement only).
// ---------------------------------------------------------------------------

enum LoopKind { kLoopModelFwd = 0, kLoopRtmFwd = 1, kLoopRevImage = 2, kLoopRevGrad = 3, kLoopKinds = 4 };

struct PendingTiming {
    hipEvent_t start, stop;
    int kind;
    int64_t launches;
};

std::atomic<int> g_timing_on{0};
std::mutex g_timing_mu;
std::vector<PendingTiming> g_timing_pending;

// Records an event pair around [begin, end) of a loop on `st`; the pair is
// resolved later by rtm_timing_read, so no host synchronisation is added.
// A roctx range over one pass of a job's launch sequence (host time of the
// enqueues; shown by rocprofv3 --marker-trace, a no-op otherwise).
struct PassRange {
    explicit PassRange(const char *name) { roctxRangePushA(name); }
    ~PassRange() { roctxRangePop(); }
    PassRange(const PassRange &) = delete;
    PassRange &operator=(const PassRange &) = delete;
};

struct LoopTimer {
    hipEvent_t a = nullptr, b = nullptr;
    int kind;
    int64_t launches;
    hipStream_t st;
    LoopTimer(int k, int64_t n, hipStream_t s, bool enable = true) : kind(k), launches(n), st(s)
    {
        if (!enable || !g_timing_on.load()) return;
        if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) {
            a = b = nullptr;
            return;
        }
        (void)hipEventRecord(a, st);
    }
    void finish()
    {
        if (!a) return;
        (void)hipEventRecord(b, st);
        std::lock_guard<std::mutex> lk(g_timing_mu);
        g_timing_pending.push_back(PendingTiming{a, b, kind, launches});
        a = b = nullptr;
    }
    ~LoopTimer()
    {
        // Loop abandoned on an error path: drop its events.
        if (a) (void)hipEventDestroy(a);
        if (b) (void)hipEventDestroy(b);
    }
};

// ---------------------------------------------------------------------------
// Grids and point operators
// ---------------------------------------------------------------------------

struct GridInfo {
    int ndim, nb;
    int64_t nx, ny, nz;
    int NX, NY, NZ;
    double h;
    Layout L;
};

int grid_info(const rtm_grid_t *g, GridInfo *gi)
{
    if (!g) return fail(RTM_EINVAL, "grid is NULL");
    if (g->ndim != 2 && g->ndim != 3) return fail(RTM_EINVAL, "ndim must be 2 or 3 (got %d)", (int)g->ndim);
    if (g->nb < 0) return fail(RTM_EINVAL, "nb must be >= 0");
    int64_t ny = g->ndim == 3 ? g->ny : 1;
    if (g->nx < 1 || g->nz < 1 || ny < 1) return fail(RTM_EINVAL, "interior extents must be >= 1");
    if (!(g->h > 0.0) || !std::isfinite(g->h)) return fail(RTM_EINVAL, "h must be positive and finite");
    int64_t NX = g->nx + 2 * (int64_t)g->nb, NZ = g->nz + 2 * (int64_t)g->nb;
    int64_t NY = g->ndim == 3 ? ny + 2 * (int64_t)g->nb : 1;
    if (NX > (1 << 28) || NY > (1 << 28) || NZ > (1 << 28)) return fail(RTM_EINVAL, "grid too large");
    gi->ndim = g->ndim;
    gi->nb = g->nb;
    gi->nx = g->nx;
    gi->ny = ny;
    gi->nz = g->nz;
    gi->NX = (int)NX;
    gi->NY = (int)NY;
    gi->NZ = (int)NZ;
    gi->h = g->h;
    gi->L = make_layout(g->ndim, (int)NX, (int)NY, (int)NZ);
    if (gi->L.total >= ((int64_t)1 << 31)) return fail(RTM_EINVAL, "field of %lld floats exceeds 2^31", (long long)gi->L.total);
    return RTM_OK;
}

struct PointOp {
    int n;
    int z[kMaxNodes], y[kMaxNodes], x[kMaxNodes];
    double w[kMaxNodes];
};

// Multilinear interpolation nodes (padded coordinates) and weights of an
// interior position; zero weights are dropped.
bool make_point(const GridInfo &g, const float *pos, PointOp *P)
{
    double q[3] = {pos[0], g.ndim == 3 ? pos[1] : 0.0, pos[2]};
    int64_t n[3] = {g.nx, g.ny, g.nz};
    int64_t i0[3];
    double fr[3];
    for (int a = 0; a < 3; ++a) {
        if (!(q[a] >= 0.0 && q[a] <= (double)(n[a] - 1))) return false;
        i0[a] = (int64_t)std::floor(q[a]);
        fr[a] = q[a] - (double)i0[a];
    }
    P->n = 0;
    for (int cz = 0; cz < 2; ++cz)
        for (int cy = 0; cy < 2; ++cy)
            for (int cx = 0; cx < 2; ++cx) {
                double w = (cx ? fr[0] : 1 - fr[0]) * (cy ? fr[1] : 1 - fr[1]) * (cz ? fr[2] : 1 - fr[2]);
                if (w == 0.0) continue;
                P->x[P->n] = (int)(i0[0] + cx + g.nb);
                P->y[P->n] = g.ndim == 3 ? (int)(i0[1] + cy + g.nb) : 0;
                P->z[P->n] = (int)(i0[2] + cz + g.nb);
                P->w[P->n] = w;
                P->n++;
            }
    return true;
}

// ---------------------------------------------------------------------------
// Jobs: one or many shots propagated together.  Every time step is one
// kernel launch covering all tiles of all shots; shots with the same padded
// model and grid share their D' array.
// ---------------------------------------------------------------------------

struct ShotIn {
    GridInfo g;
    const float *v_pad = nullptr;
    const float *wavelet = nullptr;
    float src[3] = {0, 0, 0};
    int nrec = 0;
    std::vector<float> rec;             // [nrec][3]
    const float *traces_in = nullptr;   // RTM data / VJP upstream gradient, [nrec][nt + 1]
    float *traces_out = nullptr;        // modeling output, [nrec][nt + 1]
    float *image = nullptr, *num = nullptr, *den = nullptr;  // RTM outputs (interior)
    float *grad_v_pad = nullptr, *grad_wavelet = nullptr;    // VJP outputs
    float *p_last = nullptr, *p_prev = nullptr;              // modeling: final panels
    float *snaps = nullptr;             // storage RTM: stored interior levels
    int stride = 1, phase = 0;          // storage RTM: levels k = phase (mod stride)
};

// Tiles and injection entries of one launch shape.  ents holds all source
// entries of all shots, then all receiver entries (when present).
struct Tiling {
    Tune tune{1, 18, 1, 1, 1};
    int ndim = 2;
    int steps = 1;  // 2-D: time steps per launch of the tiles (> 1: overlapping strips)
    std::vector<Tile2D> tiles;   // 2-D jobs
    std::vector<Tile3D> tiles3;  // 3-D jobs
    std::vector<InjEnt> ents;
    std::vector<Contrib> cont;
    int nsrc_ent = 0, nrec_ent = 0, nslots = 0;
    int count() const { return ndim == 3 ? (int)tiles3.size() : (int)tiles.size(); }
};

struct Counts {
    int64_t tiles_f = 0, ents_f = 0, cont_f = 0;  // forward tiling
    int64_t tiles_r = 0, ents_r = 0, cont_r = 0;  // reverse tiling
    int64_t tiles_f2 = 0, ents_f2 = 0, cont_f2 = 0;  // multi-step tilings (2-D)
    int64_t tiles_r2 = 0, ents_r2 = 0, cont_r2 = 0;
    int64_t stasks = 0, rnode = 0;
    int64_t pitems_f = 0, pitems_r = 0;  // persistent passes: work items
};

// Byte offsets of every device buffer inside the workspace.
struct WsLayout {
    size_t scal = 0, shots = 0, tiles_f = 0, ents_f = 0, cont_f = 0, tiles_r = 0, ents_r = 0, cont_r = 0;
    size_t tiles_f2 = 0, ents_f2 = 0, cont_f2 = 0, tiles_r2 = 0, ents_r2 = 0, cont_r2 = 0;
    size_t stasks = 0, rnode = 0, rw = 0;
    size_t pitems_f = 0, pitems_r = 0, pnum = 0, pcnt = 0;  // persistent passes
    std::vector<size_t> dp;                  // per D' slot
    std::vector<std::array<size_t, 8>> fld;  // per shot
    std::vector<size_t> acc0, acc1, trint, wadj;
    size_t zero_end = 0;  // fields and sums, from the first shot's first field on, end here
    size_t bytes = 0;
};

struct Job {
    int op = RTM_OP_MODEL;
    int nt = 0;
    double dt = 0.0;
    float eps = 1e-3f;
    uint32_t flags = 0;
    std::vector<ShotIn> shots;
    Tiling fw, rv;    // rv unused for modeling
    Tiling fw2, rv2;  // multi-step tilings (2-D, when the shape asks for two or three steps per launch)
    std::vector<SampleTask> stasks;
    std::vector<int> rnode;
    std::vector<float> rw;
    std::vector<int64_t> rbase;      // per shot: offset of its receivers in rnode / rw (in receivers)
    std::vector<std::array<int, 2>> srows;  // per shot: padded rows [lo, hi) holding receiver nodes
    std::vector<int> dslot;          // per shot: D' slot
    std::vector<int> slot_shot;      // per slot: first shot using it
    // persistent passes (RTM_F_PERSISTENT): work items and per-shot item
    // counts of the forward and reverse passes
    std::vector<PItem> pitems_f, pitems_r;
    std::vector<int> pnum;           // [0, nsh): forward, [nsh, 2 nsh): reverse
    WsLayout ws;
    // hipGraph of the launch schedule (plans with RTM_F_GRAPH)
    hipGraphExec_t gexec = nullptr;
    void *g_ws = nullptr;
    hipStream_t g_st = nullptr;
};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Field buffers per shot: p (2 levels) and mu (2 levels); 2-D jobs keep a
// second set for the multi-step kernels, so that the workspace size does not
// depend on the launch shape.  2-D modeling keeps, in the mu slot 2 of each
// set, the middle level that three-step launches store on the receiver rows.
int per_set(int op, int ndim) { return op == RTM_OP_MODEL ? (ndim == 2 ? 3 : 2) : 4; }
int nfields(int op, int ndim) { return per_set(op, ndim) * (ndim == 2 ? 2 : 1); }
int nfields(const Job &J) { return nfields(J.op, J.shots.empty() ? 3 : J.shots[0].g.ndim); }
// Ops with the imaging sums num (acc0) and den (acc1).
bool has_den(int op) { return op == RTM_OP_RTM || op == RTM_OP_STORAGE; }

constexpr size_t kTileBytes = sizeof(Tile2D) > sizeof(Tile3D) ? sizeof(Tile2D) : sizeof(Tile3D);

WsLayout make_ws_layout(const Job &J, const Counts &c)
{
    WsLayout w;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        off = align256(off);
        size_t o = off;
        off += bytes;
        return o;
    };
    const int nsh = (int)J.shots.size();
    const int nslot = (int)J.slot_shot.size();
    w.scal = take(sizeof(unsigned) * (64 + 2 * (size_t)nslot + (size_t)nsh));
    w.shots = take(sizeof(ShotDev) * 2 * nsh);  // two copies: field sets in either order
    w.tiles_f = take(kTileBytes * c.tiles_f);
    w.ents_f = take(sizeof(InjEnt) * c.ents_f);
    w.cont_f = take(sizeof(Contrib) * c.cont_f);
    w.tiles_r = take(kTileBytes * c.tiles_r);
    w.ents_r = take(sizeof(InjEnt) * c.ents_r);
    w.cont_r = take(sizeof(Contrib) * c.cont_r);
    w.tiles_f2 = take(kTileBytes * c.tiles_f2);
    w.ents_f2 = take(sizeof(InjEnt) * c.ents_f2);
    w.cont_f2 = take(sizeof(Contrib) * c.cont_f2);
    w.tiles_r2 = take(kTileBytes * c.tiles_r2);
    w.ents_r2 = take(sizeof(InjEnt) * c.ents_r2);
    w.cont_r2 = take(sizeof(Contrib) * c.cont_r2);
    w.stasks = take(sizeof(SampleTask) * c.stasks);
    w.rnode = take(sizeof(int) * c.rnode * kMaxNodes);
    w.rw = take(sizeof(float) * c.rnode * kMaxNodes);
    if (c.pitems_f > 0) {
        w.pitems_f = take(sizeof(PItem) * c.pitems_f);
        w.pitems_r = take(sizeof(PItem) * std::max<int64_t>(c.pitems_r, 1));
        w.pnum = take(sizeof(int) * 2 * (size_t)nsh);
        w.pcnt = take(sizeof(unsigned) * ((size_t)nsh + 1));  // per-shot counters, then the status word
    }
    for (int d = 0; d < nslot; ++d) w.dp.push_back(take(sizeof(float) * J.shots[J.slot_shot[d]].g.L.total));
    const int nf = nfields(J);
    for (int i = 0; i < nsh; ++i) {
        const ShotIn &S = J.shots[i];
        const int64_t F = S.g.L.total;
        // one region of everything that starts at zero;
        // fields 0..3: first set (p, p, mu, mu), 4..7: second set; a
        // modeling job has the two p levels of each set (and in 2-D the
        // middle-level slot 2)
        std::array<size_t, 8> f{0, 0, 0, 0, 0, 0, 0, 0};
        const int per = per_set(J.op, S.g.ndim);  // fields per set
        for (int k = 0; k < nf; ++k) f[(k / per) * 4 + k % per] = take(sizeof(float) * F);
        w.fld.push_back(f);
        w.acc0.push_back(J.op == RTM_OP_MODEL ? 0 : take(sizeof(float) * F));
        w.acc1.push_back(has_den(J.op) ? take(sizeof(float) * F) : 0);
    }
    w.zero_end = align256(off);
    for (int i = 0; i < nsh; ++i) {
        w.trint.push_back(take(sizeof(float) * (size_t)(J.nt + 1) * J.shots[i].nrec));
        w.wadj.push_back(J.op == RTM_OP_VJP ? take(sizeof(float) * (size_t)J.nt * kMaxNodes) : 0);
    }
    w.bytes = align256(off);
    return w;
}

int max_tiles(const GridInfo &g)
{
    const int64_t ny = g.ndim == 3 ? (g.NY + 3) / 4 : 1;
    return (int)(((int64_t)(g.NX + 63) / 64) * ny * (g.L.NZr / kMinZseg));
}

struct RawEnt {
    int tile, z, y, x;
    int cbeg, cend;  // its contributions, in the build's list
    int slot, shot;
};

// Builds the tiles and injection entries of every shot for one launch shape.
int build_tiling(Job &J, Tiling &T, bool with_receivers)
{
    T.tiles.clear();
    T.tiles3.clear();
    T.ents.clear();
    T.cont.clear();
    std::vector<RawEnt> se, re;
    std::vector<Contrib> pool;  // contributions of the entries
    // a march is unrolled by its queue of nine rows (planes) and checks no row of a round by itself
    if (T.tune.block == 0 && T.tune.zseg % kZUnroll != 0)
        return fail(RTM_EINVAL, "marching tiles of %d rows or planes, not a multiple of %d", T.tune.zseg, kZUnroll);
    // 2-D: one tile is TX adjacent strips (one workgroup); 3-D: one strip.
    // 2-D tiles of S > 1 steps per launch: strips of 64 vec columns starting
    // at j W - 4 (S - 1) that own W = 64 vec - 8 (S - 1) columns each
    // (neighbours overlap by 8 (S - 1)).
    const bool two = T.ndim == 2 && T.steps > 1;
    const int off = two ? 4 * (T.steps - 1) : 0;
    const int span = 64 * T.tune.vec;
    const int strip = two ? span - 2 * off : span * (T.ndim == 2 ? T.tune.tx : 1);
    const int ty = T.ndim == 3 ? T.tune.ty : 1;
    for (int s = 0; s < (int)J.shots.size(); ++s) {
        const ShotIn &S = J.shots[s];
        const GridInfo &g = S.g;
        const int NZr = g.L.NZr;
        const int ns = (g.NX + strip - 1) / strip;
        const int nys = T.ndim == 3 ? (g.NY + ty - 1) / ty : 1;
        const int nzs = (NZr + T.tune.zseg - 1) / T.tune.zseg;
        const int tbase = T.count();
        // Tiles are numbered band by band in z, row of tiles by row of tiles
        // within a band (3-D) and strip by strip within a row, so that the
        // workgroups that share lines run back to back on one XCD: adjacent
        // strips share their strip-end columns (2-D: measured 3-7 % faster
        // than strip by strip), adjacent 3-D y tiles the 4-row halos above
        // and below.  In 3-D an XCD then works on whole rows of a few y tiles;
        // with y innermost its neighbour strips were on other XCDs and every
        // strip-end line came from memory twice (612 x 612 x 356 cells, us
        // per step: forward 545 -> 520, reverse 1353 -> 1250).  A 3-D tuning
        // may number them z innermost instead (x strip, then y tile, then z
        // band).
        const bool zin = T.ndim == 3 && T.tune.zin;
        const int nA = zin ? ns : nzs, nB = nys, nC = zin ? nzs : ns;
        for (int ia = 0; ia < nA; ++ia)
            for (int ys = 0; ys < nB; ++ys)
                for (int ic = 0; ic < nC; ++ic) {
                    const int zs = zin ? ic : ia, xs = zin ? ia : ic;
                    const int z0 = zs * T.tune.zseg, z1 = std::min(z0 + T.tune.zseg, NZr);
                    if (T.ndim == 3) {
                        Tile3D t{};
                        t.shot = s;
                        t.x0 = xs * strip;
                        t.y0 = ys * ty;
                        t.z0 = z0;
                        t.z1 = z1;
                        T.tiles3.push_back(t);
                    } else {
                        Tile2D t{};
                        t.shot = s;
                        t.x0 = xs * strip - off;
                        t.z0 = z0;
                        t.z1 = z1;
                        T.tiles.push_back(t);
                    }
                }
        // (2-D multi-step: x is an owned column)
        auto tile_of = [&](int z, int y, int x) {
            if (zin) return tbase + ((x / strip) * nys + y / ty) * nzs + z / T.tune.zseg;
            return tbase + ((z / T.tune.zseg) * nys + (T.ndim == 3 ? y / ty : 0)) * ns + x / strip;
        };
        PointOp sp;
        if (!make_point(g, S.src, &sp))
            return fail(RTM_ERANGE, "shot %d: source (%g, %g, %g) outside the interior", s, S.src[0], S.src[1],
                        S.src[2]);
        const double hd = std::pow(g.h, g.ndim);
        const double h2 = g.h * g.h;
        for (int q = 0; q < sp.n; ++q) {
            const int c = (int)pool.size();
            // D (B w) = D' (h^2 W / h^d) w with D' = (v dt / h)^2.
            pool.push_back(Contrib{0, (float)(sp.w[q] * h2 / hd)});
            se.push_back(RawEnt{tile_of(sp.z[q], sp.y[q], sp.x[q]), sp.z[q], sp.y[q], sp.x[q], c, c + 1, q, s});
        }
        if (!with_receivers) continue;
        // Receiver terms by node: sorted by cell, stably, so that a node's
        // contributions stay in receiver order.  (An ordered map of nodes
        // with a list each: 2.5 ms more per call with 65536 receivers, before
        // the GPU has anything to do.)
        struct Hit {
            int64_t cell;
            int z, y, x, r;
            float w;
        };
        std::vector<Hit> hits;
        hits.reserve((size_t)S.nrec);
        for (int r = 0; r < S.nrec; ++r) {
            PointOp rp;
            if (!make_point(g, &S.rec[3 * (size_t)r], &rp))
                return fail(RTM_ERANGE, "shot %d: receiver %d outside the interior", s, r);
            // D R^T g = D' h^2 W g.
            for (int q = 0; q < rp.n; ++q)
                hits.push_back(Hit{rp.z[q] * g.L.plane + rp.y[q] * g.L.pitch + rp.x[q], rp.z[q], rp.y[q], rp.x[q], r,
                                   (float)(rp.w[q] * h2)});
        }
        auto by_cell = [](const Hit &p, const Hit &q) { return p.cell < q.cell; };
        if (!std::is_sorted(hits.begin(), hits.end(), by_cell)) std::stable_sort(hits.begin(), hits.end(), by_cell);
        for (size_t i = 0; i < hits.size();) {
            const Hit &h = hits[i];
            const int c = (int)pool.size();
            for (; i < hits.size() && hits[i].cell == h.cell; ++i) pool.push_back(Contrib{hits[i].r, hits[i].w});
            re.push_back(RawEnt{tile_of(h.z, h.y, h.x), h.z, h.y, h.x, c, (int)pool.size(), 0, s});
        }
    }
    // Multi-step tiles also list, per tile, every node inside its strip and
    // rows [z0 - 4 (S - 1), z1 + 4 (S - 1)), where the first step is
    // computed; three-step tiles also those of rows [z0 - 4, z1 + 4), where
    // the second is.
    std::vector<RawEnt> se1, re1, se2, re2;
    if (two) {
        auto widen = [&](const std::vector<RawEnt> &v, std::vector<RawEnt> &out, int ext) {
            for (const RawEnt &e : v) {
                const ShotIn &S = J.shots[e.shot];
                const int NZr = S.g.L.NZr;
                const int ns = (S.g.NX + strip - 1) / strip;
                const int nzs = (NZr + T.tune.zseg - 1) / T.tune.zseg;
                int tb = 0;  // first tile of the shot
                for (int q = 0; q < e.shot; ++q) {
                    const ShotIn &o = J.shots[q];
                    tb += ((o.g.NX + strip - 1) / strip) * ((o.g.L.NZr + T.tune.zseg - 1) / T.tune.zseg);
                }
                // ext <= 8 < zseg and 2 off < strip: the node lies in z tiles
                // zc - 1 .. zc + 1 and strips jc - 1 .. jc at most
                const int jc = (e.x + off) / strip, zc = e.z / T.tune.zseg;
                for (int zs = std::max(0, zc - 1); zs <= std::min(nzs - 1, zc + 1); ++zs)
                    for (int j = std::max(0, jc - 2); j <= std::min(ns - 1, jc + 1); ++j) {
                        const int x0 = j * strip - off;
                        const int z0 = zs * T.tune.zseg, z1 = std::min(z0 + T.tune.zseg, NZr);
                        if (e.x >= x0 && e.x < x0 + span && e.z >= z0 - ext && e.z < z1 + ext) {
                            RawEnt w = e;
                            w.tile = tb + zs * ns + j;
                            out.push_back(w);
                        }
                    }
            }
        };
        widen(se, se1, off);
        widen(re, re1, off);
        if (T.steps == 3) {
            widen(se, se2, 4);
            widen(re, re2, 4);
        }
    }
    auto order = [](const RawEnt &a, const RawEnt &b) {
        return std::tie(a.tile, a.z, a.y, a.x) < std::tie(b.tile, b.z, b.y, b.x);
    };
    std::sort(se.begin(), se.end(), order);
    std::sort(re.begin(), re.end(), order);
    std::sort(se1.begin(), se1.end(), order);
    std::sort(re1.begin(), re1.end(), order);
    std::sort(se2.begin(), se2.end(), order);
    std::sort(re2.begin(), re2.end(), order);
    for (auto &t : T.tiles)
        t.sbeg = t.send = t.rbeg = t.rend = t.s1beg = t.s1end = t.r1beg = t.r1end = t.s2beg = t.s2end = t.r2beg =
            t.r2end = 0;
    for (auto &t : T.tiles3) t.sbeg = t.send = t.rbeg = t.rend = 0;
    // kind: 0 source, 1 receivers, 2 source (first step), 3 receivers (first
    // step), 4 source (second step), 5 receivers (second step)
    auto emit = [&](std::vector<RawEnt> &v, int kind) {
        for (auto &e : v) {
            InjEnt E{e.z, e.y, e.x, (int)T.cont.size(), 0, e.slot, e.shot, 0};
            T.cont.insert(T.cont.end(), pool.begin() + e.cbeg, pool.begin() + e.cend);
            E.cend = (int)T.cont.size();
            const int idx = (int)T.ents.size();
            T.ents.push_back(E);
            int *b, *n;
            if (T.ndim == 3) {
                Tile3D &t = T.tiles3[e.tile];
                b = kind == 0 ? &t.sbeg : &t.rbeg;
                n = kind == 0 ? &t.send : &t.rend;
            } else {
                Tile2D &t = T.tiles[e.tile];
                int *bs[6] = {&t.sbeg, &t.rbeg, &t.s1beg, &t.r1beg, &t.s2beg, &t.r2beg};
                int *ns_[6] = {&t.send, &t.rend, &t.s1end, &t.r1end, &t.s2end, &t.r2end};
                b = bs[kind];
                n = ns_[kind];
            }
            if (*n == *b) *b = idx;
            *n = idx + 1;
        }
    };
    emit(se, 0);
    T.nsrc_ent = (int)se.size();
    emit(re, 1);
    T.nrec_ent = (int)re.size();
    emit(se1, 2);
    emit(re1, 3);
    emit(se2, 4);
    emit(re2, 5);
    T.nslots = (T.count() + kNumXcd - 1) / kNumXcd * kNumXcd;
    return RTM_OK;
}

// Wavefronts a 2-D shape of one step per launch gives a job.
int64_t count_tiles(const Job &J, Tune t)
{
    int64_t n = 0;
    for (const ShotIn &S : J.shots)
        n += (int64_t)((S.g.NX + 64 * t.vec * t.tx - 1) / (64 * t.vec * t.tx)) * t.tx *
             ((S.g.L.NZr + t.zseg - 1) / t.zseg);
    return n;
}

// Workgroups a 3-D shape gives a job.
int64_t count_tiles3(const Job &J, Tune t)
{
    int64_t n = 0;
    for (const ShotIn &S : J.shots)
        n += (int64_t)((S.g.NX + 64 * t.vec - 1) / (64 * t.vec)) * ((S.g.NY + t.ty - 1) / t.ty) *
             ((S.g.L.NZr + t.zseg - 1) / t.zseg);
    return n;
}

// Shape of a 3-D pass, no larger than the configured one.
//
// once: a step's arrays beyond 7/8 of the 256 MiB memory-side cache come from
// HBM whatever is done, and then the L2 serves the shared halo rows better
// without the arrays that are touched once; smaller ones live in that cache
// (us per step with / without: 612 x 612 x 356 cells forward 419 / 538,
// reverse 1096 / 1266; 300^3 reverse 250 / 329; 252^3 reverse, 416 MB, 133 /
// 157; 220^3 reverse, 276 MB, 99 / 104; 252^3 forward, 192 MB, 47 / 45; 188^3
// reverse, 171 MB, 61 / 55).  A model that several shots share is not touched
// once (with / without: 16 x 124^3 forward 111 / 99, reverse 341 / 292,
// gradient 283 / 256; 8 x 188^3 186 / 163, 548 / 476, 444 / 405), which counts
// from four shots on in a forward step and, in a reverse step of two fields,
// from eight on beyond twice the cache (4 x 304 x 337 x 43 160 / 187, 16 x 96^3
// gradient 130 / 138).  Rows of one strip are read whole by their own tiles,
// and the reverse step of a field narrower than that is better with the caches
// on all but the gradient with a model per shot (64 x 64^3 203 / 186, 50 x 54 x
// 324 x 76 1045 / 822, 30 x 56 x 107 x 92 232 / 208; that gradient goes either
// way, 14 x 38 x 132 x 186 190 / 211, 50 x 50 x 35 x 390 485 / 440).  Over 278 drawn jobs the
// rule costs forward 0.1, reverse 1.6, gradient 1.2 % against the better of the
// two for each (once for all: 3.6, 3.0, 2.1 %); with a model per shot small
// extents go either way (reverse, 16 x 124^3 339 / 309, 5 x 301 x 55 x 205
// 0.78 of the time without).
//
// In the cache a step is a matter of latency and of instructions.  Forward
// and receiver steps take the smallest tiles, one float x 4 rows x 9 planes,
// whatever the size (us per step at 1 x 4 x 9, 1 x 8 x 9, 1 x 4 x 27 and, where
// larger tiles fill the chip, 2 x 8 x 9: 64^3 7.1, 7.2, 13.8; 144^3 11.2, 11.3,
// 16.3, 15.4; 188^3 20.1, 21.2, 19.3, 21.5; 300 x 300 x 60 20.0, 20.3, 19.2,
// 22.8; over 100 sizes and batches within 1.3 % of the best on average).  The
// reverse kernel has four wavefronts per SIMD: it takes these tiles while its
// workgroups are all resident, four per CU (a fifth is soon through), also of 18
// and 27 planes if these still give 2.5 per CU, else the configured ones (1 x 4
// against 1 x 8 rows: 64^3 12.1 / 15.2, 128^3 20.6 /
// 20.9, 400 x 90 x 70, 5.0 per CU, 23.9 / 25.0, 260 x 180 x 100 at 27 planes
// 39.1 / 45.6, 188^3 53.5 / 52.1; 3 x 78 x 353 x 24
// at 27, 2.1 per CU, 33.1 / 26.6; not resident: 2 x 124^3 at 9 planes 37.2 /
// 34.5, 4 x 124^3 at 36 79.8 / 75.9).
//
// Planes per tile otherwise: the least march time.  A tile marches 8 planes
// beyond its own, and the fullest CU ends the launch: one workgroup of 16
// wavefronts fills a CU, smaller ones share it, k of them taking about 1.2 + k
// units (501 x 501 x 235 cells, one / two / 2.5 workgroups of 16 per CU: 164 /
// 170 / 199 us per step; 612 x 612 x 356 at 72 planes, 3.8 per CU, 418, at 90,
// 3.05, 477, at 63, 4.6, 444).  The reverse kernel, at two rows per wavefront, stays near its
// memory time at any height that leaves enough workgroups (316^3 at 9 to 81
// planes 297 to 325); on arrays that fit the cache the same march rule holds,
// with a floor for what a lone workgroup takes per plane (188^3 at 9, 18, 27,
// 36 planes 55.5, 67.0, 52.1, 56.9), and from 14 workgroups per CU on nine
// planes are best (4 x 156^3, 16.9 per CU, at 9, 27 and 54 planes 140, 159,
// 142; 8 x 124^3, 14: 148, 161, 147; 24 x 64^3, 12: 65.1, at 18 63.1).  So
// they are beyond the cache while a band of planes is small, which the next
// band's workgroups find in the L2 (14 x 125 x 135 x 195 at 9, 27, 54 planes
// 505, 526, 550; forward, 30 x 38 x 98 x 114 at one float x 16 rows 71, 84, 94;
// 300^3 258, 262, 289; of 4 rows where 8 compute a tenth more, 28 x 132 x 325
// 93 / 98, 50 x 50 x 35 x 390 489 / 507; single grids of 420 x 420 cells a plane 345, 339, 350,
// of 501 x 501 658, 573, 588).
enum Pass3 { kFwd3, kRecv3, kRev3 };
constexpr int64_t kCacheBytes = (int64_t)224 << 20;

int once3(const Job &J, Pass3 pass)
{
    const int64_t nsh = (int64_t)J.shots.size();
    int64_t bytes = 0;
    int NX = 0;
    for (const ShotIn &S : J.shots) {
        const GridInfo &g = S.g;
        NX = std::max(NX, g.NX);
        const int64_t all = 4 * (int64_t)g.NX * g.NY * g.NZ, in = 4 * g.nx * g.ny * g.nz;
        bytes += pass != kRev3 ? 3 * all : J.op == RTM_OP_VJP ? 6 * all : 5 * all + 2 * in;
    }
    if (bytes <= kCacheBytes) return 0;
    const bool own = (int64_t)J.slot_shot.size() == nsh;  // a model for each shot
    if (pass == kRev3 && NX <= 64 && !(J.op == RTM_OP_VJP && own)) return 0;
    if (own) return kOnce;
    return (pass != kRev3 ? nsh >= 4 : nsh >= 8 && bytes > 2 * kCacheBytes) ? 0 : kOnce;
}

Tune fit_tune3(const Job &J, Tune t, Pass3 pass)
{
    int NZr = 0, NX = 0, NY = 0;
    int64_t plane = 0;
    for (const ShotIn &S : J.shots) {
        NZr = std::max(NZr, S.g.L.NZr);
        NX = std::max(NX, S.g.NX);
        NY = std::max(NY, S.g.NY);
        plane = std::max(plane, (int64_t)S.g.NX * S.g.NY);
    }
    t.once = once3(J, pass);
    if (g_tune_exact.load()) return t;
    if (NX <= 64) t.vec = 1;  // half the lanes would be idle
    const int top = t.zseg;
    if (!t.once) {
        Tune c = t;
        c.vec = 1;
        c.ty = 4;
        for (c.zseg = kMinZseg; c.zseg <= std::min(top, 3 * kMinZseg); c.zseg += kMinZseg) {
            const double n = (double)count_tiles3(J, c) / 256.0;
            if (pass != kRev3 || (c.zseg == kMinZseg ? n <= 5.1 : n >= 2.5 && n <= 4.15)) return c;
        }
    }
    const bool full = t.ty * t.vec >= 32;  // workgroups that fill a CU
    if (!t.once || (!full && plane <= 160000)) {
        Tune c = t;
        c.zseg = kMinZseg;
        if ((double)count_tiles3(J, c) >= 256.0 * 14.0) {
            if (pass == kRev3 && c.ty == 8 && (NY + 3) / 4 * 40 <= (NY + 7) / 8 * 72) c.ty = 4;
            return c;
        }
    }
    double least = 0.0;
    for (int seg = 1; seg <= NZr / kZUnroll; ++seg) {
        Tune c = t;
        c.zseg = (NZr / kZUnroll + seg - 1) / seg * kZUnroll;
        if (c.zseg > top || (least != 0.0 && c.zseg == t.zseg)) continue;
        const double n = (double)count_tiles3(J, c) / 256.0;  // workgroups per CU
        double cost;
        if (pass != kRev3) cost = full ? (c.zseg + 8) * std::ceil(n) : (c.zseg + 6) * (1.2 + (n > 4.0 ? n : std::ceil(n)));
        else if (!t.once) cost = (c.zseg + 8) * std::max(1.13, 0.5 + 0.22 * (n + std::ceil(n)));
        else cost = n >= 16.0 && c.zseg > kMinZseg ? 1.0 : 2.0 + c.zseg;  // the tallest that leaves 16 per CU
        if (least == 0.0 || cost < least) {
            least = cost;
            t.zseg = c.zseg;
        }
    }
    t.zseg = std::min(t.zseg, top);
    return t;
}

// The configured 2-D shape of one step per launch is meant for large
// batches; a small job (a single shot of a modest grid) would leave most of
// the 256 CUs idle, so the shape is narrowed (fewer rows per tile first, then
// fewer floats per lane) until the job has at least kMinWaves wavefronts or
// the smallest shape is reached.  Results do not depend on the shape.  (The
// multi-step shape is chosen by fit_multi.)
constexpr int64_t kMinWaves = 256 * 16;

Tune fit_tune(const Job &J, Tune t)
{
    if (g_tune_exact.load()) return t;
    while (count_tiles(J, t) < kMinWaves) {
        if (t.zseg > kMinZseg) t.zseg = std::max(kMinZseg, t.zseg / 2 / kZUnroll * kZUnroll);
        else if (t.vec > 1) t.vec /= 2;
        else break;
    }
    return t;
}

// Wavefronts of a 2-D launch of `steps` time steps.
int64_t count_multi(const Job &J, int steps, int vec, int zseg)
{
    int64_t n = 0;
    const int own = 64 * vec - 8 * (steps - 1);
    for (const ShotIn &S : J.shots) n += (int64_t)((S.g.NX + own - 1) / own) * ((S.g.L.NZr + zseg - 1) / zseg);
    return n;
}

// Rows per tile of a 2-D multi-step launch: the height, from the configured
// one down, with the least march time.  A tile marches 9 (T - 1) rows beyond
// its own; a SIMD with k wavefronts takes about 0.5 + k units per row and no
// less than 2.2 (what its own latency costs a lone wavefront).  Up to three
// wavefronts per SIMD all are resident and the fullest SIMD ends the launch,
// so k lies half way to the whole number above.  Measured (us per step, forward, three steps, two floats per lane):
// 4 shots of 2301 x 751 at 18, 27, 36, 54 rows 19.4, 15.1, 16.5, 17.0; 8
// shots at 27, 36, 54, 108 rows 31.4, 31.3, 29.3, 33.0; 16 shots at 54, 108
// rows 57.1, 52.7; 24 windows at 18, 27, 36 rows 15.7, 15.5, 14.5.
int best_rows(const Job &J, int steps, int vec, int top, int least)
{
    int best = top;
    double cost = 0.0;
    for (int z : {top, 108, 54, 36, 27, 18, 9}) {
        if (z != top && (z > top || z < least)) continue;
        const double n = count_multi(J, steps, vec, z) / 1024.0;  // wavefronts per SIMD
        const double k = n <= 3.0 ? 0.5 * (n + std::ceil(n)) : n;
        const double c = (z + 9 * (steps - 1)) * std::max(2.2, 0.5 + k);
        if (cost == 0.0 || c < cost) {
            cost = c;
            best = z;
        }
    }
    return best;
}

// Shape of a 2-D multi-step launch: the configured steps and floats per lane
// while their shortest useful tiles (18 rows forward, 27 reverse: shorter
// ones march twice their rows) still give about two wavefronts per SIMD.
// Below that three steps give way to two and the lanes are narrowed.
// Measured (us per step, forward / reverse): 12 windows, three steps 9.4
// against two 9.8; 2 shots, reverse, two steps at one float 20.6 against
// three 26.4 and two at two floats 21.0; 1 shot, two steps, nine rows, two
// floats 6.6 / 13.2 against one 7.4 / 14.5; 1574 x 534, one float 4.7 / 8.9
// against two 4.8 / 10.0.
//
// Before that, a job of few blocks takes the block kernels, the smallest
// shape that keeps to its rounds of blocks: two per CU at 1/8/4 (52 and 102
// registers), one at 2/12/3; 2/16/3 (two blocks per CU forward, one reverse)
// as long as it beats the strips.  Measured (blocks, then blocks against
// strips): 1/8/4 465 2.3 / 4.0 against 3.8 / 6.5, 646 2.7 / 5.2; 2/12/3 216
// 2.5 / 4.9 against 4.0 / 6.9, 300 3.1 / 7.4; 2/16/3 255 2.95 / 6.1 against
// 4.6 / 8.8, 418 4.1 / 9.9 against 6.4 / 11.9, 616 5.3 / 14.0 against 6.6 /
// 13.0, 1232 7.9 / 23.3 against 10.8 / 20.8, 3696 20.3 against 22.8, 4928
// 32.3 against 30.0.  Two reverse steps at two floats, where three have too
// many blocks, keep to them too (432 to 493 blocks 13 to 17 against 16 to 20).
int fit_block(const Job &J, int steps, bool reverse)
{
    const int64_t most[] = {0, 512, 256, reverse ? 512 : 3700};
    for (int i = 1; i < 4; ++i) {
        const BlockShape &b = kBlockShapes[i];
        if (count_multi(J, steps, b.vec, b.waves * b.rows - 8 * (steps - 1)) <= most[i]) return i;
    }
    return 0;
}

// once, as in fit_tune3: the arrays a multi-step launch moves (the fields read
// and written, D' per model, imaging sums) beyond the 256 MiB memory-side
// cache.  Measured (us per step with / without, reverse): 3 shots of 2301 x
// 751, 246 MB, 35.2 / 31.8; 4 shots 38.3 / 39.3; 8 shots 69.1 / 72.2; 48
// shots 378 / 413; forward: 8 shots, 272 MB, 29.6 / 29.6; 48 shots 143 / 150;
// gradient: 24 windows 38.6 / 40.1.
int once_multi(const Job &J, bool reverse)
{
    int64_t bytes = 0;
    for (int s = 0; s < (int)J.shots.size(); ++s) {
        const GridInfo &g = J.shots[s].g;
        const int64_t all = 4 * (int64_t)g.NX * g.NZ, in = 4 * g.nx * g.nz;
        bytes += (reverse ? 8 : 4) * all + (!reverse ? 0 : J.op == RTM_OP_VJP ? all : 2 * in);
        if (J.slot_shot[J.dslot[s]] == s) bytes += all;
    }
    return bytes > ((int64_t)256 << 20) ? kOnce : 0;
}

Tune block_shape(Tune t)
{
    const BlockShape &b = kBlockShapes[t.block];
    t.once = 0;  // the block kernels have no such form
    t.vec = b.vec;
    t.zseg = b.waves * b.rows - 8 * (t.steps - 1);
    return t;
}

Tune fit_multi(const Job &J, Tune t, bool reverse)
{
    if (t.vec < 4) t.once = once_multi(J, reverse);
    if (g_tune_exact.load()) return t;
    if ((t.block = fit_block(J, t.steps, reverse)) != 0) return block_shape(t);
    const int least = reverse && t.steps == 3 ? 27 : 18;
    if (count_multi(J, t.steps, t.vec, std::min(t.zseg, least)) >= (reverse ? 2048 : 1900)) {
        t.zseg = best_rows(J, t.steps, t.vec, t.zseg, least);
        return t;
    }
    t.steps = 2;
    if (reverse && count_multi(J, 2, 1, 18) >= 2300) {
        t.vec = 1;
        t.zseg = best_rows(J, 2, 1, 54, 18);
    } else {
        t.vec = count_multi(J, 2, 2, kMinZseg) >= 1800 ? 2 : 1;
        if (reverse && t.vec == 2 && (t.block = fit_block(J, 2, true)) != 0) return block_shape(t);
        t.zseg = best_rows(J, 2, t.vec, 18, kMinZseg);
    }
    return t;
}

// Receiver sampling tables, D' sharing and tilings of a job.
int build_job_tables(Job &J)
{
    J.stasks.clear();
    J.rnode.clear();
    J.rw.clear();
    J.rbase.clear();
    J.srows.clear();
    J.dslot.clear();
    J.slot_shot.clear();
    int64_t base = 0;
    for (const ShotIn &S : J.shots) base += S.nrec;
    J.rnode.reserve((size_t)base * kMaxNodes);
    J.rw.reserve((size_t)base * kMaxNodes);
    base = 0;
    for (int s = 0; s < (int)J.shots.size(); ++s) {
        const ShotIn &S = J.shots[s];
        J.rbase.push_back(base);
        std::array<int, 2> rows{1 << 30, 0};
        for (int r = 0; r < S.nrec; ++r) {
            PointOp rp;
            if (!make_point(S.g, &S.rec[3 * (size_t)r], &rp))
                return fail(RTM_ERANGE, "shot %d: receiver %d (%g, %g, %g) outside the interior", s, r,
                            S.rec[3 * r], S.rec[3 * r + 1], S.rec[3 * r + 2]);
            for (int q = 0; q < kMaxNodes; ++q) {
                if (q < rp.n) {
                    rows[0] = std::min(rows[0], rp.z[q]);
                    rows[1] = std::max(rows[1], rp.z[q] + 1);
                    // below L.total, which grid_info keeps under 2^31: fits an int
                    J.rnode.push_back((int)((int64_t)rp.z[q] * S.g.L.plane + (int64_t)rp.y[q] * S.g.L.pitch + rp.x[q]));
                    J.rw.push_back((float)rp.w[q]);
                } else {
                    J.rnode.push_back(0);
                    J.rw.push_back(0.f);
                }
            }
        }
        base += S.nrec;
        J.srows.push_back(rows[1] > rows[0] ? rows : std::array<int, 2>{0, 0});
        for (int r0 = 0; r0 < S.nrec; r0 += 64) J.stasks.push_back(SampleTask{s, r0});
        int slot = -1;
        for (int d = 0; d < (int)J.slot_shot.size(); ++d) {
            const ShotIn &o = J.shots[J.slot_shot[d]];
            if (o.v_pad == S.v_pad && o.g.NX == S.g.NX && o.g.NY == S.g.NY && o.g.NZ == S.g.NZ && o.g.h == S.g.h) {
                slot = d;
                break;
            }
        }
        if (slot < 0) {
            slot = (int)J.slot_shot.size();
            J.slot_shot.push_back(s);
        }
        J.dslot.push_back(slot);
    }
    const int ndim = J.shots[0].g.ndim;
    const bool persist = (J.flags & RTM_F_PERSISTENT) != 0;
    J.fw.ndim = J.rv.ndim = J.fw2.ndim = J.rv2.ndim = ndim;
    const Tune conf_f = get_tune(0, ndim), conf_r = get_tune(J.op == RTM_OP_STORAGE ? 0 : 1, ndim);
    J.fw.tune = ndim == 3 ? fit_tune3(J, conf_f, kFwd3) : fit_tune(J, conf_f);
    if (persist) {
        // one strip per workgroup, one step per item
        J.fw.tune.tx = 1;
        J.fw.tune.steps = 1;
    }
    int rc = build_tiling(J, J.fw, false);
    if (rc) return rc;
    if (J.op != RTM_OP_MODEL) {
        // the storage reverse pass steps one field, as the forward pass does
        J.rv.tune = ndim == 3 ? fit_tune3(J, conf_r, J.op == RTM_OP_STORAGE ? kRecv3 : kRev3) : fit_tune(J, conf_r);
        if (persist) {
            J.rv.tune.tx = 1;
            J.rv.tune.steps = 1;
        }
        rc = build_tiling(J, J.rv, true);
        if (rc) return rc;
    }
    J.pitems_f.clear();
    J.pitems_r.clear();
    J.pnum.clear();
    if (persist) {
        const int nsh = (int)J.shots.size();
        J.pnum.assign(2 * (size_t)nsh, 0);
        for (int t = 0; t < (int)J.fw.tiles.size(); ++t) {
            J.pitems_f.push_back(PItem{t, J.fw.tiles[t].shot});
            J.pnum[J.fw.tiles[t].shot]++;
        }
        if (J.op == RTM_OP_MODEL)
            for (int k = 0; k < (int)J.stasks.size(); ++k) {
                J.pitems_f.push_back(PItem{-1 - k, J.stasks[k].shot});
                J.pnum[J.stasks[k].shot]++;
            }
        for (int t = 0; t < (int)J.rv.tiles.size(); ++t) {
            J.pitems_r.push_back(PItem{t, J.rv.tiles[t].shot});
            J.pnum[nsh + J.rv.tiles[t].shot]++;
        }
    }
    // Multi-step tilings (2-D): the forward one for every op, the reverse
    // one for imaging and the gradient.  Three steps per launch store the
    // middle level only on the receiver rows, so storage RTM (which copies
    // whole stored levels) takes two.  The gradient pass takes three where
    // the runtime chooses the shape and two of a configured one.  Its triple
    // (209 registers at two floats per lane) pays with many wavefronts, where
    // it saves traffic, and with few; between them, two steps can be the
    // quicker (us per step, two / three: 4 windows of 880 x 380 12.7 / 11.1,
    // 18 39.1 / 33.6, 24 50.1 / 56.2, 48 94 / 93, 96 201 / 162, 192 404 / 285;
    // 4 shots of 2381 x 831 43.5 / 52.3, 8 86 / 85, 16 175 / 149, 48 516 / 352).
    // Where it needs two strips for what two steps hold in one it is
    // slower (60 shots of 117 x 1891 95.5 / 118.5, 200 of 120 x 400 61.5 / 88.1).
    J.fw2 = Tiling{};
    J.rv2 = Tiling{};
    J.fw2.ndim = J.rv2.ndim = ndim;
    if (ndim != 2 || persist) return RTM_OK;
    if (conf_f.steps >= 2) {
        Tune t = conf_f;
        if (J.op == RTM_OP_STORAGE) t.steps = 2;
        J.fw2.tune = fit_multi(J, t, false);
        J.fw2.steps = J.fw2.tune.steps;
        if ((rc = build_tiling(J, J.fw2, false))) return rc;
    }
    if ((J.op == RTM_OP_RTM || J.op == RTM_OP_VJP) && conf_r.steps >= 2) {
        Tune t = conf_r;
        if (J.op == RTM_OP_VJP && t.steps == 3 &&
            (g_tune_exact.load() || count_multi(J, 3, t.vec, t.zseg) >= 2 * count_multi(J, 2, t.vec, t.zseg)))
            t.steps = 2;
        J.rv2.tune = fit_multi(J, t, true);
        J.rv2.steps = J.rv2.tune.steps;
        if ((rc = build_tiling(J, J.rv2, true))) return rc;
    }
    return RTM_OK;
}

Counts exact_counts(const Job &J)
{
    Counts c;
    c.tiles_f = J.fw.count();
    c.ents_f = J.fw.ents.size();
    c.cont_f = J.fw.cont.size();
    c.tiles_r = J.rv.count();
    c.ents_r = J.rv.ents.size();
    c.cont_r = J.rv.cont.size();
    c.tiles_f2 = J.fw2.count();
    c.ents_f2 = J.fw2.ents.size();
    c.cont_f2 = J.fw2.cont.size();
    c.tiles_r2 = J.rv2.count();
    c.ents_r2 = J.rv2.ents.size();
    c.cont_r2 = J.rv2.cont.size();
    c.stasks = J.stasks.size();
    c.rnode = J.rnode.size() / kMaxNodes;
    c.pitems_f = J.pitems_f.size();
    c.pitems_r = J.pitems_r.size();
    return c;
}

// Upper bounds for one shot, independent of positions and launch shape.
Counts bound_counts(const GridInfo &g, int op, int nrec)
{
    Counts c;
    c.tiles_f = max_tiles(g);
    c.ents_f = c.cont_f = kMaxNodes;
    if (op != RTM_OP_MODEL) {
        c.tiles_r = max_tiles(g);
        c.ents_r = c.cont_r = kMaxNodes + (int64_t)kMaxNodes * nrec;
    }
    if (g.ndim == 2) {
        // multi-step strips own >= 48 columns; a node lies in at most 2
        // strips x 3 tiles in z for the first step, 2 x 2 for the second
        // (three steps) and its owner: 11 entries
        const int64_t t2 = ((g.NX + 47) / 48) * (g.L.NZr / kMinZseg);
        c.tiles_f2 = t2;
        c.ents_f2 = c.cont_f2 = 11 * kMaxNodes;
        if (op == RTM_OP_RTM || op == RTM_OP_VJP) {
            c.tiles_r2 = t2;
            c.ents_r2 = c.cont_r2 = 11 * (kMaxNodes + (int64_t)kMaxNodes * nrec);
        }
    }
    c.stasks = (nrec + 63) / 64;
    c.rnode = nrec;
    return c;
}

// Device addresses of the job's buffers inside `ws`.
struct Dev {
    char *base;
    template <class T>
    T *at(size_t off) const { return (T *)(base + off); }
};

// Two shot tables: out[0 .. nsh) addresses the field sets in order, out[nsh
// .. 2 nsh) with the sets exchanged (current levels after an odd number of
// multi-step launches).
void fill_shot_devs(const Job &J, const Dev &D, std::vector<ShotDev> &out)
{
    const size_t nsh = J.shots.size();
    out.resize(2 * nsh);
    for (size_t i = 0; i < nsh; ++i) {
        const ShotIn &S = J.shots[i];
        ShotDev &d = out[i];
        std::memset(&d, 0, sizeof d);
        for (int k = 0; k < 8; ++k) d.fld[k] = J.ws.fld[i][k] ? D.at<float>(J.ws.fld[i][k]) : nullptr;
        d.acc0 = J.op == RTM_OP_MODEL ? nullptr : D.at<float>(J.ws.acc0[i]);
        d.acc1 = has_den(J.op) ? D.at<float>(J.ws.acc1[i]) : nullptr;
        d.Dp = D.at<float>(J.ws.dp[J.dslot[i]]);
        d.wav = S.wavelet;
        float *trint = D.at<float>(J.ws.trint[i]);
        d.sig = J.op == RTM_OP_MODEL ? nullptr : trint;
        d.rec_out = J.op == RTM_OP_MODEL ? trint : nullptr;
        d.traces_in = S.traces_in;
        d.traces_out = S.traces_out;
        d.rnode = D.at<int>(J.ws.rnode) + J.rbase[i] * kMaxNodes;
        d.rw = D.at<float>(J.ws.rw) + J.rbase[i] * kMaxNodes;
        d.nrec = S.nrec;
        d.ix0 = S.g.nb;
        d.ix1 = S.g.nb + (int)S.g.nx;
        d.iy0 = S.g.ndim == 3 ? S.g.nb : 0;
        d.iy1 = S.g.ndim == 3 ? S.g.nb + (int)S.g.ny : 1;
        d.iz0 = S.g.nb;
        d.iz1 = S.g.nb + (int)S.g.nz;
        d.sz0 = J.srows[i][0];
        d.sz1 = J.srows[i][1];
        d.L = S.g.L;
        ShotDev &x = out[nsh + i];
        x = d;
        for (int k = 0; k < 8; ++k) x.fld[k] = d.fld[k ^ 4];
    }
}

template <class T>
int upload(const Dev &D, size_t off, const std::vector<T> &v, hipStream_t st)
{
    if (v.empty()) return RTM_OK;
    RTM_HIP(hipMemcpyAsync(D.at<char>(off), v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, st));
    return RTM_OK;
}

// Copies the tables and shot descriptors into the workspace and, unless
// skipped, checks every D' slot's velocity range; synchronises once.
int job_upload_and_check(const Job &J, const Dev &D, std::vector<ShotDev> &shot_devs, hipStream_t st)
{
    int rc;
    fill_shot_devs(J, D, shot_devs);
    if ((rc = upload(D, J.ws.shots, shot_devs, st))) return rc;
    if ((rc = upload(D, J.ws.tiles_f, J.fw.tiles, st))) return rc;
    if ((rc = upload(D, J.ws.tiles_f, J.fw.tiles3, st))) return rc;
    if ((rc = upload(D, J.ws.tiles_r, J.rv.tiles3, st))) return rc;
    if ((rc = upload(D, J.ws.ents_f, J.fw.ents, st))) return rc;
    if ((rc = upload(D, J.ws.cont_f, J.fw.cont, st))) return rc;
    if ((rc = upload(D, J.ws.tiles_r, J.rv.tiles, st))) return rc;
    if ((rc = upload(D, J.ws.ents_r, J.rv.ents, st))) return rc;
    if ((rc = upload(D, J.ws.cont_r, J.rv.cont, st))) return rc;
    if ((rc = upload(D, J.ws.tiles_f2, J.fw2.tiles, st))) return rc;
    if ((rc = upload(D, J.ws.ents_f2, J.fw2.ents, st))) return rc;
    if ((rc = upload(D, J.ws.cont_f2, J.fw2.cont, st))) return rc;
    if ((rc = upload(D, J.ws.tiles_r2, J.rv2.tiles, st))) return rc;
    if ((rc = upload(D, J.ws.ents_r2, J.rv2.ents, st))) return rc;
    if ((rc = upload(D, J.ws.cont_r2, J.rv2.cont, st))) return rc;
    if ((rc = upload(D, J.ws.stasks, J.stasks, st))) return rc;
    if ((rc = upload(D, J.ws.rnode, J.rnode, st))) return rc;
    if ((rc = upload(D, J.ws.rw, J.rw, st))) return rc;
    if (!J.pitems_f.empty()) {
        if ((rc = upload(D, J.ws.pitems_f, J.pitems_f, st))) return rc;
        if ((rc = upload(D, J.ws.pitems_r, J.pitems_r, st))) return rc;
        if ((rc = upload(D, J.ws.pnum, J.pnum, st))) return rc;
    }
    const int nslot = (int)J.slot_shot.size();
    std::vector<unsigned> vr(2 * (size_t)nslot, 0u);
    const bool check = !(J.flags & RTM_F_SKIP_CHECK);
    unsigned *scal = D.at<unsigned>(J.ws.scal);
    if (check) {
        for (int d = 0; d < nslot; ++d) {
            const GridInfo &g = J.shots[J.slot_shot[d]].g;
            RTM_HIP(launch_vrange(J.shots[J.slot_shot[d]].v_pad, (int64_t)g.NX * g.NY * g.NZ, scal + 64 + 2 * d, st));
        }
        RTM_HIP(hipMemcpyAsync(vr.data(), scal + 64, vr.size() * sizeof(unsigned), hipMemcpyDeviceToHost, st));
    }
    RTM_HIP(hipStreamSynchronize(st));
    if (check) {
        for (int d = 0; d < nslot; ++d) {
            const ShotIn &S = J.shots[J.slot_shot[d]];
            float vmax, vmin;
            std::memcpy(&vmax, &vr[2 * d], 4);
            std::memcpy(&vmin, &vr[2 * d + 1], 4);
            if (vr[2 * d] >= 0x7f800000u || !(vmin >= 0.f) || !(vmax > 0.f))
                return fail(RTM_ENUMERIC, "shot %d: velocity must be finite, >= 0 and not all 0 (max bits 0x%08x, min %g)",
                            J.slot_shot[d], vr[2 * d], (double)vmin);
            const double limit = std::sqrt(315.0 / (512.0 * S.g.ndim));
            const double courant = (double)vmax * J.dt / S.g.h;
            if (!(courant < limit))
                return fail(RTM_ECFL, "shot %d: max(v) dt / h = %.6f >= stability limit %.6f", J.slot_shot[d],
                            courant, limit);
        }
    }
    return RTM_OK;
}

// The device work of a job, after the upload (capturable in a hipGraph:
// kernel launches only).
int job_launch(const Job &J, const Dev &D, hipStream_t st, const rtm_probe_t *probe, bool timed)
{
    const ShotDev *table = D.at<ShotDev>(J.ws.shots);
    const int nsh = (int)J.shots.size();
    const int nt = J.nt;
    // Current shot table: 0 while the latest levels are in the first field
    // set, 1 after an odd number of multi-step launches.
    int cur = 0;
    auto SH = [&]() { return table + (size_t)cur * nsh; };
    auto fld_of = [&](int i, int k) { return D.at<float>(J.ws.fld[i][cur ? (k ^ 4) : k]); };
    unsigned *scal = D.at<unsigned>(J.ws.scal);
    // Two-step launches write the second field set: every level they touch
    // must have a buffer.
    for (int i = 0; i < nsh; ++i) {
        const bool need_p = J.fw2.steps > 1 || J.rv2.steps > 1, need_mu = J.rv2.steps > 1;
        const bool need_mid = J.op == RTM_OP_MODEL && J.fw2.steps == 3;
        if ((need_p && !(J.ws.fld[i][4] && J.ws.fld[i][5])) || (need_mu && !(J.ws.fld[i][6] && J.ws.fld[i][7])) ||
            (need_mid && !(J.ws.fld[i][2] && J.ws.fld[i][6])))
            return fail(RTM_EINVAL, "internal: shot %d lacks the second field set of multi-step launches", i);
    }
    for (int d = 0; d < (int)J.slot_shot.size(); ++d) {
        const ShotIn &S = J.shots[J.slot_shot[d]];
        RTM_HIP(launch_build_dp(S.g.L, S.v_pad, (float)(J.dt / S.g.h), D.at<float>(J.ws.dp[d]), st));
    }
    // Fields and sums of every shot, one region: a launch per field and shot
    // left the GPU idle between them (48 shots, imaging: 480 launches, 2.3 ms
    // and as much again in gaps).
    RTM_HIP(launch_zero(D.at<char>(J.ws.fld[0][0]), J.ws.zero_end - J.ws.fld[0][0], st));
    int maxrec = 0;
    for (int i = 0; i < nsh; ++i) {
        maxrec = std::max(maxrec, J.shots[i].nrec);
        if (J.op == RTM_OP_VJP && J.shots[i].grad_wavelet)
            RTM_HIP(launch_fill(D.at<float>(J.ws.wadj[i]), (int64_t)nt * kMaxNodes, 0.f, st));
    }
    if (J.op != RTM_OP_MODEL) RTM_HIP(launch_traces(table, nsh, maxrec, nt + 1, true, st));
    // Forward pass (Algorithm 1; in RTM only the last two panels are kept).
    {
        const PassRange pass("rtm:forward");
        const bool sample = J.op == RTM_OP_MODEL;
        const Tile2D *tiles = D.at<Tile2D>(J.ws.tiles_f);
        const InjEnt *ents = D.at<InjEnt>(J.ws.ents_f);
        const Contrib *cont = D.at<Contrib>(J.ws.cont_f);
        const SampleTask *stasks = D.at<SampleTask>(J.ws.stasks);
        const int ntiles = J.fw.count();
        const int nsample = sample ? (int)J.stasks.size() : 0;
        const bool two = J.fw.ndim == 2 && J.fw2.steps > 1;
        const int fs = two ? J.fw2.steps : 1;
        const bool persist = !J.pitems_f.empty();
        LoopTimer timer(sample ? kLoopModelFwd : kLoopRtmFwd, persist ? 1 : nt / fs + nt % fs, st, timed);
        // Storage RTM: copy the interior of each stored level p^m once it
        // is current (before the step that overwrites p^{m-1} with p^{m+1}).
        auto keep = [&](int m) -> int {
            if (J.op != RTM_OP_STORAGE || m >= nt) return RTM_OK;
            const ShotIn &S = J.shots[0];
            if (m < S.phase || (m - S.phase) % S.stride != 0) return RTM_OK;
            const int64_t ncell = S.g.nx * S.g.ny * S.g.nz;
            RTM_HIP(launch_snap_store(SH(), 0, m & 1, ncell, S.snaps + (int64_t)((m - S.phase) / S.stride) * ncell,
                                      st));
            return RTM_OK;
        };
        int rc = RTM_OK;
        int n = 0;
        if (persist) {
            // every forward step in one launch; counters and status start at zero
            unsigned *cnt = D.at<unsigned>(J.ws.pcnt);
            RTM_HIP(launch_fill((float *)cnt, nsh + 1, 0.f, st));
            RTM_HIP(launch_fwd2d_persist(J.fw.tune.vec, SH(), tiles, D.at<PItem>(J.ws.pitems_f),
                                         (int)J.pitems_f.size(), D.at<int>(J.ws.pnum), ents, cont,
                                         sample ? stasks : nullptr, 0, nt, cnt, cnt + nsh, g_persist_wait_ms.load(),
                                         st));
            n = nt;
        }
        if (fs == 3) {
            // steps n .. n + 2 per launch; each launch records d^{n-2},
            // d^{n-1}, d^n (no stored levels: not for storage RTM)
            for (; n + 3 <= nt; n += 3) {
                RTM_HIP(launch_fwd2d_t3(J.fw2.tune.code(), SH(), D.at<Tile2D>(J.ws.tiles_f2), J.fw2.count(),
                                        J.fw2.nslots, D.at<InjEnt>(J.ws.ents_f2), D.at<Contrib>(J.ws.cont_f2),
                                        sample ? stasks : nullptr, nsample, n, st));
                cur ^= 1;
            }
            // the last launch's middle level (field 6 of the current table)
            // and level n - 1, which a one-step launch would overwrite
            if (sample && n >= 3) {
                RTM_HIP(launch_sample(SH(), stasks, nsample, n - 2, 6, st));
                RTM_HIP(launch_sample(SH(), stasks, nsample, n - 1, (n - 1) & 1, st));
            }
        } else if (two) {
            // steps n, n + 1 per launch; each launch records d^{n-1}, d^n
            for (; n + 2 <= nt; n += 2) {
                if ((rc = keep(n))) return rc;
                RTM_HIP(launch_fwd2d_t2(J.fw2.tune.code(), SH(), D.at<Tile2D>(J.ws.tiles_f2), J.fw2.count(),
                                        J.fw2.nslots, D.at<InjEnt>(J.ws.ents_f2), D.at<Contrib>(J.ws.cont_f2),
                                        sample ? stasks : nullptr, nsample, n, st));
                cur ^= 1;
                if ((rc = keep(n + 1))) return rc;
            }
            // an odd last step overwrites level n - 1: record it first
            if (sample && n < nt && n >= 1) RTM_HIP(launch_sample(SH(), stasks, nsample, n - 1, (n - 1) & 1, st));
        }
        for (; n < nt; ++n) {
            if ((rc = keep(n))) return rc;
            if (J.fw.ndim == 3)
                RTM_HIP(launch_fwd3d(J.fw.tune.code(), J.fw.tune.ty, SH(), (const Tile3D *)tiles, ntiles, J.fw.nslots,
                                     ents, cont, sample ? stasks : nullptr, nsample, n, st));
            else
                RTM_HIP(launch_fwd2d(J.fw.tune.vec, J.fw.tune.tx, SH(), tiles, ntiles, J.fw.nslots, ents, cont,
                                     sample ? stasks : nullptr, nsample, n, st));
        }
        timer.finish();
        if (sample) {
            if (fs == 2 && nt % 2 == 0 && nt >= 2)
                RTM_HIP(launch_sample(SH(), stasks, nsample, nt - 1, (nt - 1) & 1, st));
            RTM_HIP(launch_sample(SH(), stasks, nsample, nt, nt & 1, st));
        }
    }
    if (J.op == RTM_OP_MODEL) {
        RTM_HIP(launch_traces(table, nsh, maxrec, nt + 1, false, st));
        for (int i = 0; i < nsh; ++i) {
            const ShotIn &S = J.shots[i];
            if (S.p_last) RTM_HIP(launch_unpack(S.g.L, fld_of(i, nt & 1), S.p_last, st));
            if (S.p_prev) RTM_HIP(launch_unpack(S.g.L, fld_of(i, (nt + 1) & 1), S.p_prev, st));
        }
        return RTM_OK;
    }
    // Reverse pass (Algorithm 3): mu^{nt} = D' h^2 R^T g^{nt}, mu^{nt+1} = 0,
    // then one fused launch per step k = nt-1 .. 0 (or per pair of steps).
    const PassRange pass(J.op == RTM_OP_VJP ? "rtm:reverse_grad" : "rtm:reverse_image");
    const bool grad = J.op == RTM_OP_VJP;
    const Tile2D *tiles = D.at<Tile2D>(J.ws.tiles_r);
    const InjEnt *ents = D.at<InjEnt>(J.ws.ents_r);
    const Contrib *cont = D.at<Contrib>(J.ws.cont_r);
    RTM_HIP(launch_inj_set(SH(), ents, J.rv.nsrc_ent, J.rv.nsrc_ent + J.rv.nrec_ent, cont, nt, st));
    const int ntiles = J.rv.count();
    if (J.op == RTM_OP_STORAGE) {
        // Algorithm 2: the receiver wavefield alone, imaging at the stored levels.
        const ShotIn &S = J.shots[0];
        const int64_t ncell = S.g.nx * S.g.ny * S.g.nz;
        LoopTimer timer(kLoopRevImage, nt, st, timed);
        for (int k = nt - 1; k >= 0; --k) {
            const bool stored = k >= S.phase && (k - S.phase) % S.stride == 0;
            const float *snap = stored ? S.snaps + (int64_t)((k - S.phase) / S.stride) * ncell : nullptr;
            if (J.rv.ndim == 3)
                RTM_HIP(launch_recv3d(J.rv.tune.code(), J.rv.tune.ty, SH(), (const Tile3D *)tiles, ntiles, J.rv.nslots,
                                      ents, cont, k, snap, st));
            else
                RTM_HIP(launch_recv2d(J.rv.tune.vec, J.rv.tune.tx, SH(), tiles, ntiles, J.rv.nslots, ents, cont, k,
                                      snap, st));
        }
        timer.finish();
        unsigned *dmax = scal + 64 + 2 * J.slot_shot.size();
        RTM_HIP(launch_den_max(SH(), 1, S.g.ny * S.g.nz, S.g.nx, dmax, st));
        RTM_HIP(launch_image(SH(), 0, 1, S.g.ny * S.g.nz, S.g.nx, dmax, J.eps, S.image, 0, S.num, S.den, st));
        return RTM_OK;
    }
    const int reinject = (J.flags & RTM_F_NO_REINJECT) ? 0 : 1;
    const bool probing = probe && probe->snap_k >= 0;
    const bool two = J.rv.ndim == 2 && J.rv2.steps > 1 && !probing;
    const int rs = two ? J.rv2.steps : 1;
    // wadj is recorded for a single-shot job only (its kernel argument is one
    // buffer); batched VJPs do not return wavelet gradients.
    float *wadj = (grad && nsh == 1 && J.shots[0].grad_wavelet) ? D.at<float>(J.ws.wadj[0]) : nullptr;
    const bool persist = !J.pitems_f.empty() && !probing;
    LoopTimer timer(grad ? kLoopRevGrad : kLoopRevImage, persist ? 1 : nt / rs + nt % rs, st, timed && !probing);
    int k = nt - 1;
    if (persist) {
        // every reverse step in one launch; the status word keeps the forward pass's
        unsigned *cnt = D.at<unsigned>(J.ws.pcnt);
        RTM_HIP(launch_fill((float *)cnt, nsh, 0.f, st));
        RTM_HIP(launch_rev2d_persist(J.rv.tune.vec, grad, SH(), tiles, D.at<PItem>(J.ws.pitems_r),
                                     (int)J.pitems_r.size(), D.at<int>(J.ws.pnum) + nsh, ents, cont, nt - 1, nt,
                                     reinject, wadj, cnt, cnt + nsh, g_persist_wait_ms.load(), st));
        k = -1;
    }
    if (rs == 3) {
        for (; k >= 2; k -= 3) {
            const Tile2D *t2 = D.at<Tile2D>(J.ws.tiles_r2);
            const InjEnt *e2 = D.at<InjEnt>(J.ws.ents_r2);
            const Contrib *c2 = D.at<Contrib>(J.ws.cont_r2);
            if (grad)
                RTM_HIP(launch_rev2d_t3_grad(J.rv2.tune.code(), SH(), t2, J.rv2.count(), J.rv2.nslots, e2, c2, k, reinject,
                                             wadj, st));
            else
                RTM_HIP(launch_rev2d_t3(J.rv2.tune.code(), SH(), t2, J.rv2.count(), J.rv2.nslots, e2, c2, k, reinject, st));
            cur ^= 1;
        }
    } else if (two) {
        for (; k >= 1; k -= 2) {
            RTM_HIP(launch_rev2d_t2(J.rv2.tune.code(), grad, SH(), D.at<Tile2D>(J.ws.tiles_r2), J.rv2.count(),
                                    J.rv2.nslots, D.at<InjEnt>(J.ws.ents_r2), D.at<Contrib>(J.ws.cont_r2), k, reinject,
                                    wadj, st));
            cur ^= 1;
        }
    }
    for (; k >= 0; --k) {
        if (J.rv.ndim == 3)
            RTM_HIP(launch_rev3d(J.rv.tune.code(), J.rv.tune.ty, grad, SH(), (const Tile3D *)tiles, ntiles, J.rv.nslots,
                                 ents, cont, k, reinject, wadj, st));
        else
            RTM_HIP(launch_rev2d(J.rv.tune.vec, J.rv.tune.tx, grad, SH(), tiles, ntiles, J.rv.nslots, ents, cont, k,
                                 reinject, wadj, st));
        if (probing) {
            const ShotIn &S = J.shots[0];
            if (k - 1 == probe->snap_k && probe->snap_p)
                RTM_HIP(launch_unpack(S.g.L, fld_of(0, (k - 1) & 1), probe->snap_p, st));
            if (k == probe->snap_k && probe->snap_mu)
                RTM_HIP(launch_unpack(S.g.L, fld_of(0, 2 + (k & 1)), probe->snap_mu, st));
        }
    }
    timer.finish();
    // Finalisation: stream-ordered, so shots may share an image buffer; shots
    // in a row that do are added in one launch, in their order.
    if (grad) {
        for (int i = 0; i < nsh; ++i) {
            const ShotIn &S = J.shots[i];
            RTM_HIP(launch_grad(SH(), i, (int64_t)S.g.NX * S.g.NY * S.g.NZ, S.v_pad, (float)J.dt, S.grad_v_pad, st));
            if (S.grad_wavelet && nsh == 1)
                RTM_HIP(launch_wadj(D.at<float>(J.ws.wadj[i]), nt, (float)(1.0 / (S.g.h * S.g.h)), S.grad_wavelet, st));
        }
        return RTM_OK;
    }
    unsigned *dmax = scal + 64 + 2 * J.slot_shot.size();
    int64_t rows = 0, len = 0;
    for (const ShotIn &S : J.shots) {
        rows = std::max(rows, S.g.ny * S.g.nz);
        len = std::max(len, S.g.nx);
    }
    RTM_HIP(launch_den_max(SH(), nsh, rows, len, dmax, st));
    for (int i = 0, m; i < nsh; i += m) {
        const ShotIn &S = J.shots[i];
        auto joins = [&](const ShotIn &o) {
            return o.image == S.image && !o.num && !o.den && o.g.nx == S.g.nx && o.g.ny == S.g.ny && o.g.nz == S.g.nz;
        };
        for (m = 1; S.image && !S.num && !S.den && i + m < nsh && joins(J.shots[i + m]);) ++m;
        RTM_HIP(launch_image(SH(), i, m, S.g.ny * S.g.nz, S.g.nx, dmax, J.eps, S.image,
                             (J.flags & RTM_F_ACCUMULATE) ? 1 : 0, S.num, S.den, st));
    }
    return RTM_OK;
}

int check_ws(const Job &J, void *ws, size_t ws_bytes)
{
    if (!ws) return fail(RTM_EWORKSPACE, "workspace is NULL (%zu bytes needed)", J.ws.bytes);
    if (((uintptr_t)ws & 255) != 0) return fail(RTM_EWORKSPACE, "workspace must be 256-byte aligned");
    if (ws_bytes < J.ws.bytes) return fail(RTM_EWORKSPACE, "workspace of %zu bytes < %zu needed", ws_bytes, J.ws.bytes);
    return RTM_OK;
}

// Eager execution of a job (single-shot entry points and plans without a graph).
int job_run(Job &J, void *ws, size_t ws_bytes, hipStream_t st, const rtm_probe_t *probe)
{
    int rc = check_ws(J, ws, ws_bytes);
    if (rc) return rc;
    Dev D{(char *)ws};
    std::vector<ShotDev> shot_devs;
    if ((rc = job_upload_and_check(J, D, shot_devs, st))) return rc;
    if ((rc = job_launch(J, D, st, probe, true))) return rc;
    if (!(J.flags & RTM_F_CHECK_FINITE)) return RTM_OK;
    // Outputs checked for NaN / Inf: an unstable run (or a non-finite input
    // that the velocity check does not cover, such as the wavelet or the
    // traces) is reported instead of returned silently.
    unsigned *flag = D.at<unsigned>(J.ws.scal);
    RTM_HIP(launch_fill((float *)flag, 1, 0.f, st));  // zero bits
    for (const ShotIn &S : J.shots) {
        const int64_t ni = S.g.nx * S.g.ny * S.g.nz, np = (int64_t)S.g.NX * S.g.NY * S.g.NZ;
        if (J.op == RTM_OP_MODEL) RTM_HIP(launch_nonfinite(S.traces_out, (int64_t)S.nrec * (J.nt + 1), flag, st));
        if (has_den(J.op)) RTM_HIP(launch_nonfinite(S.image, ni, flag, st));
        if (J.op == RTM_OP_VJP) RTM_HIP(launch_nonfinite(S.grad_v_pad, np, flag, st));
    }
    unsigned h = 0;
    RTM_HIP(hipMemcpyAsync(&h, flag, sizeof h, hipMemcpyDeviceToHost, st));
    RTM_HIP(hipStreamSynchronize(st));
    if (h) return fail(RTM_ENUMERIC, "non-finite values in the output (unstable run or non-finite wavelet / traces)");
    return RTM_OK;
}

int check_common(const rtm_grid_t *grid, const float *v_pad, double dt, int32_t nt, const float *wavelet,
                 const float *src, int32_t nrec, const float *rec, GridInfo *g)
{
    int rc = grid_info(grid, g);
    if (rc) return rc;
    if (!v_pad) return fail(RTM_EINVAL, "v_pad is NULL");
    if (!(dt > 0.0) || !std::isfinite(dt)) return fail(RTM_EINVAL, "dt must be positive and finite");
    if (nt < 1) return fail(RTM_EINVAL, "nt must be >= 1");
    if (!wavelet) return fail(RTM_EINVAL, "wavelet is NULL");
    if (!src) return fail(RTM_EINVAL, "src is NULL");
    if (nrec < 1) return fail(RTM_EINVAL, "nrec must be >= 1");
    if (!rec) return fail(RTM_EINVAL, "rec is NULL");
    if ((int64_t)(nt + 1) * nrec >= ((int64_t)1 << 31)) return fail(RTM_EINVAL, "(nt + 1) * nrec too large");
    return RTM_OK;
}

// A one-shot job whose workspace layout uses position-independent bounds,
// so that rtm_workspace_bytes can size it without the acquisition.
int single_job(Job &J, int op, const GridInfo &g, const float *v_pad, double dt, int nt, const float *wavelet,
               const float *src, int nrec, const float *rec, uint32_t flags)
{
    J.op = op;
    J.nt = nt;
    J.dt = dt;
    J.flags = flags;
    ShotIn S;
    S.g = g;
    S.v_pad = v_pad;
    S.wavelet = wavelet;
    std::memcpy(S.src, src, sizeof S.src);
    S.nrec = nrec;
    S.rec.assign(rec, rec + 3 * (size_t)nrec);
    J.shots.push_back(std::move(S));
    int rc = build_job_tables(J);
    if (rc) return rc;
    J.ws = make_ws_layout(J, bound_counts(g, op, nrec));
    return RTM_OK;
}

size_t single_bytes(const GridInfo &g, int op, int nrec, int nt)
{
    Job J;
    J.op = op;
    J.nt = nt;
    ShotIn S;
    S.g = g;
    S.nrec = nrec;
    J.shots.push_back(S);
    J.slot_shot.push_back(0);
    J.dslot.push_back(0);
    return make_ws_layout(J, bound_counts(g, op, nrec)).bytes;
}

// Band options from the ABI struct: flags checked, taper table built on the
// host (Eqs. (4)-(5) in double, rounded once to FP32).
int band_opts(const GridInfo &g, const rtm_rbc_opts_t *o, BandOpts *b)
{
    std::memset(b, 0, sizeof *b);
    if (!o) return RTM_OK;
    if (o->flags & ~(RTM_RBC_TAPER | RTM_RBC_FREE_SURFACE)) return fail(RTM_EINVAL, "unknown band flags 0x%x", o->flags);
    b->flags = (o->flags & RTM_RBC_TAPER ? kBandTaper : 0u) | (o->flags & RTM_RBC_FREE_SURFACE ? kBandFreeSurface : 0u);
    if (o->flags & RTM_RBC_TAPER) {
        const double a = o->taper_alpha;
        if (!(a >= 0.0 && a <= 1.0)) return fail(RTM_EINVAL, "taper_alpha must be in [0, 1] (got %g)", a);
        if (g.nb > kMaxTaper) return fail(RTM_EINVAL, "taper needs nb <= %d (got %d)", kMaxTaper, g.nb);
        for (int i = 1; i <= g.nb; ++i) {
            if (g.nb == 1) {
                b->c[0] = 1.0f;
                break;
            }
            const double x = (double)i, n1 = (double)(g.nb - 1);
            const double lin = ((double)g.nb - x) / n1;                       // Eq. (4)
            const double gau = std::exp(-120.0 * (x - 1.0) * (x - 1.0) / (n1 * n1));  // Eq. (5)
            b->c[i - 1] = (float)(a * lin + (1.0 - a) * gau);
        }
    }
    return RTM_OK;
}

int pad_common(const rtm_grid_t *grid, const float *v_int, const rtm_rbc_opts_t *opts, const float *g_pad,
               float *out, void *ws, size_t ws_bytes, void *stream, bool adjoint)
{
    t_err.clear();
    GridInfo g;
    int rc = grid_info(grid, &g);
    if (rc) return rc;
    if (!v_int || !out || (adjoint && !g_pad)) return fail(RTM_EINVAL, "NULL array argument");
    if (!opts) return fail(RTM_EINVAL, "opts is NULL");
    BandOpts b;
    if ((rc = band_opts(g, opts, &b))) return rc;
    hipStream_t st = (hipStream_t)stream;
    const unsigned *cap_bits = nullptr;
    if (!(opts->v_cap > 0.f)) {
        if (!ws || ws_bytes < 256 || ((uintptr_t)ws & 255))
            return fail(RTM_EWORKSPACE, "v_cap <= 0 needs an aligned workspace of 256 bytes");
        RTM_HIP(launch_vmax(v_int, g.nx * g.ny * g.nz, (unsigned *)ws, st));
        cap_bits = (const unsigned *)ws;
    }
    if (adjoint)
        RTM_HIP(launch_pad_adjoint(g.ndim, g.nb, g.nx, g.ny, g.nz, v_int, opts->seed, opts->v_cap, cap_bits, b, g_pad,
                                   out, st));
    else
        RTM_HIP(launch_rbc_pad(g.ndim, g.nb, g.nx, g.ny, g.nz, v_int, opts->seed, opts->v_cap, cap_bits, b, out, st));
    return RTM_OK;
}

}  // namespace

// ===========================================================================
// Batch plans
// ===========================================================================

struct rtm_plan {
    Job job;
};

// ===========================================================================
// C ABI
// ===========================================================================

extern "C" {

int rtm_abi_version(void) { return RTM_ABI_VERSION; }

const char *rtm_last_error(void) { return t_err.c_str(); }

int rtm_set_tuning(int op, int vec, int zseg)
{
    if (op == RTM_TUNE_EXACT || op == 0) {
        g_tune_exact = (op == RTM_TUNE_EXACT) ? (vec != 0) : 0;
        return RTM_OK;
    }
    if (vec != 1 && vec != 2 && vec != 4) return fail(RTM_EINVAL, "vec must be 1, 2 or 4");
    if (zseg < kMinZseg || zseg > 4095 || zseg % kZUnroll != 0)
        return fail(RTM_EINVAL, "zseg must be a multiple of %d in [%d, 4095]", kZUnroll, kMinZseg);
    if (op != RTM_OP_MODEL && op != RTM_OP_RTM && op != RTM_OP_VJP) return fail(RTM_EINVAL, "unknown op %d", op);
    std::atomic<int> &g = op == RTM_OP_MODEL ? g_tune2d_fwd : g_tune2d_rev;
    g = (g.load() & ~0xffffff) | (vec << 16) | zseg;  // keeps the strips per workgroup
    return RTM_OK;
}

int rtm_set_tuning2d(int op, int vec, int tx, int zseg)
{
    if (vec != 1 && vec != 2 && vec != 4) return fail(RTM_EINVAL, "vec must be 1, 2 or 4");
    if (tx != 1 && tx != 2 && tx != 4) return fail(RTM_EINVAL, "tx must be 1, 2 or 4");
    if (zseg < kMinZseg || zseg > 4095 || zseg % kZUnroll != 0)
        return fail(RTM_EINVAL, "zseg must be a multiple of %d in [%d, 4095]", kZUnroll, kMinZseg);
    if (op != RTM_OP_MODEL && op != RTM_OP_RTM && op != RTM_OP_VJP) return fail(RTM_EINVAL, "unknown op %d", op);
    std::atomic<int> &g = op == RTM_OP_MODEL ? g_tune2d_fwd : g_tune2d_rev;
    g = (g.load() & (0x3 << 28)) | (tx << 24) | (vec << 16) | zseg;  // keeps the steps per launch
    return RTM_OK;
}

int rtm_set_steps_per_launch(int op, int steps)
{
    if (steps < 1 || steps > 3) return fail(RTM_EINVAL, "steps must be 1, 2 or 3");
    if (op != RTM_OP_MODEL && op != RTM_OP_RTM && op != RTM_OP_VJP) return fail(RTM_EINVAL, "unknown op %d", op);
    std::atomic<int> &g = op == RTM_OP_MODEL ? g_tune2d_fwd : g_tune2d_rev;
    g = (g.load() & ~(0x3 << 28)) | ((steps - 1) << 28);
    return RTM_OK;
}

int rtm_get_steps_per_launch(int op, int *steps)
{
    if (!steps) return fail(RTM_EINVAL, "NULL output");
    if (op != RTM_OP_MODEL && op != RTM_OP_RTM && op != RTM_OP_VJP) return fail(RTM_EINVAL, "unknown op %d", op);
    *steps = get_tune(op == RTM_OP_MODEL ? 0 : 1, 2).steps;
    return RTM_OK;
}

int rtm_get_tuning2d(int op, int *vec, int *tx, int *zseg)
{
    if (!vec || !tx || !zseg) return fail(RTM_EINVAL, "NULL output");
    if (op != RTM_OP_MODEL && op != RTM_OP_RTM && op != RTM_OP_VJP) return fail(RTM_EINVAL, "unknown op %d", op);
    Tune t = get_tune(op == RTM_OP_MODEL ? 0 : 1, 2);
    *vec = t.vec;
    *tx = t.tx;
    *zseg = t.zseg;
    return RTM_OK;
}

int rtm_set_tuning3d(int op, int vec, int ty, int zseg)
{
    if (vec != 1 && vec != 2 && vec != 4) return fail(RTM_EINVAL, "vec must be 1, 2 or 4");
    if (ty != 4 && ty != 8 && ty != 16) return fail(RTM_EINVAL, "ty must be 4, 8 or 16");
    // 16-row workgroups (1024 threads, at most 128 registers a lane): the
    // forward update at vec 1 or 2, the fused reverse at vec 1 only.
    if (ty == 16 && (vec > 2 || (op != RTM_OP_MODEL && vec != 1)))
        return fail(RTM_EINVAL, "ty 16 needs vec 1 (reverse) or vec <= 2 (forward)");
    if (zseg < kMinZseg || zseg > 4095 || zseg % kZUnroll != 0)
        return fail(RTM_EINVAL, "zseg must be a multiple of %d in [%d, 4095]", kZUnroll, kMinZseg);
    if (op != RTM_OP_MODEL && op != RTM_OP_RTM && op != RTM_OP_VJP) return fail(RTM_EINVAL, "unknown op %d", op);
    std::atomic<int> &g = op == RTM_OP_MODEL ? g_tune3d_fwd : g_tune3d_rev;
    g = (vec << 24) | (ty << 16) | (g.load() & (1 << 15)) | zseg;  // the tile order is kept
    return RTM_OK;
}

int rtm_set_tile_order3d(int op, int z_inner)
{
    if (z_inner != 0 && z_inner != 1) return fail(RTM_EINVAL, "z_inner must be 0 or 1");
    if (op != RTM_OP_MODEL && op != RTM_OP_RTM && op != RTM_OP_VJP) return fail(RTM_EINVAL, "unknown op %d", op);
    std::atomic<int> &g = op == RTM_OP_MODEL ? g_tune3d_fwd : g_tune3d_rev;
    g = (g.load() & ~(1 << 15)) | (z_inner << 15);
    return RTM_OK;
}

int rtm_get_tile_order3d(int op, int *z_inner)
{
    if (!z_inner) return fail(RTM_EINVAL, "NULL output");
    if (op != RTM_OP_MODEL && op != RTM_OP_RTM && op != RTM_OP_VJP) return fail(RTM_EINVAL, "unknown op %d", op);
    *z_inner = get_tune(op == RTM_OP_MODEL ? 0 : 1, 3).zin;
    return RTM_OK;
}

int rtm_get_tuning3d(int op, int *vec, int *ty, int *zseg)
{
    if (!vec || !ty || !zseg) return fail(RTM_EINVAL, "NULL output");
    if (op != RTM_OP_MODEL && op != RTM_OP_RTM && op != RTM_OP_VJP) return fail(RTM_EINVAL, "unknown op %d", op);
    Tune t = get_tune(op == RTM_OP_MODEL ? 0 : 1, 3);
    *vec = t.vec;
    *ty = t.ty;
    *zseg = t.zseg;
    return RTM_OK;
}

int rtm_get_tuning(int op, int *vec, int *zseg)
{
    if (!vec || !zseg) return fail(RTM_EINVAL, "NULL output");
    if (op == RTM_TUNE_EXACT) {
        *vec = g_tune_exact.load();
        *zseg = 0;
        return RTM_OK;
    }
    if (op != RTM_OP_MODEL && op != RTM_OP_RTM && op != RTM_OP_VJP) return fail(RTM_EINVAL, "unknown op %d", op);
    Tune t = get_tune(op == RTM_OP_MODEL ? 0 : 1, 2);
    *vec = t.vec;
    *zseg = t.zseg;
    return RTM_OK;
}

int rtm_set_persist_wait(double ms)
{
    if (!(ms >= 0.0) || !(ms <= 3.6e6)) return fail(RTM_EINVAL, "wait limit must be in [0, 3.6e6] ms");
    g_persist_wait_ms = ms;
    return RTM_OK;
}

int rtm_get_persist_wait(double *ms)
{
    if (!ms) return fail(RTM_EINVAL, "NULL output");
    *ms = g_persist_wait_ms.load();
    return RTM_OK;
}

int rtm_timing_enable(int on)
{
    g_timing_on = on ? 1 : 0;
    return RTM_OK;
}

int rtm_timing_read(double *ms, int64_t *launches)
{
    if (!ms || !launches) return fail(RTM_EINVAL, "NULL output");
    for (int k = 0; k < kLoopKinds; ++k) {
        ms[k] = 0.0;
        launches[k] = 0;
    }
    std::vector<PendingTiming> pend;
    {
        std::lock_guard<std::mutex> lk(g_timing_mu);
        pend.swap(g_timing_pending);
    }
    int rc = RTM_OK;
    for (auto &p : pend) {
        float t = 0.f;
        hipError_t e = hipEventSynchronize(p.stop);
        if (e == hipSuccess) e = hipEventElapsedTime(&t, p.start, p.stop);
        if (e == hipSuccess) {
            ms[p.kind] += t;
            launches[p.kind] += p.launches;
        } else {
            rc = fail(RTM_EHIP, "event timing: %s", hipGetErrorString(e));
        }
        (void)hipEventDestroy(p.start);
        (void)hipEventDestroy(p.stop);
    }
    return rc;
}

int rtm_workspace_bytes(const rtm_grid_t *grid, int op, int32_t nrec, int32_t nt, size_t *bytes)
{
    t_err.clear();
    GridInfo g;
    int rc = grid_info(grid, &g);
    if (rc) return rc;
    if (!bytes) return fail(RTM_EINVAL, "bytes is NULL");
    if (op < RTM_OP_RBC_PAD || op > RTM_OP_STORAGE) return fail(RTM_EINVAL, "unknown op %d", op);
    if (op == RTM_OP_RBC_PAD) {
        *bytes = 256;
        return RTM_OK;
    }
    if (nrec < 1 || nt < 1) return fail(RTM_EINVAL, "nrec and nt must be >= 1");
    *bytes = single_bytes(g, op, nrec, nt);
    return RTM_OK;
}

int rtm_rbc_pad_ex(const rtm_grid_t *grid, const float *v_int, const rtm_rbc_opts_t *opts, float *v_pad, void *ws,
                   size_t ws_bytes, void *stream)
{
    return pad_common(grid, v_int, opts, nullptr, v_pad, ws, ws_bytes, stream, false);
}

int rtm_pad_adjoint_ex(const rtm_grid_t *grid, const float *v_int, const rtm_rbc_opts_t *opts, const float *grad_v_pad,
                       float *grad_v_int, void *ws, size_t ws_bytes, void *stream)
{
    return pad_common(grid, v_int, opts, grad_v_pad, grad_v_int, ws, ws_bytes, stream, true);
}

int rtm_rbc_pad(const rtm_grid_t *grid, const float *v_int, uint64_t seed, float v_cap, float *v_pad, void *ws,
                size_t ws_bytes, void *stream)
{
    const rtm_rbc_opts_t o{seed, v_cap, 0u, 0.0};
    return pad_common(grid, v_int, &o, nullptr, v_pad, ws, ws_bytes, stream, false);
}

int rtm_pad_adjoint(const rtm_grid_t *grid, const float *v_int, uint64_t seed, float v_cap, const float *grad_v_pad,
                    float *grad_v_int, void *ws, size_t ws_bytes, void *stream)
{
    const rtm_rbc_opts_t o{seed, v_cap, 0u, 0.0};
    return pad_common(grid, v_int, &o, grad_v_pad, grad_v_int, ws, ws_bytes, stream, true);
}

int rtm_model_shot(const rtm_grid_t *grid, const float *v_pad, double dt, int32_t nt, const float *wavelet,
                   const float *src, int32_t nrec, const float *rec, float *traces, float *p_last, float *p_prev,
                   uint32_t flags, void *ws, size_t ws_bytes, void *stream)
{
    t_err.clear();
    GridInfo g;
    int rc = check_common(grid, v_pad, dt, nt, wavelet, src, nrec, rec, &g);
    if (rc) return rc;
    if (!traces) return fail(RTM_EINVAL, "traces is NULL");
    Job J;
    if ((rc = single_job(J, RTM_OP_MODEL, g, v_pad, dt, nt, wavelet, src, nrec, rec, flags))) return rc;
    J.shots[0].traces_out = traces;
    J.shots[0].p_last = p_last;
    J.shots[0].p_prev = p_prev;
    return job_run(J, ws, ws_bytes, (hipStream_t)stream, nullptr);
}

int rtm_rtm_shot(const rtm_grid_t *grid, const float *v_pad, double dt, int32_t nt, const float *wavelet,
                 const float *src, int32_t nrec, const float *rec, const float *traces, float eps_rel, float *image,
                 float *num, float *den, const rtm_probe_t *probe, uint32_t flags, void *ws, size_t ws_bytes,
                 void *stream)
{
    t_err.clear();
    GridInfo g;
    int rc = check_common(grid, v_pad, dt, nt, wavelet, src, nrec, rec, &g);
    if (rc) return rc;
    if (!traces) return fail(RTM_EINVAL, "traces is NULL");
    if (!image) return fail(RTM_EINVAL, "image is NULL");
    if (!(eps_rel >= 0.f) || !std::isfinite(eps_rel)) return fail(RTM_EINVAL, "eps_rel must be finite and >= 0");
    if (probe && probe->snap_k >= 0 && probe->snap_k > nt - 2)
        return fail(RTM_EINVAL, "probe step %d outside [0, nt - 2]", (int)probe->snap_k);
    Job J;
    if ((rc = single_job(J, RTM_OP_RTM, g, v_pad, dt, nt, wavelet, src, nrec, rec, flags & ~RTM_F_ACCUMULATE)))
        return rc;
    J.eps = eps_rel;
    J.shots[0].traces_in = traces;
    J.shots[0].image = image;
    J.shots[0].num = num;
    J.shots[0].den = den;
    return job_run(J, ws, ws_bytes, (hipStream_t)stream, probe);
}

int rtm_nyquist_stride(double dt, double f_max, double f_min, int32_t *stride)
{
    t_err.clear();
    if (!stride) return fail(RTM_EINVAL, "stride is NULL");
    if (!(dt > 0.0) || !std::isfinite(dt)) return fail(RTM_EINVAL, "dt must be positive and finite");
    if (!(f_min >= 0.0) || !(f_max > f_min) || !std::isfinite(f_max))
        return fail(RTM_EINVAL, "need 0 <= f_min < f_max, finite (got %g, %g)", f_min, f_max);
    // Eq. (7); the small allowance keeps exact ratios such as 5 ms / 0.5 ms at 10
    const double ratio = 1.0 / (2.0 * (f_max - f_min) * dt);
    const double steps = std::floor(ratio * (1.0 + 1e-12));
    *stride = (int32_t)std::max(1.0, std::min(steps, 1073741824.0));
    return RTM_OK;
}

int rtm_storage_count(int32_t nt, int32_t stride, int32_t phase, int64_t *count)
{
    t_err.clear();
    if (!count) return fail(RTM_EINVAL, "count is NULL");
    if (nt < 1) return fail(RTM_EINVAL, "nt must be >= 1");
    if (stride < 1 || phase < 0 || phase >= stride)
        return fail(RTM_EINVAL, "need stride >= 1 and 0 <= phase < stride (got %d, %d)", (int)stride, (int)phase);
    *count = phase < nt ? (int64_t)(nt - 1 - phase) / stride + 1 : 0;
    return RTM_OK;
}

int rtm_storage_shot(const rtm_grid_t *grid, const float *v_pad, double dt, int32_t nt, const float *wavelet,
                     const float *src, int32_t nrec, const float *rec, const float *traces, int32_t stride,
                     int32_t phase, float eps_rel, float *image, float *num, float *den, float *snapshots,
                     size_t snapshot_bytes, uint32_t flags, void *ws, size_t ws_bytes, void *stream)
{
    t_err.clear();
    GridInfo g;
    int rc = check_common(grid, v_pad, dt, nt, wavelet, src, nrec, rec, &g);
    if (rc) return rc;
    if (!traces) return fail(RTM_EINVAL, "traces is NULL");
    if (!image) return fail(RTM_EINVAL, "image is NULL");
    if (!(eps_rel >= 0.f) || !std::isfinite(eps_rel)) return fail(RTM_EINVAL, "eps_rel must be finite and >= 0");
    int64_t count = 0;
    if ((rc = rtm_storage_count(nt, stride, phase, &count))) return rc;
    const int64_t ncell = g.nx * g.ny * g.nz;
    if (count > 0 && !snapshots) return fail(RTM_EINVAL, "snapshots is NULL");
    if ((double)count * (double)ncell * 4.0 > (double)snapshot_bytes)
        return fail(RTM_EINVAL, "snapshots: %lld levels of %lld cells need %.0f bytes, %zu given", (long long)count,
                    (long long)ncell, (double)count * (double)ncell * 4.0, snapshot_bytes);
    if (flags & ~(RTM_F_SKIP_CHECK | RTM_F_CHECK_FINITE))
        return fail(RTM_EINVAL, "unsupported flags 0x%x", (unsigned)flags);
    Job J;
    if ((rc = single_job(J, RTM_OP_STORAGE, g, v_pad, dt, nt, wavelet, src, nrec, rec, flags))) return rc;
    J.eps = eps_rel;
    ShotIn &S = J.shots[0];
    S.traces_in = traces;
    S.image = image;
    S.num = num;
    S.den = den;
    S.snaps = snapshots;
    S.stride = stride;
    S.phase = phase;
    return job_run(J, ws, ws_bytes, (hipStream_t)stream, nullptr);
}

int rtm_model_shot_vjp(const rtm_grid_t *grid, const float *v_pad, double dt, int32_t nt, const float *wavelet,
                       const float *src, int32_t nrec, const float *rec, const float *grad_traces, float *grad_v_pad,
                       float *grad_wavelet, uint32_t flags, void *ws, size_t ws_bytes, void *stream)
{
    t_err.clear();
    GridInfo g;
    int rc = check_common(grid, v_pad, dt, nt, wavelet, src, nrec, rec, &g);
    if (rc) return rc;
    if (!grad_traces) return fail(RTM_EINVAL, "grad_traces is NULL");
    if (!grad_v_pad) return fail(RTM_EINVAL, "grad_v_pad is NULL");
    Job J;
    if ((rc = single_job(J, RTM_OP_VJP, g, v_pad, dt, nt, wavelet, src, nrec, rec, flags & ~RTM_F_NO_REINJECT)))
        return rc;
    J.shots[0].traces_in = grad_traces;
    J.shots[0].grad_v_pad = grad_v_pad;
    J.shots[0].grad_wavelet = grad_wavelet;
    return job_run(J, ws, ws_bytes, (hipStream_t)stream, nullptr);
}

int rtm_batch_plan(int op, int32_t nshots, const rtm_shot_desc_t *descs, double dt, int32_t nt, float eps_rel,
                   uint32_t flags, rtm_plan_t **plan, size_t *ws_bytes)
{
    t_err.clear();
    if (!plan || !ws_bytes) return fail(RTM_EINVAL, "plan and ws_bytes must be non-NULL");
    *plan = nullptr;
    if (op != RTM_OP_MODEL && op != RTM_OP_RTM && op != RTM_OP_VJP) return fail(RTM_EINVAL, "unknown op %d", op);
    if (nshots < 1 || !descs) return fail(RTM_EINVAL, "need at least one shot");
    if (!(dt > 0.0) || !std::isfinite(dt)) return fail(RTM_EINVAL, "dt must be positive and finite");
    if (nt < 1) return fail(RTM_EINVAL, "nt must be >= 1");
    if (op == RTM_OP_RTM && (!(eps_rel >= 0.f) || !std::isfinite(eps_rel)))
        return fail(RTM_EINVAL, "eps_rel must be finite and >= 0");
    if ((flags & RTM_F_PERSISTENT) && (flags & RTM_F_GRAPH))
        return fail(RTM_EINVAL, "RTM_F_PERSISTENT checks its run's status and cannot be combined with RTM_F_GRAPH");
    if ((flags & RTM_F_PERSISTENT) && descs[0].grid.ndim != 2)
        return fail(RTM_EINVAL, "RTM_F_PERSISTENT is implemented for 2-D shots");
    rtm_plan *P = new (std::nothrow) rtm_plan;
    if (!P) return fail(RTM_EINVAL, "out of host memory");
    Job &J = P->job;
    J.op = op;
    J.nt = nt;
    J.dt = dt;
    J.eps = eps_rel;
    J.flags = flags;
    for (int s = 0; s < nshots; ++s) {
        const rtm_shot_desc_t &d = descs[s];
        ShotIn S;
        int rc = grid_info(&d.grid, &S.g);
        if (!rc && s > 0 && S.g.ndim != J.shots[0].g.ndim)
            rc = fail(RTM_EINVAL, "shot %d: all shots of a batch must have the same dimension", s);
        if (!rc && (!d.v_pad || !d.wavelet)) rc = fail(RTM_EINVAL, "shot %d: v_pad and wavelet are required", s);
        if (!rc && (d.nrec < 1 || !d.rec)) rc = fail(RTM_EINVAL, "shot %d: at least one receiver is required", s);
        if (!rc && (int64_t)(nt + 1) * d.nrec >= ((int64_t)1 << 31)) rc = fail(RTM_EINVAL, "shot %d: too many samples", s);
        if (!rc && op == RTM_OP_MODEL && !d.traces_out) rc = fail(RTM_EINVAL, "shot %d: traces_out is required", s);
        if (!rc && op != RTM_OP_MODEL && !d.traces_in) rc = fail(RTM_EINVAL, "shot %d: traces_in is required", s);
        if (!rc && op == RTM_OP_RTM && !d.image) rc = fail(RTM_EINVAL, "shot %d: image is required", s);
        if (!rc && op == RTM_OP_VJP && !d.grad_v_pad) rc = fail(RTM_EINVAL, "shot %d: grad_v_pad is required", s);
        if (rc) {
            delete P;
            return rc;
        }
        S.v_pad = d.v_pad;
        S.wavelet = d.wavelet;
        std::memcpy(S.src, d.src, sizeof S.src);
        S.nrec = d.nrec;
        S.rec.assign(d.rec, d.rec + 3 * (size_t)d.nrec);
        S.traces_in = d.traces_in;
        S.traces_out = d.traces_out;
        S.image = d.image;
        S.grad_v_pad = d.grad_v_pad;
        J.shots.push_back(std::move(S));
    }
    int rc = build_job_tables(J);
    if (rc) {
        delete P;
        return rc;
    }
    J.ws = make_ws_layout(J, exact_counts(J));
    *ws_bytes = J.ws.bytes;
    *plan = P;
    return RTM_OK;
}

int rtm_batch_run(rtm_plan_t *plan, void *ws, size_t ws_bytes, void *stream)
{
    t_err.clear();
    if (!plan) return fail(RTM_EINVAL, "plan is NULL");
    Job &J = plan->job;
    hipStream_t st = (hipStream_t)stream;
    int rc = check_ws(J, ws, ws_bytes);
    if (rc) return rc;
    Dev D{(char *)ws};
    std::vector<ShotDev> shot_devs;
    if ((rc = job_upload_and_check(J, D, shot_devs, st))) return rc;
    if (J.flags & RTM_F_PERSISTENT) {
        if ((rc = job_launch(J, D, st, nullptr, true))) return rc;
        unsigned status = 0;
        RTM_HIP(hipMemcpyAsync(&status, D.at<unsigned>(J.ws.pcnt) + J.shots.size(), sizeof status,
                               hipMemcpyDeviceToHost, st));
        RTM_HIP(hipStreamSynchronize(st));
        if (status)
            return fail(RTM_EHIP, "persistent run stopped: a workgroup waited more than %g ms for its shot's "
                                  "previous step (not all workgroups resident?); outputs are invalid",
                        g_persist_wait_ms.load());
        return RTM_OK;
    }
    if (!(J.flags & RTM_F_GRAPH)) return job_launch(J, D, st, nullptr, true);
    if (!st) return fail(RTM_EINVAL, "RTM_F_GRAPH needs a non-NULL stream (the NULL stream cannot be captured)");
    if (J.gexec && (J.g_ws != ws || J.g_st != st)) {
        (void)hipGraphExecDestroy(J.gexec);
        J.gexec = nullptr;
    }
    if (!J.gexec) {
        hipGraph_t graph = nullptr;
        RTM_HIP(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal));
        rc = job_launch(J, D, st, nullptr, false);
        hipError_t e = hipStreamEndCapture(st, &graph);
        if (rc) {
            if (graph) (void)hipGraphDestroy(graph);
            return rc;
        }
        if (e != hipSuccess) return fail(RTM_EHIP, "hipStreamEndCapture: %s", hipGetErrorString(e));
        e = hipGraphInstantiate(&J.gexec, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e != hipSuccess) {
            J.gexec = nullptr;
            return fail(RTM_EHIP, "hipGraphInstantiate: %s", hipGetErrorString(e));
        }
        J.g_ws = ws;
        J.g_st = st;
    }
    RTM_HIP(hipGraphLaunch(J.gexec, st));
    return RTM_OK;
}

int rtm_window_extract(int64_t nz, int64_t nx_global, int64_t x0, int64_t width, const float *global, float *window,
                       void *stream)
{
    t_err.clear();
    if (nz < 1 || nx_global < 1 || width < 1 || x0 < 0 || x0 + width > nx_global)
        return fail(RTM_EINVAL, "window [%lld, %lld) outside [0, %lld)", (long long)x0, (long long)(x0 + width),
                    (long long)nx_global);
    if (!global || !window) return fail(RTM_EINVAL, "NULL array");
    RTM_HIP(launch_window((float *)global, nullptr, window, nz, nx_global, x0, width, 0, (hipStream_t)stream));
    return RTM_OK;
}

int rtm_window_accumulate(int64_t nz, int64_t nx_global, int64_t x0, int64_t width, const float *window,
                          float *global, void *stream)
{
    t_err.clear();
    if (nz < 1 || nx_global < 1 || width < 1 || x0 < 0 || x0 + width > nx_global)
        return fail(RTM_EINVAL, "window [%lld, %lld) outside [0, %lld)", (long long)x0, (long long)(x0 + width),
                    (long long)nx_global);
    if (!global || !window) return fail(RTM_EINVAL, "NULL array");
    RTM_HIP(launch_window(global, window, nullptr, nz, nx_global, x0, width, 1, (hipStream_t)stream));
    return RTM_OK;
}

int rtm_misfit_ws_bytes(size_t *bytes)
{
    if (!bytes) return fail(RTM_EINVAL, "bytes is NULL");
    *bytes = align256(misfit_ws_bytes());
    return RTM_OK;
}

int rtm_l2_misfit(int64_t n, const float *d, const float *d_obs, float *residual, double *J, void *ws,
                  size_t ws_bytes, void *stream)
{
    t_err.clear();
    if (n < 1 || !d || !d_obs || !J) return fail(RTM_EINVAL, "bad arguments");
    if (!ws || ws_bytes < misfit_ws_bytes() || ((uintptr_t)ws & 255))
        return fail(RTM_EWORKSPACE, "misfit workspace of %zu aligned bytes needed", misfit_ws_bytes());
    RTM_HIP(launch_misfit(d, d_obs, residual, n, ws, J, (hipStream_t)stream));
    return RTM_OK;
}

int rtm_stream_copy(const void *src, void *dst, size_t bytes, int blocks_per_cu, void *stream)
{
    t_err.clear();
    if (!src || !dst) return fail(RTM_EINVAL, "NULL buffer");
    if (((uintptr_t)src & 15) || ((uintptr_t)dst & 15) || (bytes & 15))
        return fail(RTM_EINVAL, "buffers and size must be multiples of 16 bytes");
    if (blocks_per_cu < 1 || blocks_per_cu > 64) return fail(RTM_EINVAL, "blocks_per_cu must be in [1, 64]");
    const uintptr_t a = (uintptr_t)src, b = (uintptr_t)dst;
    if (a < b + bytes && b < a + bytes && bytes > 0) return fail(RTM_EINVAL, "buffers overlap");
    RTM_HIP(launch_stream_copy(src, dst, (int64_t)(bytes / 16), blocks_per_cu, (hipStream_t)stream));
    return RTM_OK;
}

int rtm_batch_shape(const rtm_plan_t *plan, int reverse, rtm_launch_shape_t *shape)
{
    t_err.clear();
    if (!plan || !shape) return fail(RTM_EINVAL, "plan and shape must be non-NULL");
    if (reverse != 0 && reverse != 1) return fail(RTM_EINVAL, "reverse must be 0 or 1");
    const Job &J = plan->job;
    if (reverse && J.op == RTM_OP_MODEL) return fail(RTM_EINVAL, "a modeling plan has no reverse pass");
    const Tiling &one = reverse ? J.rv : J.fw, &multi = reverse ? J.rv2 : J.fw2;
    const Tiling &T = multi.steps > 1 ? multi : one;  // as job_launch chooses
    *shape = rtm_launch_shape_t{T.steps, T.tune.vec, T.tune.zseg, T.ndim == 3 ? T.tune.ty : 1,
                                T.ndim == 2 && T.steps == 1 ? T.tune.tx : 1, kBlockShapes[T.tune.block].waves,
                                T.tune.once ? 1 : 0, T.count()};
    return RTM_OK;
}

int rtm_batch_free(rtm_plan_t *plan)
{
    if (!plan) return RTM_OK;
    if (plan->job.gexec) (void)hipGraphExecDestroy(plan->job.gexec);
    delete plan;
    return RTM_OK;
}

}  // extern "C"
