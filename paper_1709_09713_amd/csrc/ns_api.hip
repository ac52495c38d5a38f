// ns_api.hip -- the C ABI (include/ns_tgv.h): argument validation,
// workspace layout and the per-step launch sequence of the three algorithm
// classes.  Every call validates first and enqueues nothing on failure.
#include <cmath>
#include <cstring>

#include "ns_common.hpp"
#include "ns_kernels.hpp"

namespace ns {

Consts make_consts(const ns_params *p)
{
    Consts c;
    c.nx = p->n[0];
    c.ny = p->n[1];
    c.nz = p->n[2];
    c.nxy = c.nx * c.ny;
    c.N = (int64_t)c.nxy * c.nz;
    double h[3];
    for (int d = 0; d < 3; ++d) {
        h[d] = p->length[d] / p->n[d];
        c.c1[d] = 1.0 / (12.0 * h[d]);
        c.c2[d] = 1.0 / (12.0 * h[d] * h[d]);
    }
    c.gm1 = p->gamma - 1.0;
    c.gM2 = p->gamma * p->mach * p->mach;
    c.inv_re = 1.0 / p->reynolds;   // 0 for +INFINITY
    c.kappa = 1.0 / (c.gm1 * p->mach * p->mach * p->prandtl * p->reynolds);
    c.rho_ref = 1.0;
    c.p_ref = 1.0 / c.gM2;
    c.rhoE_ref = c.p_ref / c.gm1;
    c.H_ref = c.rhoE_ref + c.p_ref;
    c.vol = h[0] * h[1] * h[2];
    c.inv_npts = 1.0 / (double)c.N;
    return c;
}


constexpr int kMinZChunk = 1;
// Launch settings of ns_set_fused_config / ns_set_fused_order: one copy per
// calling thread, so threads that drive solves of different shapes do not
// see each other's settings.
static thread_local int g_tile = -1;
static thread_local int g_zchunk = 0;
static thread_local int g_order = 0;

// Default z-chunk: a block marches zchunk + 4 planes (+ 5 for the
// tiles 8-10), and the grid runs in ceil(blocks / resident) rounds of
// resident blocks, so the time of a stage goes as rounds x planes.  Pick the
// number of chunks along z that minimises it (fewest blocks on a tie), and
// return that cost too.
static int zchunk_for(const Consts &c, int tile, int64_t resident, int64_t *cost_out)
{
    int bx, by;
    tile_dims(tile, &bx, &by);
    const int64_t nxy = (int64_t)((c.nx + bx - 1) / bx) * ((c.ny + by - 1) / by);
    int best_z = c.nz;
    int64_t best_cost = -1;
    // k chunks of z planes, for each z the smallest k
    for (int k = 1;;) {
        const int z = (c.nz + k - 1) / k;
        const int64_t rounds = (k * nxy + resident - 1) / resident;
        const int64_t planes = z + fused_extra_planes(tile);
        const int64_t cost = rounds * planes;
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best_z = z;
        }
        if (z <= kMinZChunk) break;
        k = (c.nz + z - 2) / (z - 1);
    }
    if (cost_out) *cost_out = best_cost;
    return best_z;
}

// Blocks of a tile that the device holds at once (512 on MI355X for the
// one-thread tiles of FP32 storage, 256 for 32x8 in three groups); when the
// device cannot be queried, 512 is assumed.
static int64_t resident_blocks(ns_precision prec, int tile)
{
    const int r = fused_resident_blocks(prec, tile);
    return r > 0 ? r : 512;
}

static int default_zchunk(const Consts &c, ns_precision prec, int tile)
{
    return zchunk_for(c, tile, resident_blocks(prec, tile), nullptr);
}

// Compute units of the current device: the blocks it holds of the 32x8
// three-group kernel, one each.
static int64_t compute_units()
{
    const int r = fused_resident_blocks(NS_FP64, TILE_32x8_3G);
    return r > 0 ? r : 256;
}

// FP64 on grids that leave most compute units with one block: a plane of a
// 16x8 block takes about two thirds of the time of a plane of a 32x8 block,
// so the narrow tile is faster where one block per compute unit and its longer
// chunks still come to less.  Measured, 16x8 | 32x8, us per RK3 step: 48^3
// 32.6 | 39.1, 56^3 43.6 | 46.4, 64^3 48.3 | 49.5, 80^3 75.0 | 75.7, 88^3
// 119.1 | 96.1, 96^3 126.9 | 104.1, 101x77x53 95.5 | 75.8, 200x20x20 33.7 |
// 36.1.  Both give the same bits.
static int default_fp64_tile(const Consts &c, int *zchunk)
{
    const int64_t cus = compute_units();
    int64_t narrow, wide;
    const int z9 = zchunk_for(c, TILE_32x8_3G, cus, &wide);
    if (fused_num_blocks(c, TILE_16x8_3G, c.nz) <= cus) {
        const int z8 = zchunk_for(c, TILE_16x8_3G, cus, &narrow);
        if (fused_num_blocks(c, TILE_16x8_3G, z8) <= cus && 2 * narrow < 3 * wide) {
            *zchunk = z8;
            return TILE_16x8_3G;
        }
    }
    *zchunk = z9;
    return TILE_32x8_3G;
}

// FP32 storage: a plane of the one-thread 32x8 kernel, two blocks a compute
// unit, takes 2.0 us, one of the three-group kernel, one block a compute unit,
// 1.2 us, so that kernel is taken where its longer chunks come to at most 1.8
// times the planes (not 2.0/1.2: on larger grids, which memory bounds, the
// one-thread kernel's second block hides more).  Of the cubes that bricks do not
// take, 49^3 to 96^3, 113^3 to 116^3 and 121^3 to 124^3.  Measured, one thread |
// three groups, us per RK3 step: 56^3 40.1 | 37.4, 64^3 42.7 | 40.2, 80^3 63.9 |
// 62.2, 88^3 76.3 | 79.0, 101x77x53 66.5 | 63.0, 96^3 84.3 | 82.1, 104^3 126.0 |
// 125.1, 112^3 131.0 | 136.1, 114^3 160.6 | 151.8, 122^3 187 | 179, 128^3 168.4 |
// 171.3, 144^3 279 | 297, 160^3 298 | 340, 256^3 1113 | 1234.  Both give the same bits; the
// direction-grouped order is compiled for the one-thread kernel only.
static int default_fp32_tile(const Consts &c, int *zchunk)
{
    int64_t one = 0, three = 0;
    const int z0 = zchunk_for(c, TILE_32x8, resident_blocks(NS_FP32_STORE, TILE_32x8), &one);
    const int z9 = zchunk_for(c, TILE_32x8_3G, resident_blocks(NS_FP32_STORE, TILE_32x8_3G), &three);
    if (g_order == 0 && 5 * three <= 9 * one) {
        *zchunk = z9;
        return TILE_32x8_3G;
    }
    *zchunk = z0;
    return TILE_32x8;
}

// Launch shape: an explicit tile (>= 0) / zchunk (> 0) wins, else the
// calling thread's setting of ns_set_fused_config, else the default.
static void choose_config(const Consts &c, ns_precision prec, int tile_in, int zchunk_in, int *tile,
                          int *zchunk)
{
    int t = tile_in >= 0 ? tile_in : g_tile;
    int z = tile_in >= 0 ? zchunk_in : g_zchunk;
    if (zchunk_in > 0) z = zchunk_in;
    // defaults measured on MI355X: FP64 runs fastest with the three-group
    // kernel on grids from 40^3 to 512^3; FP32 storage takes it on grids of about
    // a block a compute unit (default_fp32_tile), else the one-thread 32x8 kernel
    if (t < 0 || t >= TILE_COUNT) {
        if (z <= 0)
            t = prec == NS_FP64 ? default_fp64_tile(c, &z) : default_fp32_tile(c, &z);
        else
            t = (prec == NS_FP64) ? TILE_32x8_3G : TILE_32x8;
    }
    if (z <= 0) z = default_zchunk(c, prec, t);
    if (z < kMinZChunk) z = kMinZChunk;
    if (z > c.nz) z = c.nz;
    *tile = t;
    *zchunk = z;
}

static void choose_config(const Consts &c, ns_precision prec, int *tile, int *zchunk)
{
    choose_config(c, prec, -1, 0, tile, zchunk);
}

// Blocks whose diagnostic partials the workspace has room for.
static int64_t max_partial_blocks(const Consts &c)
{
    int64_t m = diag_num_blocks(c);
    for (int t = 0; t < TILE_COUNT; ++t) {
        const int64_t b = fused_num_blocks(c, t, kMinZChunk);
        if (b > m) m = b;
    }
    return m;
}

// The brick kernels run small grids whose launch shape is left to the library
// (no tile, z-chunk or order asked for by the call or the thread); returns the
// planes of a brick, 0 for the march.  Two planes where that gives at most one
// brick per compute unit, else four planes as long as the device holds all
// bricks at once: two (FP64) or four (FP32 storage) fit the LDS of a compute
// unit.  Measured, us per RK3 step, bricks | best march: FP64 16^3 14.2 | 20.9,
// 24^3 14.8 | 21.5, 32^3 16.9 | 23.2, 36^3 27.1 | 28.8, 40^3 27.8 | 30.4, 44^3
// 37.5 | 32.4, 64x40x28 (560 bricks) 36.8 | 29.7; FP32 storage 16^3 13.5 | 21.9,
// 32^3 15.5 | 22.9, 40^3 19.0 | 27.5, 48^3 27.9 | 29.7, 60^3 43.6 | 40.7, 64^3
// 48.7 | 40.2.  Two planes against four: 16^3 FP64 14.6 | 16.3, 32^3 (512 of
// two) 19.5 | 18.4.  The bricks may not outnumber the blocks that the workspace has
// diagnostic partials for: those of a march of one-plane chunks, which are fewer
// on some grids of an odd number of planes (16x165x5: 252 two-plane bricks, 210
// blocks of 8x8).
static int choose_brick(const Consts &c, ns_precision prec, int tile_in, int zchunk_in)
{
    const bool automatic = tile_in < 0 && zchunk_in <= 0 && g_tile < 0 && g_zchunk <= 0 && g_order == 0;
    if (!automatic) return 0;
    const int64_t cus = compute_units(), room = max_partial_blocks(c);
    const int64_t two = brick_num_blocks(c, 2), four = brick_num_blocks(c, 4);
    if (two <= cus && two <= room) return 2;
    if (four <= (prec == NS_FP64 ? 2 : 4) * cus && four <= room) return 4;
    return 0;
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Layout {
    size_t partial, rec, acc, b1, b2, stored, G, total;
};

// Scratch layout.  The diagnostic partials and one ns_diag record come
// first, so every workspace size returned by ns_workspace_bytes also serves
// diagnostics().
static Layout layout(const Consts &c, ns_algo algo, ns_precision prec)
{
    Layout L;
    size_t off = 0;
    const size_t n5 = 5 * (size_t)c.N;
    L.partial = off;
    off = align256(off + (size_t)max_partial_blocks(c) * kDiag * sizeof(double));
    L.rec = off;
    off = align256(off + sizeof(ns_diag));
    const size_t stage_elt = (prec == NS_FP64) ? sizeof(double) : sizeof(float);
    L.acc = off;
    off = align256(off + n5 * sizeof(double));
    L.b1 = off;
    off = align256(off + n5 * stage_elt);
    L.b2 = off;
    off = align256(off + n5 * stage_elt);
    L.stored = L.G = 0;
    if (algo == NS_ALGO_SOME) {
        L.G = off;
        off = align256(off + rs_workspace_doubles(c) * sizeof(double));
    }
    if (algo == NS_ALGO_STORED) {
        off = align256(off + n5 * sizeof(double));   // a residual array, unused now: the size stays
        L.stored = off;
        off = align256(off + stored_workspace_doubles(c) * sizeof(double));
    }
    L.total = off;
    return L;
}

static size_t diag_bytes(const Consts &c)
{
    return align256((size_t)max_partial_blocks(c) * kDiag * sizeof(double)) + align256(sizeof(ns_diag));
}

static bool finite_pos(double x) { return std::isfinite(x) && x > 0.0; }

static ns_status check_params(const ns_params *p)
{
    if (!p) return NS_ERR_ARG;
    int64_t n = 1;
    for (int d = 0; d < 3; ++d) {
        if (p->n[d] < 5 || p->n[d] > 2048) return NS_ERR_SHAPE;
        n *= p->n[d];
        if (!finite_pos(p->length[d])) return NS_ERR_ARG;
    }
    if (n >= ((int64_t)1 << 31)) return NS_ERR_SHAPE;
    if (!std::isfinite(p->gamma) || !(p->gamma > 1.0)) return NS_ERR_ARG;
    if (!finite_pos(p->prandtl) || !finite_pos(p->mach)) return NS_ERR_ARG;
    if (std::isnan(p->reynolds) || !(p->reynolds > 0.0)) return NS_ERR_ARG;
    return NS_OK;
}

ns_status validate_params(const ns_params *p) { return check_params(p); }

static bool valid_algo(int a) { return a == NS_ALGO_STORED || a == NS_ALGO_FUSED || a == NS_ALGO_SOME; }
static bool valid_prec(int q) { return q == NS_FP64 || q == NS_FP32_STORE; }

static ns_status check_work(const void *work, size_t have, size_t need)
{
    if (need > 0 && !work) return NS_ERR_ARG;
    if (have < need) return NS_ERR_WORKSPACE;
    if (((uintptr_t)work & 255) != 0) return NS_ERR_WORKSPACE;
    return NS_OK;
}

// State, Q and R arrays must be 16-byte aligned (the stage kernels load
// x-neighbour pairs of doubles with one 16-byte access); diagnostics
// records 8-byte aligned.
static bool aligned(const void *ptr, uintptr_t a) { return ((uintptr_t)ptr & (a - 1)) == 0; }

template <typename T>
static T *at(void *work, size_t off)
{
    return (T *)((char *)work + off);
}

ns_status make_fused_plan(const ns_params *p, ns_precision prec, int tile, int zchunk,
                          double *state, void *work, size_t work_bytes, FusedPlan *out)
{
    ns_status st = check_params(p);
    if (st != NS_OK) return st;
    if (!valid_prec(prec) || !state || !out || !aligned(state, 16)) return NS_ERR_ARG;
    if (tile < -1 || tile >= TILE_COUNT || zchunk < 0 || (zchunk > 0 && zchunk < kMinZChunk))
        return NS_ERR_ARG;
    const Consts c = make_consts(p);
    const Layout L = layout(c, NS_ALGO_FUSED, prec);
    st = check_work(work, work_bytes, L.total);
    if (st != NS_OK) return st;
    FusedPlan f;
    f.c = c;
    f.prec = prec;
    choose_config(c, prec, tile, zchunk, &f.tile, &f.zchunk);
    f.order = g_order;
    if (!fused_order_supported(f.tile, f.order)) return NS_ERR_UNSUPPORTED;
    f.brick = choose_brick(c, prec, tile, zchunk);
    f.nblk = f.brick ? brick_num_blocks(c, f.brick) : fused_num_blocks(c, f.tile, f.zchunk);
    f.state = state;
    f.partial = at<double>(work, L.partial);
    f.acc = at<double>(work, L.acc);
    f.b1 = at<void>(work, L.b1);
    f.b2 = at<void>(work, L.b2);
    *out = f;
    return NS_OK;
}

// One RK3 step of the fused class: stage 1 Q^n -> b1 (next stage input)
// and the accumulator (plus the diagnostics partials of Q^n when diag_out
// is given), stage 2 b1 -> b2 with the accumulator in place (and the partials
// reduced into *diag_out), stage 3 b2 -> Q^{n+1} in the state buffer.
hipError_t enqueue_fused_step(const FusedPlan &f, double dt, ns_diag *diag_out, hipStream_t s)
{
    auto launch = [&](const StageArgs &a) {
        if (!f.brick) return launch_fused_stage(f.c, a, f.prec, f.tile, s);
        return f.prec == NS_FP64 ? launch_brick_stage(f.c, a, f.brick, s) : launch_brick32_stage(f.c, a, f.brick, s);
    };
    StageArgs a = {};
    a.zchunk = f.zchunk;
    a.order = f.order;
    a.qin = f.state;
    a.qout = f.b1;
    a.acc_out = f.acc;
    a.a_dt = rk_a(0) * dt;
    a.b_dt = rk_b(0) * dt;
    a.mode = 1;
    a.diag_partial = diag_out ? f.partial : nullptr;
    hipError_t e = launch(a);
    if (e != hipSuccess) return e;
    a.qin = f.b1;
    a.acc_in = f.acc;
    a.acc_out = f.acc;
    a.qout = f.b2;
    a.a_dt = rk_a(1) * dt;
    a.b_dt = rk_b(1) * dt;
    a.mode = 2;
    a.diag_partial = nullptr;
    a.fin_partial = f.partial;
    a.fin_blocks = (int)f.nblk;   // below 2^31 points / 64
    a.fin_out = diag_out;
    e = launch(a);
    if (e != hipSuccess) return e;
    a.fin_out = nullptr;
    a.qin = f.b2;
    a.acc_in = f.acc;
    a.acc_out = nullptr;
    a.qout = f.state;
    a.a_dt = rk_a(2) * dt;
    a.b_dt = 0.0;
    a.mode = 3;
    return launch(a);
}

}  // namespace ns

using namespace ns;

extern "C" {

const char *ns_status_string(ns_status s)
{
    switch (s) {
    case NS_OK: return "NS_OK";
    case NS_ERR_ARG: return "NS_ERR_ARG: invalid argument";
    case NS_ERR_SHAPE: return "NS_ERR_SHAPE: grid size out of range";
    case NS_ERR_WORKSPACE: return "NS_ERR_WORKSPACE: workspace too small or misaligned";
    case NS_ERR_DEVICE: return "NS_ERR_DEVICE: HIP error";
    case NS_ERR_NONFINITE: return "NS_ERR_NONFINITE: non-finite diagnostics";
    case NS_ERR_NOMEM: return "NS_ERR_NOMEM: device memory allocation failed";
    case NS_ERR_UNSUPPORTED: return "NS_ERR_UNSUPPORTED: combination not provided";
    }
    return "unknown ns_status";
}

size_t ns_state_bytes(const ns_params *p)
{
    if (check_params(p) != NS_OK) return 0;
    return 5 * (size_t)p->n[0] * p->n[1] * p->n[2] * sizeof(double);
}

size_t ns_workspace_bytes(const ns_params *p, ns_algo algo, ns_precision prec)
{
    if (check_params(p) != NS_OK || !valid_algo(algo) || !valid_prec(prec)) return 0;
    if (algo != NS_ALGO_FUSED && prec != NS_FP64) return 0;
    return layout(make_consts(p), algo, prec).total;
}

ns_status ns_set_fused_config(int32_t tile, int32_t zchunk)
{
    if (tile < -1 || tile >= TILE_COUNT || zchunk < 0) return NS_ERR_ARG;
    if (zchunk > 0 && zchunk < kMinZChunk) return NS_ERR_ARG;
    g_tile = tile;
    g_zchunk = zchunk;
    return NS_OK;
}

ns_status ns_set_fused_order(int32_t order)
{
    if (order != 0 && order != 1) return NS_ERR_ARG;
    g_order = order;
    return NS_OK;
}

int32_t ns_get_fused_order(void) { return g_order; }

ns_status ns_get_fused_config(const ns_params *p, ns_precision prec, int32_t *tile,
                              int32_t *zchunk)
{
    ns_status st = check_params(p);
    if (st != NS_OK) return st;
    if (!tile || !zchunk || !valid_prec(prec)) return NS_ERR_ARG;
    int t, z;
    choose_config(make_consts(p), prec, &t, &z);
    *tile = t;
    *zchunk = z;
    return NS_OK;
}

ns_status tgv_init(const ns_params *p, double *state, void *stream)
{
    ns_status st = check_params(p);
    if (st != NS_OK) return st;
    if (!state || !aligned(state, 16)) return NS_ERR_ARG;
    const Consts c = make_consts(p);
    NS_HIP_OK(launch_tgv_init(c, p, state, (hipStream_t)stream));
    return NS_OK;
}

ns_status ns_residual(const ns_params *p, ns_algo algo, const double *Q, double *R, void *work,
                      size_t work_bytes, void *stream)
{
    ns_status st = check_params(p);
    if (st != NS_OK) return st;
    if (!valid_algo(algo) || !Q || !R || !aligned(Q, 16) || !aligned(R, 16)) return NS_ERR_ARG;
    const Consts c = make_consts(p);
    const size_t n5b = 5 * (size_t)c.N * sizeof(double);
    if ((const char *)Q < (const char *)R + n5b && (const char *)R < (const char *)Q + n5b)
        return NS_ERR_ARG;   // overlap
    hipStream_t s = (hipStream_t)stream;
    if (algo == NS_ALGO_FUSED) {
        int tile, zc;
        choose_config(c, NS_FP64, &tile, &zc);
        const int order = g_order;
        if (!fused_order_supported(tile, order)) return NS_ERR_UNSUPPORTED;
        StageArgs a = {};
        a.order = order;
        a.qin = Q;
        a.rout = R;
        a.mode = 0;
        a.zchunk = zc;
        const int brick = choose_brick(c, NS_FP64, -1, 0);
        NS_HIP_OK(brick ? launch_brick_stage(c, a, brick, s) : launch_fused_stage(c, a, NS_FP64, tile, s));
        return NS_OK;
    }
    const Layout L = layout(c, algo, NS_FP64);
    st = check_work(work, work_bytes, L.total);
    if (st != NS_OK) return st;
    if (algo == NS_ALGO_SOME) {
        NS_HIP_OK(rs_stage(c, Q, at<double>(work, L.G), nullptr, nullptr, nullptr, R, 0.0, 0.0, 0,
                           default_zchunk(c, NS_FP64, TILE_32x8_3G), s));
        return NS_OK;
    }
    StageArgs a = {};
    a.qin = Q;
    a.rout = R;
    NS_HIP_OK(stored_stage(c, a, at<double>(work, L.stored), s));
    return NS_OK;
}

ns_status rk3_step(const ns_params *p, ns_algo algo, ns_precision prec, double dt, int32_t nsteps,
                   double *state, void *work, size_t work_bytes, ns_diag *diag_dev, void *stream)
{
    ns_status st = check_params(p);
    if (st != NS_OK) return st;
    if (!valid_algo(algo) || !valid_prec(prec) || !state || !aligned(state, 16)) return NS_ERR_ARG;
    if (diag_dev && !aligned(diag_dev, 8)) return NS_ERR_ARG;
    if (!std::isfinite(dt) || !(dt > 0.0) || nsteps < 0) return NS_ERR_ARG;
    if (algo != NS_ALGO_FUSED && prec != NS_FP64) return NS_ERR_UNSUPPORTED;
    const Consts c = make_consts(p);
    const Layout L = layout(c, algo, prec);
    st = check_work(work, work_bytes, L.total);
    if (st != NS_OK) return st;
    if (nsteps == 0) return NS_OK;
    hipStream_t s = (hipStream_t)stream;
    double *partial = at<double>(work, L.partial);
    double *acc = at<double>(work, L.acc);
    void *b1 = at<void>(work, L.b1);
    void *b2 = at<void>(work, L.b2);

    if (algo == NS_ALGO_FUSED) {
        FusedPlan f;
        st = make_fused_plan(p, prec, -1, 0, state, work, work_bytes, &f);
        if (st != NS_OK) return st;
        for (int32_t step = 0; step < nsteps; ++step)
            NS_HIP_OK(enqueue_fused_step(f, dt, diag_dev ? diag_dev + step : nullptr, s));
        return NS_OK;
    }

    if (algo == NS_ALGO_SOME) {
        double *G = at<double>(work, L.G);
        double *q1 = (double *)b1, *q2 = (double *)b2;
        const int zc = default_zchunk(c, NS_FP64, TILE_32x8_3G);
        for (int32_t step = 0; step < nsteps; ++step) {
            if (diag_dev) {
                NS_HIP_OK(launch_diag_partials(c, state, partial, s));
                NS_HIP_OK(launch_diag_finalize(c, partial, diag_num_blocks(c), diag_dev + step, s));
            }
            NS_HIP_OK(rs_stage(c, state, G, nullptr, acc, q1, nullptr, rk_a(0) * dt, rk_b(0) * dt, 1, zc, s));
            NS_HIP_OK(rs_stage(c, q1, G, acc, acc, q2, nullptr, rk_a(1) * dt, rk_b(1) * dt, 2, zc, s));
            NS_HIP_OK(rs_stage(c, q2, G, acc, nullptr, state, nullptr, rk_a(2) * dt, 0.0, 3, zc, s));
        }
        return NS_OK;
    }

    // stored-derivative class
    double *D = at<double>(work, L.stored);
    double *q1 = (double *)b1, *q2 = (double *)b2;
    for (int32_t step = 0; step < nsteps; ++step) {
        if (diag_dev) {
            NS_HIP_OK(launch_diag_partials(c, state, partial, s));
            NS_HIP_OK(launch_diag_finalize(c, partial, diag_num_blocks(c), diag_dev + step, s));
        }
        for (int k = 0; k < 3; ++k) {
            StageArgs a = {};
            a.qin = k == 0 ? state : k == 1 ? q1 : q2;
            a.acc_in = acc;
            a.acc_out = acc;
            a.qout = k == 0 ? q1 : k == 1 ? q2 : state;
            a.a_dt = rk_a(k) * dt;
            a.b_dt = rk_b(k) * dt;
            a.mode = k + 1;
            NS_HIP_OK(stored_stage(c, a, D, s));
        }
    }
    return NS_OK;
}

ns_status ns_stage_stream(const ns_params *p, int32_t stage, double *state, void *work,
                          size_t work_bytes, void *stream)
{
    ns_status st = check_params(p);
    if (st != NS_OK) return st;
    if (stage < 1 || stage > 3 || !state || !aligned(state, 16)) return NS_ERR_ARG;
    const Consts c = make_consts(p);
    const Layout L = layout(c, NS_ALGO_FUSED, NS_FP64);
    st = check_work(work, work_bytes, L.total);
    if (st != NS_OK) return st;
    double *acc = at<double>(work, L.acc);
    double *b1 = at<double>(work, L.b1), *b2 = at<double>(work, L.b2);
    const int64_t n5 = 5 * c.N;
    hipStream_t s = (hipStream_t)stream;
    if (stage == 1) NS_HIP_OK(launch_stream_stage(1, n5, state, nullptr, acc, b1, s));
    if (stage == 2) NS_HIP_OK(launch_stream_stage(2, n5, b1, acc, acc, b2, s));
    if (stage == 3) NS_HIP_OK(launch_stream_stage(3, n5, b2, acc, nullptr, state, s));
    return NS_OK;
}

ns_status diagnostics(const ns_params *p, const double *state, ns_diag *out_host, void *work,
                      size_t work_bytes, void *stream)
{
    ns_status st = check_params(p);
    if (st != NS_OK) return st;
    if (!state || !out_host || !aligned(state, 16)) return NS_ERR_ARG;
    const Consts c = make_consts(p);
    const Layout L = layout(c, NS_ALGO_FUSED, NS_FP64);
    st = check_work(work, work_bytes, diag_bytes(c));
    if (st != NS_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    double *partial = at<double>(work, L.partial);
    ns_diag *rec = at<ns_diag>(work, L.rec);
    NS_HIP_OK(launch_diag_partials(c, state, partial, s));
    NS_HIP_OK(launch_diag_finalize(c, partial, diag_num_blocks(c), rec, s));
    NS_HIP_OK(hipMemcpyAsync(out_host, rec, sizeof(ns_diag), hipMemcpyDeviceToHost, s));
    NS_HIP_OK(hipStreamSynchronize(s));
    const double *v = (const double *)out_host;
    for (int k = 0; k < 8; ++k)
        if (!std::isfinite(v[k])) return NS_ERR_NONFINITE;
    return NS_OK;
}

}  // extern "C"
