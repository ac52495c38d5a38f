// Host-only check of the launch shapes that the library chooses by itself.
// Linked with ns_api.hip in place of the kernels: what a call would launch is
// printed, one line per call read from standard input (precision nx ny nz), for a
// device of 256 compute units.
#include <cstdio>
#include <cstdlib>

#include "../paper_1709_09713_amd/csrc/ns_kernels.hpp"

namespace ns {

namespace {
int g_brick, g_tile, g_zchunk;
int64_t g_blocks;
int64_t div_up(int64_t a, int64_t b) { return (a + b - 1) / b; }
}  // namespace

void tile_dims(int tile, int *bx, int *by)
{
    static const int x[TILE_COUNT] = {32, 16, 64, 32, 16, 32, 16, 8, 16, 32, 16};
    static const int y[TILE_COUNT] = {8, 16, 4, 16, 8, 4, 4, 8, 8, 8, 4};
    *bx = x[tile];
    *by = y[tile];
}
int64_t fused_num_blocks(const Consts &c, int tile, int zchunk)
{
    int bx, by;
    tile_dims(tile, &bx, &by);
    return div_up(c.nx, bx) * div_up(c.ny, by) * div_up(c.nz, zchunk);
}
bool split_tile(int tile) { return tile >= TILE_16x8_3G && tile <= TILE_16x4_3G; }
bool fused_order_supported(int, int order) { return order == 0; }
int fused_extra_planes(int tile) { return split_tile(tile) ? 5 : 4; }
int fused_resident_blocks(ns_precision, int tile) { return tile == TILE_32x8_3G ? 256 : 512; }
int64_t brick_num_blocks(const Consts &c, int bz) { return div_up(c.nx, 8) * div_up(c.ny, 4) * div_up(c.nz, bz); }
int64_t diag_num_blocks(const Consts &c) { return div_up(c.N, 256); }

hipError_t launch_fused_stage(const Consts &c, const StageArgs &s, ns_precision, int tile, hipStream_t)
{
    g_brick = 0;
    g_tile = tile;
    g_zchunk = s.zchunk;
    g_blocks = fused_num_blocks(c, tile, s.zchunk);
    return hipSuccess;
}
static hipError_t brick(const Consts &c, int bz)
{
    g_brick = bz;
    g_blocks = brick_num_blocks(c, bz);
    return hipSuccess;
}
hipError_t launch_brick_stage(const Consts &c, const StageArgs &, int bz, hipStream_t) { return brick(c, bz); }
hipError_t launch_brick32_stage(const Consts &c, const StageArgs &, int bz, hipStream_t) { return brick(c, bz); }
hipError_t launch_diag_partials(const Consts &, const double *, double *, hipStream_t) { return hipSuccess; }
hipError_t launch_diag_finalize(const Consts &, const double *, int64_t, ns_diag *, hipStream_t) { return hipSuccess; }
hipError_t launch_stream_stage(int, int64_t, const double *, const double *, double *, double *, hipStream_t) { return hipSuccess; }
hipError_t launch_tgv_init(const Consts &, const ns_params *, double *, hipStream_t) { return hipSuccess; }
size_t stored_workspace_doubles(const Consts &c) { return c.N; }
size_t rs_workspace_doubles(const Consts &c) { return c.N; }
hipError_t rs_stage(const Consts &, const double *, double *, const double *, double *, double *, double *, double,
                    double, int, int, hipStream_t) { return hipSuccess; }
hipError_t stored_stage(const Consts &, const StageArgs &, double *, hipStream_t) { return hipSuccess; }

}  // namespace ns

extern "C" {
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
}

int main()
{
    int prec, nx, ny, nz;
    char *memory = (char *)((uintptr_t)1 << 40);   // addresses only; nothing is read or written
    while (std::scanf("%d %d %d %d", &prec, &nx, &ny, &nz) == 4) {
        ns_params p = {};
        p.n[0] = nx, p.n[1] = ny, p.n[2] = nz;
        for (double &l : p.length) l = 6.283185307179586;
        p.gamma = 1.4, p.prandtl = 0.71, p.reynolds = 1600.0, p.mach = 0.1;
        const size_t wb = ns_workspace_bytes(&p, NS_ALGO_FUSED, (ns_precision)prec);
        if (rk3_step(&p, NS_ALGO_FUSED, (ns_precision)prec, 1e-3, 1, (double *)memory,
                     memory + ((size_t)1 << 39), wb, (ns_diag *)(memory + ((size_t)1 << 38)), nullptr) != NS_OK)
            return 1;
        // the partials take 64 bytes a block and are followed by the accumulator and the two stage buffers
        const size_t n5 = 5 * (size_t)nx * ny * nz, rest = n5 * 8 + 2 * n5 * (prec == NS_FP64 ? 8 : 4);
        std::printf("%d %d %d %d\n", ns::g_brick, ns::g_brick ? -1 : ns::g_tile, ns::g_brick ? -1 : ns::g_zchunk,
                    (size_t)ns::g_blocks * 64 + rest <= wb);
    }
    return 0;
}
