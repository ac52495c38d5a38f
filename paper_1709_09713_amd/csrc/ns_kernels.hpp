// ns_kernels.hpp -- launch interfaces of the device kernels (host side).
#pragma once

#include "ns_common.hpp"

namespace ns {

// Column-tile shapes of the fused kernel.  Tiles 0-7: threads = BX * BY,
// one z column each (ns_fused.hip).  Tiles 8-10 (_3G) split each column over
// three groups of waves (FP64 ns_trio.hip, FP32 storage ns_trio32.hip).  Chosen
// per problem by the autotuner or by the default rule.
enum {
    TILE_32x8 = 0, TILE_16x16 = 1, TILE_64x4 = 2, TILE_32x16 = 3,
    TILE_16x8 = 4, TILE_32x4 = 5, TILE_16x4 = 6, TILE_8x8 = 7,
    TILE_16x8_3G = 8, TILE_32x8_3G = 9, TILE_16x4_3G = 10, TILE_COUNT = 11
};

// One fused launch: residual only (mode 0) or RK stage 1..3.
struct StageArgs {
    const void *qin;        // stencil input state (double, or float deviations)
    const double *acc_in;   // RK accumulator in (stages 2, 3)
    double *acc_out;        // RK accumulator out (stages 1, 2)
    void *qout;             // stage output (stages 1, 2: next stage input; 3: state)
    double *rout;           // residual output (mode 0)
    double a_dt, b_dt;      // a_k dt and b_k dt
    int mode;               // 0 = residual, 1..3 = RK stage
    int zchunk;             // planes per block along z
    double *diag_partial;   // per-block diagnostic partial sums, or nullptr
    const double *grad;     // stored velocity gradients (intermediate-storage class)
    int order;              // in-plane evaluation order: 0 by equation, 1 by direction
    // stage 2 after a stage 1 with diagnostics: reduce its partials (the count
    // beside the other ints: eight bytes more put the grid's size, which follows
    // the arguments, on a cache line of its own, 0.2 us a stage at 16^3)
    int fin_blocks;
    const double *fin_partial;
    ns_diag *fin_out;       // nullptr: nothing to reduce
};

// Stage 2 reduces the partial sums that stage 1 left: its launch has one more
// z layer, in front, whose first block does it (one wave, fixed order) while
// the other blocks run the stage.  As a launch of its own between the stages
// it took 4 us, a fifth of a step at 16^3.  Returns the number of leading
// layers without tiles, or -1 for a block of that layer, which is done.
__device__ __forceinline__ int finalize_layer(const Consts &c, const StageArgs &s)
{
    if (s.fin_out == nullptr) return 0;
    if (blockIdx.z != 0) return 1;
    if ((blockIdx.x | blockIdx.y) == 0 && threadIdx.y * blockDim.x + threadIdx.x < 64) {
        const int t = threadIdx.y * blockDim.x + threadIdx.x;
        double v[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
        for (int b = t; b < s.fin_blocks; b += 64)
#pragma unroll
            for (int q = 0; q < 7; ++q) v[q] += s.fin_partial[(int64_t)b * kDiag + q];
#pragma unroll
        for (int q = 0; q < 7; ++q) v[q] = wave_sum(v[q]);
        if (t == 63) write_diag(c, v, s.fin_out);
    }
    return -1;
}

void tile_dims(int tile, int *bx, int *by);
int64_t fused_num_blocks(const Consts &c, int tile, int zchunk);
bool fused_order_supported(int tile, int order);
// Stage-kernel blocks resident on the current device at once (0 if the
// device cannot be queried).
int fused_resident_blocks(ns_precision prec, int tile);
hipError_t launch_fused_stage(const Consts &c, const StageArgs &s, ns_precision prec,
                              int tile, hipStream_t st);
// The split-column kernels (tiles 8-10; trio_: FP64, trio32_: FP32 storage):
// stage launch and resident blocks.
bool split_tile(int tile);
int trio32_resident_blocks(int tile);
hipError_t launch_trio32_stage(const Consts &c, const StageArgs &s, int tile, hipStream_t st);
int trio_resident_blocks(int tile);
hipError_t launch_trio_stage(const Consts &c, const StageArgs &s, int tile, hipStream_t st);
// The 32x8 three-group kernel with the velocity gradients taken from s.grad.
hipError_t launch_trio_grad(const Consts &c, const StageArgs &s, hipStream_t st);
// The brick kernels of small grids, bricks of bz = 2 or 4 planes: FP64
// (ns_brick.hip), same results as tiles 8-10 bit for bit, and FP32 storage
// (ns_brick32.hip), same results as tiles 0-7 bit for bit.
int64_t brick_num_blocks(const Consts &c, int bz);
hipError_t launch_brick_stage(const Consts &c, const StageArgs &s, int bz, hipStream_t st);
hipError_t launch_brick32_stage(const Consts &c, const StageArgs &s, int bz, hipStream_t st);
// Planes a block marches beyond its chunk (halo and pipeline depth).
int fused_extra_planes(int tile);

// Argument check of an ns_params (grid range, finite positive lengths and
// physics); NS_OK, NS_ERR_ARG or NS_ERR_SHAPE.
ns_status validate_params(const ns_params *p);

// A validated fused-class RK3 plan for one solve: constants, launch shape
// and the carve-up of its workspace.  rk3_step and the batch scheduler
// enqueue steps through it, so both run the same launches.
struct FusedPlan {
    Consts c;
    ns_precision prec;
    int tile, zchunk, order;
    int brick;           // planes of a brick, 0: the march of tile and zchunk
    int64_t nblk;
    double *state, *partial, *acc;
    void *b1, *b2;
};
// tile -1 / zchunk 0 take the calling thread's or the default launch shape.
// Validates everything (params, precision, shape, workspace) first.
ns_status make_fused_plan(const ns_params *p, ns_precision prec, int tile, int zchunk,
                          double *state, void *work, size_t work_bytes, FusedPlan *out);
hipError_t enqueue_fused_step(const FusedPlan &f, double dt, ns_diag *diag_out, hipStream_t s);

// Diagnostics: per-block partial sums of a state, then a one-block fixed-order
// final reduction into an ns_diag record.
int64_t diag_num_blocks(const Consts &c);
hipError_t launch_diag_partials(const Consts &c, const double *state, double *partial,
                                hipStream_t st);
hipError_t launch_diag_finalize(const Consts &c, const double *partial, int64_t nblocks,
                                ns_diag *out, hipStream_t st);

// The bytes of one fused FP64 RK stage (1..3) over the same buffers, with
// a pointwise update instead of the residual (the achievable ceiling of the
// stage kernel's memory traffic).  n5 = number of doubles in a field set.
hipError_t launch_stream_stage(int stage, int64_t n5, const double *qin, const double *acc_in,
                               double *acc_out, double *qout, hipStream_t st);

// Taylor-Green initial state.
hipError_t launch_tgv_init(const Consts &c, const ns_params *p, double *state, hipStream_t st);

// Stored-derivative (baseline) class.
size_t stored_workspace_doubles(const Consts &c);
// Intermediate-storage class: nine gradient arrays; one stage = gradient
// sweep + residual/RK sweep (mode 0 writes R to rout).
size_t rs_workspace_doubles(const Consts &c);
// zchunk: planes per block of the second sweep.
hipError_t rs_stage(const Consts &c, const double *qin, double *G, const double *acc_in,
                    double *acc_out, double *qout, double *rout, double a_dt, double b_dt,
                    int mode, int zchunk, hipStream_t st);
// One stage: the 60 derivative arrays into D, then residual and RK update
// (s as for the fused kernel; s.mode 0 writes R to s.rout).
hipError_t stored_stage(const Consts &c, const StageArgs &s, double *D, hipStream_t st);

}  // namespace ns
