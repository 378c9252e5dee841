// Four Jacobi steps per pass over memory (deep_dev.hpp): box descriptors, the
// rule that admits a grid and chooses the variant, and the launchers.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "kernels.hpp"

namespace od {

constexpr int kDeepSteps = 4, kDeep2dSteps = 8;

// One workgroup's work: the lanes cover the vectors [ws, ws + LX) along x (see
// DeepPlan::vx) and the rows [ys, ys + EY), march z and write the vectors
// [wo0, wo1), rows [yo0, yo1) and planes [z0, z1) four steps later.
struct DeepTile {
    int32_t ws, ys;
    int32_t wo0, wo1, yo0, yo1;
    int32_t z0, z1;
};
static_assert(sizeof(DeepTile) == 32, "DeepTile layout");

// What a four-step pass needs of the grid on the device.  The chare of a cell
// follows from one index per axis (a regular decomposition's chare
// coordinates, or explicit blocks' owner-grid coordinates and `owner`).
struct DeepMap {
    void* arena;
    const BlockDev* blocks;
    const int32_t* vx;         // first cell of each vector along x, and nx behind the last
    const int32_t* vi;         // index of each vector
    const int32_t* iy;         // index of each row
    const int32_t* iz;         // index of each plane
    const int32_t* zn;         // first plane behind it that may belong to other chares
    const int32_t* owner;      // null: the combined index is the chare
    const int32_t* corigin;
    const int32_t* dir_pb;
    int32_t k[2];
    int32_t nv, ny, nz;        // vectors, rows, planes
};

struct DeepPlan {
    int rows = 0;                      // rows of a lane's strip: 4 (serving fp32: 2), 1 for small grids, 0 in 2D
    int waves = 0;                     // of a workgroup
    bool ragged = false;               // some vectors are not full
    std::vector<DeepTile> tiles;       // in launch order; empty: the grid has no four-step passes
    std::vector<int32_t> vx, vi;       // as in DeepMap
    bool by_tiles = false;             // the planned tiles are estimated to be quicker
    // message-driven, us: what a pass gains on pairs, how much longer a launch of
    // boxes takes to start than one of tiles, and what a further launch of tiles
    // for the rest of a count adds
    double gain = 0, start = 0, rest = 0;
};

// Lane coverage: LX vectors of 16 bytes by EY rows.
void deep_shape(int dtype_bytes, const DeepPlan& d, int* lx, int* ey);
// Boxes for a grid of that form, whose passes by tiles are of tile_steps steps.
DeepPlan deep_plan(const Plan& p, int dtype_bytes, od_exec exec, int tile_steps);
// The boxes of a served solve: workgroups of kServeWaves waves in either type,
// at most kServeBoxes of them (a slot's dependency lists hold 26 for each).
constexpr int kServeWaves = 8, kServeBoxes = 2048;
// ring: cells beside what is written that its lanes cover along x and y, the
// steps of its longest pass.
DeepPlan deep_plan_serve(const Plan& p, int dtype_bytes, int ring);
// vx, vi, iy, iz and zn of DeepMap one after another; `at`: where each begins.
std::vector<int32_t> deep_tables(const Plan& p, const DeepPlan& d, size_t at[5]);

// What a served solve's tasks read, in its slot of the control region:
// positions are bytes from the server's arena.
struct ServeSolve {
    int64_t arena, blocks, corigin, dir_pb, tiles, tab[5];
    int32_t k[2], nv, ny, nz;
    int32_t rows, ragged;
    int32_t check_every, max_iters, passes;   // steps between checks, at most; passes between checks
};
static_assert(sizeof(ServeSolve) == 120, "ServeSolve layout");
// Passes of a solve: every interval between checks (the last one ends at the
// cap) takes the fewest, its first one the steps that fours leave over.
inline int32_t serve_passes(int32_t steps) { return steps > 0 ? 1 + (steps - 1) / kDeepSteps : 0; }
inline int32_t serve_target(int32_t check_every, int32_t max_iters) {
    return check_every > 0 ? max_iters / check_every * serve_passes(check_every) + serve_passes(max_iters % check_every)
                           : serve_passes(max_iters);
}
// Iterations done after a decision pass.
inline int32_t serve_iters(int32_t check_every, int32_t max_iters, int32_t pass) {
    return pass >= serve_target(check_every, max_iters) ? max_iters : pass / serve_passes(check_every) * check_every;
}

// One pass: reads parity `parity`, writes the field four steps later into
// parity ^ 1; res zeroing as launch_sweep, and with want_res the residual of
// the fourth step.
hipError_t launch_deep(int dtype_bytes, const DeepPlan& d, hipStream_t st, const DeepMap& g, const DeepTile* tiles,
                       int parity, unsigned long long* res, int32_t zero_lo, int32_t zero_hi, int hints,
                       bool want_res);

// Every pass of an iteration count in one cooperative launch of `grid`
// workgroups (at most deep_max_grid); bar / err as launch_persistent.
hipError_t launch_deep_persistent(int dtype_bytes, const DeepPlan& d, hipStream_t st, int grid, const DeepMap& g,
                                  const DeepTile* tiles, int parity, int64_t passes, unsigned long long* res,
                                  unsigned int* bar, unsigned int* err, int64_t wait_ticks, int hints, bool want_res);
// The message-driven scheduler over boxes: a scheduler step is one pass.
hipError_t launch_deep_msg(int dtype_bytes, const DeepPlan& d, hipStream_t st, int grid, const MsgArgs& a,
                           const DeepMap& g, const DeepTile* tiles);
// Eight steps of the 2D 5-point stencil (deep2d.hip); `rows` is 0, and vectors
// are 32 bytes.
DeepPlan deep_plan2d(const Plan& p, int dtype_bytes);
hipError_t launch_deep2d(int dtype_bytes, const DeepPlan& d, hipStream_t st, const DeepMap& g, const DeepTile* tiles,
                         int parity, unsigned long long* res, int32_t zero_lo, int32_t zero_hi, int hints,
                         bool want_res);
// Boxes in launch order: workgroup w runs on XCD w % 8, each XCD a contiguous run.
std::vector<DeepTile> xcd_runs(const std::vector<DeepTile>& list);

// Workgroups of either cooperative form that are co-resident on the device.
int deep_max_grid(int dtype_bytes, const DeepPlan& d);
hipError_t launch_fill_i32(hipStream_t st, int32_t* p, int32_t n, int32_t v);

// For each box the boxes whose written cells its lanes read, and those that
// read its own (CSR, ascending, symmetric).
void deep_deps(const DeepPlan& d, int dtype_bytes, std::vector<int32_t>& ptr, std::vector<int32_t>& idx,
               int ring = kDeepSteps);

}  // namespace od
