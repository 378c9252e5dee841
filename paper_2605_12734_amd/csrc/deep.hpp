// Four Jacobi steps per pass over memory (deep.hip): tile descriptors, the
// rule that admits a grid, and the launcher.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "kernels.hpp"

namespace od {

constexpr int kDeepSteps = 4;

// One workgroup's work: the lanes cover the cells [xs, xs + EX) x
// [ys, ys + EY) of the grid (global interior coordinates), march z and write
// the cells [xo0, xo1) x [yo0, yo1) x [z0, z1) four steps later.
struct DeepTile {
    int32_t xs, ys;
    int32_t xo0, xo1, yo0, yo1;
    int32_t z0, z1;
};
static_assert(sizeof(DeepTile) == 32, "DeepTile layout");

// What a four-step pass needs of the grid: the chare of a cell from one
// index per axis (a regular decomposition's chare coordinates, or explicit
// blocks' owner-grid coordinates and `owner`), and for each plane the first
// plane behind it that may belong to other chares.
struct DeepMap {
    void* arena;
    const BlockDev* blocks;
    const int32_t* ix;
    const int32_t* iy;
    const int32_t* iz;
    const int32_t* zn;
    const int32_t* owner;      // null: the index is the chare
    const int32_t* corigin;
    const int32_t* dir_pb;
    int32_t k[2];
    int32_t n[3];
};

// Lane coverage of a dtype's tile: EX x EY cells.
void deep_shape(int dtype_bytes, int* ex, int* ey);
// The grid's tiles for four-step passes in launch order; empty where the
// plan does not meet the rule (see deep.hip).
std::vector<DeepTile> deep_tiles(const Plan& p, int dtype_bytes);

// One pass: reads parity `parity`, writes the field four steps later into
// parity ^ 1; res zeroing as launch_sweep, and with want_res the residual of
// the fourth step.
hipError_t launch_deep(int dtype_bytes, hipStream_t st, const DeepMap& g, const DeepTile* tiles, int32_t ntiles,
                       int parity, unsigned long long* res, int32_t zero_lo, int32_t zero_hi, int hints,
                       bool want_res);


// Every pass of an iteration count in one cooperative launch of `grid`
// workgroups (at most deep_max_grid); bar / err as launch_persistent.
hipError_t launch_deep_persistent(int dtype_bytes, hipStream_t st, int grid, const DeepMap& g, const DeepTile* tiles,
                                  int32_t ntiles, int parity, int64_t passes, unsigned long long* res,
                                  unsigned int* bar, unsigned int* err, int64_t wait_ticks, int hints, bool want_res);
// The message-driven scheduler over boxes: a scheduler step is one pass.
hipError_t launch_deep_msg(int dtype_bytes, hipStream_t st, int grid, const MsgArgs& a, const DeepMap& g,
                           const DeepTile* tiles);
// Workgroups of either cooperative form that are co-resident on the device.
int deep_max_grid(int dtype_bytes);
hipError_t launch_fill_i32(hipStream_t st, int32_t* p, int32_t n, int32_t v);

// For each box the boxes whose written cells its lanes read, and those that
// read its own (CSR, ascending, symmetric).
void deep_deps(const std::vector<DeepTile>& t, int dtype_bytes, std::vector<int32_t>& ptr, std::vector<int32_t>& idx);

}  // namespace od
