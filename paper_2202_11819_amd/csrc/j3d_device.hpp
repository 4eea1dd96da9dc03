// j3d_device.hpp -- small HIP runtime helpers shared by the solver, batch and pool.
#pragma once

#include <hip/hip_runtime_api.h>

#include "j3d_host.hpp"

namespace j3d {

// EDEVICE with the HIP error text when `e` is not hipSuccess.
j3d_status hip_status(hipError_t e, const char *what);
inline j3d_status hip_status(int e, const char *what) { return hip_status((hipError_t)e, what); }

// The current device must be a gfx950; fills its compute-unit count.
j3d_status require_device(int *device, int *cus);

// Upload a plan's tables to the arena: blocks, problems, per-axis maps, one-sweep
// tiles and multi-sweep tiles (none without a shape), with one wait at the end.
// With a wait after each table and each problem's maps, creating a 64^3 solver
// took 80 us (now 59) and a batch of 48 small problems 1.11 ms (now 0.48).
j3d_status upload_tables(const Plan &plan, const std::vector<Tile> &tiles, const MultiPlan &m, char *arena,
                         hipStream_t stream);

// Upload a tile list to the arena's tile table.
j3d_status upload_tiles(const Plan &plan, const std::vector<Tile> &tiles, char *arena,
                        hipStream_t stream);

// Launch arguments of a plan's multi-sweep launches: everything but the tiles
// to run, the parity and the sweep count.
MultiArgs multi_args(const Plan &plan, char *arena);

// For the library's own checks, exported but no part of its interface: GRAPH and
// TWO_SWEEP runs of this solver take launches of this shape from now on, for any
// number of sweeps; sweeps receives its sweeps per launch.  EINVAL for an unknown
// shape or one the grid's blocks do not allow.  Shape -1 changes nothing: sweeps
// receives those per launch of a GRAPH run of 50.
extern "C" j3d_status j3d_check_multi_shape(j3d_solver *s, int32_t shape, int32_t *sweeps);

// Seeded initialisation of every problem of a plan (interior of parity 0,
// halo storage of both parities).
j3d_status init_fields(const Plan &plan, char *arena, hipStream_t stream);

// Pack, exchange and unpack (Fig. 1 / Fig. 3) of parity `parity` for blocks
// [b0, b1): afterwards every interior-face halo equals the neighbour's face.
j3d_status refresh_halos(const Plan &plan, char *arena, int32_t b0, int32_t b1, int parity,
                         hipStream_t stream);

// Dense interior of problem `i` to/from `dense` (device or host), parity `parity`.
j3d_status copy_dense(const Plan &plan, char *arena, int32_t i, int parity, double *dense,
                      int dense_on_device, bool to_dense, hipStream_t stream);

}  // namespace j3d
