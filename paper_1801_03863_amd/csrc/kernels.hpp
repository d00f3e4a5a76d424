// kernels.hpp -- launch interface between the host runtime and the HIP
// kernels of the fused stream-and-collide step.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lbm {

enum Storage { ST_F64 = 0, ST_F32N64 = 1, ST_F32 = 2, ST_F16DEV = 3 };
enum Coll { CO_MINXENT4 = 0, CO_MINXENT2 = 1, CO_SRT = 2, CO_TRT = 3, CO_MRT = 4 };
enum Bc { BC_PERIODIC = 0, BC_TUBE = 1, BC_CAVITY = 2, BC_BOX = 3 };

// Status record of one instance (device memory).
struct DevStatus {
    uint32_t flags;
    int32_t pad;
    uint64_t first;  // (step << 32) | node of the first unstable node; all ones until then
    int64_t guarded;
};

// One lattice instance as the kernels see it.  Populations of instance i
// live in b planes of `plane` elements starting at element `offset` of each
// of the two buffers; node (x, y) is element y*pitch + x of a plane (D2Q9
// rows start on whole 128-byte lines; elements x >= nx of a row are padding
// that no kernel reads).  Node numbers (status, host fields) stay y*nx + x.
struct Inst {
    int32_t nx, ny;
    int32_t pitch;   // row stride in elements (>= nx)
    int64_t offset;
    int64_t plane;
    double omega;    // 1/tau
    double omega2;   // 1/tau2
    double u_lid;
    double rho0;
    double lid[9];   // equilibrium of (rho0, (u_lid, 0))
    int64_t stop;    // batched: the instance takes no step from this step index on
};

// Byte offset of node (x, y) in a plane whose rows are `pitch` elements apart:
// the row's in 64 bits, since a plane may hold 4 GiB and more.
__host__ __device__ inline int64_t plane_bytes(int x, int y, int pitch, int elem)
{
    return (int64_t)y * pitch * elem + (int64_t)x * elem;
}

// Tile of the on-chip window shapes: tw x th nodes, gx x gy tiles.
struct WindowTile {
    int32_t tw, th, gx, gy;
};

// Everything a step launch needs besides the buffers.
struct StepArgs {
    const Inst *inst;       // device table (batched) -- or nullptr
    Inst one;               // the single instance (non-batched launches)
    DevStatus *status;      // one record per instance
    const int64_t *step_base;  // if not null, added to `step` on the error path
    const int32_t *tile_inst;  // batched: instance of each tile
    const int32_t *tile_first; // batched: first node of each tile, or of 2D tiles (two-step shapes, register
                               // pipelines) the index ty * tiles_x + tx within the instance
    int64_t step;
    int32_t bc;
    int32_t ntiles;
    int32_t tiles_x;        // single D2Q9: tiles along x
    int32_t tile_rows;      // register pipeline: rows of a tile
    int32_t tall;           // single register pipeline: tile rows of tile_rows rows; the rest have low_rows
    int32_t low_rows;
    int32_t xcd_swizzle;
    float fp16_scale;       // FP16DEV: 2^k
    float fp16_iscale;      // 2^-k
    int32_t max_steps;      // shapes taking several steps per launch: steps this launch takes
    WindowTile win;         // on-chip window shapes
};

// Host-side launchers (return hipError_t of the launch).
int d2q9_variant_count(int coll);
const char *d2q9_variant_name(int coll, int variant);
// Steps one launch of a single-lattice D2Q9 shape takes at most (1; 2 for the
// temporally blocked shapes; more for the on-chip window shapes, where a
// lattice may allow fewer: d2q9_window_best; StepArgs::max_steps sets fewer),
// whether it is a window shape, and the host-side set-up a shape needs before
// its first launch (call outside stream capture).
int d2q9_variant_steps(int coll, int variant);
bool d2q9_variant_window(int coll, int variant);
// Shape a single lattice runs in unless another is set: the fastest by the
// estimates above its definition, among shape 0, the window shapes and the
// register pipelines (none of which needs set-up).
int d2q9_default_variant(int storage, int coll, int nx, int ny, int bc);
hipError_t prepare_d2q9_variant(int st, int coll, int variant);
hipError_t launch_d2q9_step(int storage, int coll, int variant, const void *src, void *dst,
                            const StepArgs &a, hipStream_t s);
hipError_t launch_d2q9_batch_step(int storage, int coll, int variant, const void *src, void *dst,
                                  const StepArgs &a, hipStream_t s);
// On-chip window shapes (window.hip).  Nodes a window may hold; which of nk step
// counts per launch takes the fewest microseconds per step on one lattice, the
// first of equal ones, with that estimate and the tile (-1 if none of their windows
// fits, or none takes less than `below`); and the launch (StepArgs::win holds
// the tile, max_steps at most the count it was planned for).
constexpr int kWindowCus = 256;  // compute units the tiles are spread over
int d2q9_window_cap(int storage);
int d2q9_window_best(int storage, int coll, int nx, int ny, int bc, const int *ks, int nk, double below,
                     WindowTile *tile, double *us_per_step);
hipError_t launch_d2q9_window(int storage, int coll, const void *src, void *dst, const StepArgs &a, hipStream_t s);
// Register-pipeline shapes (pipeline.hip): whether a shape is one; the tile
// rows for launches of k steps of one lattice, with the estimated
// microseconds per step (no rows, and 1e30, if that is not less than `below`); and one launcher per collision rule, for
// windows of k steps (2 to 4; a batch may take fewer, a single lattice takes
// k) with tiles of a.tile_rows rows.
bool d2q9_variant_pipe(int coll, int variant);
int d2q9_variant_rows(int coll, int variant);  // fixed tile rows of such a shape, or 0: d2q9_pipe_rows
int d2q9_pipe_rows(int storage, int coll, int nx, int ny, int k, double *us_per_step, double below = 1e30);
hipError_t launch_d2q9_pipe_0(int storage, int k, int batch, const void *src, void *dst, const StepArgs &a,
                              hipStream_t s);
hipError_t launch_d2q9_pipe_1(int storage, int k, int batch, const void *src, void *dst, const StepArgs &a,
                              hipStream_t s);
hipError_t launch_d2q9_pipe_2(int storage, int k, int batch, const void *src, void *dst, const StepArgs &a,
                              hipStream_t s);
hipError_t launch_d2q9_pipe_3(int storage, int k, int batch, const void *src, void *dst, const StepArgs &a,
                              hipStream_t s);
hipError_t launch_d2q9_pipe_4(int storage, int k, int batch, const void *src, void *dst, const StepArgs &a,
                              hipStream_t s);
int d1q3_variant_count();
const char *d1q3_variant_name(int variant);
int d1q3_variant_steps(int variant);  // steps one launch takes at most (StepArgs::max_steps sets fewer)
int d1q3_default_variant(int batch, int64_t nodes);  // shape a context of that many nodes starts in
hipError_t launch_d1q3_step(int storage, int variant, const void *src, void *dst, const StepArgs &a,
                            hipStream_t s);
hipError_t launch_d1q3_batch_step(int storage, int variant, const void *src, void *dst,
                                  const StepArgs &a, hipStream_t s);
// D1Q3 shapes with the nodes in registers (tube.hip), n = 2, 4 or 8 per lane.
hipError_t launch_d1q3_regs(int storage, int n, int batch, const void *src, void *dst, const StepArgs &a,
                            hipStream_t s);
// Batch of small D2Q9 lattices resident in LDS: one workgroup per instance
// (a.ntiles = instances) runs nsteps steps in one launch; dst receives the
// final state (it may equal src).
hipError_t launch_d2q9_lds(int storage, int coll, const void *src, void *dst, const StepArgs &a, int nsteps,
                           int block, size_t smem_bytes, hipStream_t s);
// Batched shapes: count (MinxEnt4 D2Q9 batches also have two-step shapes),
// steps per launch, the shape whose kernel takes a launch of one step (0 for the
// register shapes), nodes per tile of the tile table (negative for 2D tiles:
// -(width * 4096 + rows)), name, the shape a D2Q9 batch of these n instances
// starts in, and the host-side set-up before a shape's first launch.
int batch_variant_count(int lattice, int coll);
int batch_variant_steps(int lattice, int coll, int variant);
int batch_one_step(int lattice, int coll, int variant);
int batch_tile_nodes(int lattice, int coll, int variant);
const char *batch_variant_name(int lattice, int coll, int variant);
int batch_default_variant(int storage, int coll, const Inst *inst, int n);
hipError_t prepare_batch_variant(int st, int coll, int variant);

// Nodes [g0, g1) of all instances counted one after another.
struct NodeRange {
    const Inst *inst;       // device table, or nullptr: `one`
    const int64_t *prefix;  // device: number of the first node of each instance
    Inst one;
    int32_t n, bc;
    int64_t g0, g1;
};

// Set the state of a range of nodes: pre-shifted equilibrium of FP64 fields
// (node g is element g - g0 of each), or FP64 populations f (of all nodes: b
// planes per instance).
hipError_t launch_init(int lattice, int storage, const NodeRange &r, const double *rho, const double *ux,
                       const double *uy, const double *f, void *buf, float fp16_scale, hipStream_t s);
// Gather the pre-collision populations of a range of nodes and write either
// their moments (any of rho, ux, uy may be null) or the populations (f: planes
// fstride apart), as doubles.  Node g is element g - g0 of every array, in
// device memory or host memory the device can write.
hipError_t launch_gather(int lattice, int storage, const NodeRange &r, const void *buf, double *rho, double *ux,
                         double *uy, double *f, int64_t fstride, float fp16_iscale, hipStream_t s);

hipError_t launch_copy(void *dst, const void *src, size_t bytes, hipStream_t s);
hipError_t launch_add_step_base(int64_t *base, int64_t n, hipStream_t s);
hipError_t launch_set_step_base(int64_t *base, int64_t v, hipStream_t s);
hipError_t launch_clear_status(DevStatus *st, int n, hipStream_t s);

}  // namespace lbm
