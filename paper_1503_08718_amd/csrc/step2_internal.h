// Internal interface of the two-steps-per-pass kernels (step2_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "lbm_internal.h"

namespace mrt {

// How a cell is cut into blocks: tiles of tr rows, z-chunks of nz / nchunks
// planes; vec nodes per thread.
struct Step2Shape {
    int vec = 0;  // 0: the cell takes single steps
    int tr = 0, ntiles = 0, nchunks = 0, threads = 0;
    size_t lds = 0;
};

// whether the cell's storage and boundaries allow two steps per pass
template <typename real>
bool step2_takes(const Cell<real> &c);

// the fastest shape for these extents by the measured model, or vec = 0 where
// single steps are faster
template <typename real>
Step2Shape step2_shape(int nx, int ny, int nz, int nphase);

// state at t -> state at t + 2 (moment storage); c.src and c.dst as for launch_step
template <typename real>
hipError_t launch_step2(const Cell<real> &c, const Step2Shape &g, hipStream_t s);

// Population storage (pop2_kernels.hip): the same three.
template <typename real>
bool pop2_takes(const Cell<real> &c);
template <typename real>
Step2Shape pop2_shape(int nx, int ny, int nz, int nphase);
template <typename real>
hipError_t launch_pop2(const Cell<real> &c, const Step2Shape &g, hipStream_t s);

// The same for many cells of moment storage in one launch.  tiles: int4 (cell, first row, first
// plane, rows | planes << 16), one block each, rows = 0: an empty tile; the
// table holds 8 * chunk tiles and block b takes tile (b % 8) * chunk + b / 8.
struct Step2Batch {
    int vec = 0;       // 0: the batch takes single steps
    int threads = 0, planes = 0;
    bool ragged = false;
    int gaxis = 0;     // the cells' gradient axis
    size_t lds = 0, state_bytes = 0;
};

struct Step2Extent {
    int nx, ny, nz, nphase, gaxis;
};

// the fastest block size and chunk length for these cells by the model
template <typename real>
Step2Batch step2_batch_shape(const Step2Extent *cells, int n);

// rows of a cell's tiles under that shape
template <typename real>
int step2_batch_rows(const Step2Batch &g, const Step2Extent &c);

template <typename real>
hipError_t launch_batch2(const Cell<real> *cells, const int4 *tiles, int chunk, const Step2Batch &g, int parity,
                         hipStream_t s);

}  // namespace mrt
