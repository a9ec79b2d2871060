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

}  // namespace mrt
