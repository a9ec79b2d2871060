// Internal interface of the kernel that carries small cells through several
// steps per launch (box_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "lbm_internal.h"

namespace mrt {

struct BoxShape {
    int steps = 0;  // at most this many steps per launch; 0: the cell is not small
    int ty = 0, tz = 0, threads = 0;
};

// the fastest shape by the measured model, if it beats `other` us per step
template <typename real>
BoxShape box_shape(int nx, int ny, int nz, int nphase, double other);

// whether storage and boundaries allow it
template <typename real>
bool box_takes(const Cell<real> &c);

// state at t -> state at t + steps, 1 <= steps <= g.steps
template <typename real>
hipError_t launch_box(const Cell<real> &c, const BoxShape &g, int steps, hipStream_t s);

}  // namespace mrt
