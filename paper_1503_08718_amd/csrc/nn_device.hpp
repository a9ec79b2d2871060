// Types and voxel addressing shared by the warm-start network's kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "nn_internal.h"

namespace mrt {

typedef __bf16 bf16;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8 zero8() {
    bf16x8 z;
#pragma unroll
    for (int e = 0; e < 8; e++) z[e] = (bf16)0.0f;
    return z;
}

}  // namespace mrt
