// What the kernels that compare vectors with centroids share (filter_kernels.hip, filter_groups.hip): the layout of the re-ordered
// centroids and of their constants is described at filter_prep_kernel.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "group_cost.hpp"

namespace dessert {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int FILTER_TG = 4;                      // centroid tiles per LDS group
constexpr int32_t FILTER_PAD_INIT = -(1 << 23);   // rows past the last centroid start from it: a value of -2^24

// accumulator register r of lane half g holds tile row 8*(r/4) + 4*g + r%4
__host__ __device__ inline uint32_t tile_row(uint32_t r, uint32_t g) { return 8 * (r / 4) + 4 * g + (r % 4); }

__device__ __forceinline__ int32_t max3(int32_t a, int32_t b, int32_t c) {  // one v_max3_i32
    const int32_t ab = a > b ? a : b;
    return ab > c ? ab : c;
}

__device__ __forceinline__ int32_t med3_i32(int32_t x, int32_t y, int32_t z) {
    int32_t r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(y), "v"(z));
    return r;
}

}  // namespace dessert
