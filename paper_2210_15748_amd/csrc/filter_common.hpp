// What the kernels that compare vectors with centroids share (filter_kernels.hip, filter_groups.hip): the layout of the re-ordered
// centroids and of their constants is described at filter_prep_kernel.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

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

// Assignment by groups of centroids (filter_groups.hip): what its launches tell each other.
constexpr uint32_t GROUP_TRIAL = 4096;   // vectors that tell whether the groups pay
struct GroupCtl {
    uint32_t groups;    // groups of centroids
    uint32_t radius2;   // largest squared distance of a centroid from its group's leader
    uint32_t easy;      // vectors of the trial that need one group only
    uint32_t rest;      // vectors left to a comparison with every centroid
};
__host__ __device__ inline uint32_t groups_room(uint32_t K) { return K / 3; }   // more groups are not made
// Groups in vain: too many of them, or too many vectors near to more than one.  Reading a group per vector and the list of the rest cost
// something too, hence 0.7 and not 1.
__device__ __forceinline__ bool groups_pay(const GroupCtl& c, uint32_t K) {
    if (c.groups == 0 || c.groups > groups_room(K)) return false;
    return (uint64_t)(GROUP_TRIAL - c.easy) * K + (uint64_t)GROUP_TRIAL * c.groups <= (uint64_t)GROUP_TRIAL * K / 10 * 7;
}

}  // namespace dessert
