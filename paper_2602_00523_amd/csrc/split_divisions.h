// Divisions of the sizes that decide how attention is cut into workgroups, also for the host, which checks them over their range.
#pragma once
#include <hip/hip_runtime.h>

namespace sage {

// x / y for 0 <= x, 1 <= y, where quotient(x, y) is by_reciprocal(x, a reciprocal of y that is at most one ulp off): below 2^21,
// x + 1/2 over y is at least 1/2 / y away from an integer, and two roundings and that reciprocal move it by less than
// (x + 1/2) / y * 2^-22.
__host__ __device__ __forceinline__ int by_reciprocal(int x, float reciprocal) {
    return static_cast<int>((static_cast<float>(x) + 0.5f) * reciprocal);
}
template <class Quotient>
__host__ __device__ __forceinline__ int div_floor(int x, int y, Quotient quotient) {
    if (__builtin_expect(x < (1 << 21), 1)) return quotient(x, y);   // (uniform, and what there is: 67 million positions)
    return x / y;
}
// x / groups for x <= 256 and up to four column groups
__host__ __device__ __forceinline__ int per_group(int x, int groups) {
    return (x * (groups == 1 ? 65536 : groups == 2 ? 32768 : groups == 3 ? 21846 : 16384)) >> 16;   // (no branches)
}

}  // namespace sage
