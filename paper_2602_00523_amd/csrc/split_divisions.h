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

// x / y for 0 <= x < 2^24 and 2 <= y <= 256 as the upper word of x times inverse(y): the inverse is less than y / 2^32 of itself too large,
// which x times moves the quotient by less than 1 / y.
__host__ __device__ __forceinline__ unsigned inverse(int y) { return static_cast<unsigned>(((1ull << 32) + static_cast<unsigned>(y) - 1) / static_cast<unsigned>(y)); }
__host__ __device__ __forceinline__ int by_product(int x, unsigned inverse_of_y) {
    return static_cast<int>((static_cast<unsigned long long>(static_cast<unsigned>(x)) * inverse_of_y) >> 32);
}
// x / cost rounded up for 0 <= x, x + cost below 2^31 and a cost of 1, 3 or 4 (the factors are 2^31 over the cost, rounded up)
__host__ __device__ __forceinline__ int div_up_by_cost(int x, int cost) {
    const unsigned up = static_cast<unsigned>(x + cost - 1);
    return static_cast<int>((2ull * up * (cost == 1 ? 0x80000000u : cost == 3 ? 0x2AAAAAABu : 0x20000000u)) >> 32);
}

}  // namespace sage
