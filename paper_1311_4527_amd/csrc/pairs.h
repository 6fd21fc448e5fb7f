// The cyclic walk over the pairs of p agents (a batch's groups): blocks of 64
// agents against offsets, so that lanes stay full.
#pragma once
#include <hip/hip_runtime.h>

namespace twa {

constexpr int kGroupCpw = 2;  // break-point intervals per item of a group's collision walk
constexpr int kGroupSpan = 4; // offsets per item of the cyclic walk

// items of the cyclic walk per block of intervals
__host__ __device__ __forceinline__ int cyclic_items(int p) {
    return ((p + 63) >> 6) * ((p / 2 + kGroupSpan - 1) / kGroupSpan);
}

// Pair of lane `lane` at offset d of block b; false where it stands for none.
__host__ __device__ __forceinline__ bool group_pair(int p, int b, int d, int lane, int *i, int *j) {
    const int x = 64 * b + lane;
    if (x >= p || d > p / 2 || (2 * d == p && x >= d)) return false;
    const int y = x + d >= p ? x + d - p : x + d;
    *i = x < y ? x : y, *j = x < y ? y : x;
    return true;
}

} // namespace twa
