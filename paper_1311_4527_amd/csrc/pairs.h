// Walks over the pairs i < j of p agents by waves of 64 lanes: the cyclic one of
// a batch's groups (blocks of 64 agents against offsets, so that lanes stay
// full), and those of the persistent batch by rows of the pair triangle.
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

// Rows of the pair triangle that a wave of the activity-bit stream takes
// together (coll_rows_bits); 1024 / 2048 agents and 32 walls: 2 rows 14.8 / 45.6
// us, 4 rows 14.0 / 40.7, 6 rows 14.5 / 39.3.
constexpr int kRows = 4;

// Tasks (kRows rows from a multiple of kRows, J) of the activity-bit walk in
// chunk column J before the last (64 J + 63 rows), and in all of an interval.
__host__ __device__ __forceinline__ int walk_tasks(int J) { return 64 / kRows * (J + 1); }
__host__ __device__ __forceinline__ int bits_walk(int p) {
    const int last = (p - 1) >> 6;
    return 32 / kRows * last * (last + 1) + ((64 * last + 63 < p - 1 ? 64 * last + 63 : p - 1) + kRows - 1) / kRows;
}
// Task w of the walk: rows from *i0 on of column *J.
__host__ __device__ __forceinline__ void bits_task(int p, int w, int *i0, int *J) {
    for (*J = 0; *J < (p - 1) >> 6 && w >= walk_tasks(*J); ++*J) w -= walk_tasks(*J);
    *i0 = kRows * w;
}

// Tasks of the row chunks (i, i + 1 + 64 k + lane) of p agents, and the one that
// comes w-th: the 64 rows of one chunk each, the 64 of two, ..., for each k
// (found without a division: the walk is short, and waits for it).
__host__ __device__ __forceinline__ int pair_chunks(int p) {
    const int c = (p - 1 + 63) >> 6; // of row 0
    return 32 * c * (c - 1) + c * (p - 1 - 64 * (c - 1));
}
__host__ __device__ __forceinline__ void pair_chunk(int p, int w, int *i, int *j0) {
    int c = 1, k = 0;
    for (; w >= 64 * c; ++c) w -= 64 * c;
    const int left = p - 1 - 64 * (c - 1), rows = left < 64 ? left : 64;
    for (; w >= rows; ++k) w -= rows;
    *i = p - 2 - 64 * (c - 1) - w;
    *j0 = *i + 1 + 64 * k;
}

} // namespace twa
