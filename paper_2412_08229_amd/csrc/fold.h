// Placement of the first layer's input rows for the reflection fold, shared
// by the matrix-core network kernels: the 28 rows (27 moments and the bias
// row 27) grouped by the parity class of their Hermite multi-index into 10
// K-steps of 4 slots.
#pragma once

#include "d3q27.h"

namespace nco {

constexpr int KSTEPS = 10;          // K-steps of the eight parity-class products
constexpr int GT_STRIDE = 12;       // ints per (axis permutation, lane group) in the gather table
constexpr int GT_ENTRIES = 6 * 4 * GT_STRIDE;

// K-step -> parity class ci = cx + 2 cy + 4 cz of the W1 rows it holds.
__host__ __device__ constexpr int step_class(int st) {
    constexpr int c[KSTEPS] = {0, 0, 0, 1, 2, 4, 3, 5, 6, 7};
    return c[st];
}

// Parity class of row k of M (the bias row 27 and padding rows count as 0).
inline int row_class(int k) {
    if (k >= 27) return 0;
    const int t = row_tensor(k);
    return (t % 3) % 2 + 2 * (((t / 3) % 3) % 2) + 4 * ((t / 9) % 2);
}

// Canonical placement of the 28 K rows into the 10 K-steps x 4 slots; -1
// marks an empty slot.
inline void class_slots(int slot_row[KSTEPS][4]) {
    int fill[KSTEPS] = {0};
    for (int st = 0; st < KSTEPS; ++st)
        for (int q = 0; q < 4; ++q) slot_row[st][q] = -1;
    for (int k = 0; k < 28; ++k) {
        const int ci = row_class(k);
        for (int st = 0; st < KSTEPS; ++st)
            if (step_class(st) == ci && fill[st] < 4) {
                slot_row[st][fill[st]++] = k;
                break;
            }
    }
}

// XCD-aware block order: workgroups are dispatched to the 8 XCDs in turn
// (workgroup b to XCD b mod 8), each XCD with its own L2.  Block b takes
// the logical block that makes the blocks of one XCD a contiguous run of
// the lattice (XCD x: its i-th block is the i-th of the x-th run), so the
// halo rows that neighbouring blocks share, and the second pull after the
// network, meet in that XCD's L2.  A bijection of [0, n): the results do
// not depend on it.
__device__ __forceinline__ int xcd_block(int b, int n) {
    constexpr int XCDS = 8;
    const int x = b % XCDS, i = b / XCDS, q = n / XCDS, r = n % XCDS;
    return x * q + min(x, r) + i;
}

}  // namespace nco
