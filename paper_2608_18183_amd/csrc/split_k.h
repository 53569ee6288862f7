// How the O and W2 products cut their contraction, and the room their partial
// sums take (host code, no device types).
#pragma once
#include <algorithm>
#include <cstddef>

namespace hbsjd {

// K parts of a product of N x K weights over up to m_cap rows
inline int split_for(int m_cap, int N, int K) {
    // enough (tile, split) pairs for about two 64x64 workgroups per CU, at most
    // four parts, each a whole number of 64-deep steps
    const long tiles = (long)((m_cap + 63) / 64) * (N / 64);
    int want = (int)((512 + tiles - 1) / tiles);
    want = want < 1 ? 1 : (want > 4 ? 4 : want);
    const int steps = K / 64;
    int sp = 1;
    for (int c = 1; c <= want; ++c)
        if (steps % c == 0) sp = c;
    return sp;
}

// Rows of d partial sums that launches of rows_a and of rows_b rows (0: no such
// launch) need, of a model of width d and MLP width f. K parts times rows is
// not monotonic in the rows: a launch of fewer rows may cut K into more parts
// and need more room than one of more rows. The fp32 path writes one part.
inline size_t partial_sum_rows(long rows_a, long rows_b, int d, int f, bool f16) {
    size_t room = 0;
    for (const long rows : {rows_a, rows_b})
        if (rows > 0) {
            const int parts =
                f16 ? std::max(split_for((int)rows, d, d), split_for((int)rows, d, f)) : 1;
            room = std::max(room, (size_t)parts * rows);
        }
    return room;
}

}  // namespace hbsjd
