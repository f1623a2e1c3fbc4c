// Shapes of the antidiagonal kernels' tables (kernels_ct.hip).  Plain C++ (no HIP), so that a
// host program can walk every read of a slab.
#pragma once

#include <cstddef>

namespace pvi {

// Compile-time bound of the kernels' rows for R <= 24 orders, and the entries of one level's
// packed weights (whole registers of 16).  A slab's rows and reads go by the bound, so 9 to 12
// orders have one of their own: FP64 sweeps of m = 6 with rows of 16 and of 12 take 258 and
// 229 us at 9 orders (the plain kernels 233), 842 and 788 at 11 (797).
constexpr int c_tri_bound(int R) {
    return R <= 8 ? 8 : R <= 12 ? 12 : R <= 16 ? 16 : R <= 21 ? 21 : 24;
}
constexpr size_t c_tri_weights(int R) {
    return (size_t)((c_tri_bound(R) * (c_tri_bound(R) + 1) / 2 + 15) / 16 * 16);
}
// The fewest orders whose rows have the bound rc.
constexpr int c_tri_least(int rc) {
    return rc == 8 ? 1 : rc == 12 ? 9 : rc == 16 ? 13 : rc == 21 ? 17 : 22;
}

// The vectors D[s] of a lane are loaded eight entries at a time (kTriLoad), so entries
// s >= R are loaded too; no row that exists uses them.  A slab holds R of them, with rows of
// rc: this is the place in it that entry s is loaded from, always inside.  (Entries below
// c_tri_least(rc) need no look at R: their place stays a constant of the instruction.)
constexpr int kTriLoad = 8;
constexpr int c_top_entry(int s, int R, int rc) {
    return s < c_tri_least(rc) || s < R ? s : R - 1;
}

// c_top_kernel: low-digit values per workgroup, rows that one 16-byte-a-lane staging
// instruction moves, and bytes of one slab of R x rc rows, whole staging instructions.
constexpr int kTopLo = 16;
constexpr int c_top_rows(int value_bytes) { return 64 * 16 / (kTopLo * value_bytes); }
constexpr size_t c_top_slab(int R, int value_bytes) {
    return (size_t)((R * c_tri_bound(R) + c_top_rows(value_bytes) - 1) / c_top_rows(value_bytes)) *
           c_top_rows(value_bytes) * kTopLo * value_bytes;
}
// Two slabs, then best and second best value and the best order of R x kTopLo states.
constexpr size_t c_top_lds(int R, int value_bytes) {
    return 2 * c_top_slab(R, value_bytes) +
           (size_t)R * kTopLo * (2 * sizeof(double) + sizeof(int));
}

}  // namespace pvi
