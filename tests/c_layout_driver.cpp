// Walks every LDS read of c_top_kernel's vectors (kernels_ct.hip) for every order count and
// value size, with the layout functions that the kernel itself uses (c_layout.h).  Prints the
// first read outside its slab and returns 1, else the number of reads walked.
#include <algorithm>
#include <cstdio>

#include "c_layout.h"

int main() {
    using namespace pvi;
    long long reads = 0;
    for (int B : {4, 8})
        for (int R = 1; R <= 24; ++R) {
            const int RC = c_tri_bound(R), row = kTopLo * B, waves = (2 * R - 1 + 3) / 4;
            if (R > RC || R < c_tri_least(RC)) return std::printf("bound of R=%d\n", R), 1;
            const int slab = (int)c_top_slab(R, B);
            // staging: whole instructions of c_top_rows rows
            for (int i = 0; i < R * RC; i += c_top_rows(B))
                if (i * row + 1024 > slab) return std::printf("staging R=%d\n", R), 1;
            if (2 * slab > (int)c_top_lds(R, B) || c_top_lds(R, B) > 159 * 1024)
                return std::printf("size R=%d\n", R), 1;
            for (int ym = 0; ym < R; ++ym)
                for (int w = 0; w < waves; ++w)
                    for (int lane = 0; lane < 64; ++lane) {
                        const int tb = 4 * w - ym, t = tb + lane / kTopLo, nr = R - ym;
                        const int rlo = std::max(0, tb - (R - 1)), rhi = std::min(nr - 1, tb + 3);
                        if (rlo > rhi) continue;
                        const int base = (ym & 1) * slab + lane % kTopLo * B;
                        const int top = base + (R - 1) * row;
                        for (int b = 0; b < RC; b += kTriLoad)
                            for (int s = b; b <= rhi && s < b + kTriLoad && s < RC; ++s, ++reads) {
                                const int e = c_top_entry(s, R, RC);
                                const int at = std::min(std::max(base + (t - s) * row, base), top) +
                                               e * RC * row;
                                if (at < (ym & 1) * slab ||
                                    at + B > (ym & 1) * slab + R * RC * row || (s < R && e != s))
                                    return std::printf("read B=%d R=%d ym=%d s=%d: %d of %d\n", B, R,
                                                       ym, s, at, 2 * slab),
                                           1;
                            }
                    }
        }
    std::printf("%lld\n", reads);
    return 0;
}
