// Host-side check of the rule that lets four wavefronts share a row where several giant-step sums are formed (csrc/kernels.h, __host__
// __device__).  Prints "OK" or the first failure.
#include <stdio.h>
#include "../../paper_2310_16530_amd/csrc/kernels.h"

#define FAIL(...) return printf(__VA_ARGS__), printf("\n"), 1

int main() {
    for (u32 rows = 1; rows <= 20000; rows++)
        for (u32 n = 1; n <= CKKS_DH_CHUNK; n++) {
            const u32 w = sums_waves(rows, n);
            if (w != 1 && w != 4) FAIL("%u wavefronts", w);
            if (n == 1 && w != 1) FAIL("one rotation shared, %u rows", rows);
            if (w == 4 && rows >= 1792) FAIL("%u rows, %u rotations shared", rows, n);
            if (w == 4 && (sums_waves(rows - 1, n) != 4 && rows > 1)) FAIL("%u rows, %u rotations: fewer rows not shared", rows, n);
        }
    // the ends of the ranges that were measured
    if (sums_waves(768, 2) != 4 || sums_waves(960, 2) != 1) FAIL("two rotations");
    if (sums_waves(1024, 3) != 4 || sums_waves(1536, 3) != 1) FAIL("three rotations");
    if (sums_waves(1728, 4) != 4 || sums_waves(1728, 16) != 4) FAIL("four and more");
    printf("OK\n");
    return 0;
}
