// Host-side check of the order of workgroups that hold a limb each (whole_decode in csrc/ntt.h): every limb of every instance
// comes once, and no XCD (workgroup number mod 8) gets more than a quarter above its even share, rounded up to whole workgroups.
// Prints "OK <count>" or the first failure.
#include <stdio.h>
#include <vector>
#include "../../paper_2310_16530_amd/csrc/ntt.h"

int main() {
    long n = 0;
    for (u32 limbs = 1; limbs <= 70; limbs++)
        for (u32 insts : {1u, 2u, 3u, 7u, 8u, 16u, 33u, 128u}) {
            std::vector<int> seen(limbs * insts);
            u32 per[8] = {};
            const u32 grid = (limbs + 7) / 8 * 8 * insts;
            for (u32 b = 0; b < grid; b++) {
                u32 l, inst;
                if (!whole_decode(b, insts, limbs, l, inst)) continue;
                if (l >= limbs || inst >= insts || seen[l * insts + inst]++) { printf("limbs %u inst %u: block %u\n", limbs, insts, b); return 1; }
                per[b & 7]++;
            }
            u32 total = 0, most = 0;
            for (u32 x : per) total += x, most = x > most ? x : most;
            if (total != limbs * insts) { printf("limbs %u inst %u: %u decoded\n", limbs, insts, total); return 1; }
            if (most > (total * 5 + 31) / 32 && most > (total + 7) / 8) { printf("limbs %u inst %u: %u on one XCD of %u\n", limbs, insts, most, total); return 1; }
            n++;
        }
    printf("OK %ld\n", n);
    return 0;
}
