// Host-side check of what narrow primes (csrc/modarith.h) leave unreduced, against 128-bit integers: eight forward stages in a row from
// canonical words and from |x| <= q/2, their range, five products of the results with residues added up, and the product that ends a
// ModDown.  Prints "OK <count>" or the first failure.
#include <stdio.h>
#include <stdlib.h>
#include <math.h>
#include "../../paper_2310_16530_amd/csrc/modarith.h"

typedef __int128 i128;
static u64 rng_state = 0x2545F4914F6CDD1Dull;
static u64 rnd() { rng_state ^= rng_state << 13; rng_state ^= rng_state >> 7; rng_state ^= rng_state << 17; return rng_state; }
static long long imod(i128 x, long long q) { long long r = (long long)(x % q); return r < 0 ? r + q : r; }
#define FAIL(...) return printf(__VA_ARGS__), printf("\n"), 1

static int check_prime(u64 q, unsigned long long* count) {
    PrimeConst pc = {};
    pc.q = q, pc.qd = (double)q, pc.qinv = 1.0 / (double)q, pc.fp = 1, pc.narrow = q <= CKKS_FP_NARROW_MAX;
    const FpAr::Mod m = FpAr::mod(pc);
    if (!FpAr::narrow(m)) FAIL("%llu is not narrow", (unsigned long long)q);
    const double qd = (double)q;
    for (int it = 0; it < 4000; it++) {
        const bool centred = it & 1;
        static double x[256];
        static long long ref[256];
        for (int k = 0; k < 256; k++) {
            const long long half = (long long)(q / 2);
            const long long v = centred ? ((it & 2) ? ((rnd() & 1) ? half : -half) : (long long)(rnd() % q) - half)
                                        : (long long)((it & 2) ? q - 1 - rnd() % 3 : rnd() % q);
            x[k] = (double)v, ref[k] = imod(v, (long long)q);
        }
        for (int s = 0; s < 8; s++) {
            const int d = 128 >> s;
            for (int k = 0; k < 256; k++) {
                if (k & d) continue;
                // residues whose products leave a remainder near q/2 make the sums grow: try a few
                u64 w = rnd() % q;
                if (it & 4)
                    for (int t = 0; t < 6; t++) {
                        const u64 c = rnd() % q;
                        if (fabs(x[k] + FpAr::mulmod_lazy(x[k + d], (double)c, m)) > fabs(x[k] + FpAr::mulmod_lazy(x[k + d], (double)w, m))) w = c;
                    }
                const FpAr::Tw tw = {(double)w};
                FpAr::bfly_fwd<false>(x[k], x[k + d], tw, m);
                const long long t = imod((i128)ref[k + d] * (i128)w, (long long)q), X = ref[k];
                ref[k] = imod((i128)X + t, (long long)q), ref[k + d] = imod((i128)X - t, (long long)q);
            }
        }
        for (int k = 0; k < 256; k++) {
            const double most = centred ? 10.5 : 12.6;
            if (x[k] != floor(x[k]) || fabs(x[k]) > most * qd) FAIL("range q=%llu x=%.0f", (unsigned long long)q, x[k]);
            if (imod((i128)(long long)x[k], (long long)q) != ref[k] || (long long)FpAr::canon(x[k], m) != ref[k]) FAIL("stages q=%llu k=%d", (unsigned long long)q, k);
            double same[1] = {x[k]};
            FpAr::mid_reduce(same, m);
            if (same[0] != x[k]) FAIL("a narrow prime reduces");
        }
        // five products on what a sum keeps after a reduction
        for (int k = 0; k + 5 <= 256; k += 5) {
            if (!centred) break;
            double acc = (double)(q / 2);
            i128 want = (i128)(long long)acc;
            for (int j = 0; j < 5; j++) {
                const u64 key = (it & 2) ? q - 1 - rnd() % 3 : rnd() % q;
                const double p = FpAr::mulmod_lazy(x[k + j], (double)key, m);
                if (fabs(p) > 2.6 * qd) FAIL("product q=%llu p=%.0f", (unsigned long long)q, p);
                FpAr::acc_mac(acc, x[k + j], key, m);
                want += (i128)(long long)x[k + j] * (i128)key;
            }
            if (fabs(acc) > 13.6 * qd || fabs(acc) >= 9007199254740992.0) FAIL("sum q=%llu acc=%.0f", (unsigned long long)q, acc);
            if (imod((i128)(long long)acc, (long long)q) != imod(want, (long long)q)) FAIL("sum q=%llu", (unsigned long long)q);
            const double fin = FpAr::acc_finish(acc, m);
            const u64 pinv = rnd() % q;
            const double end = FpAr::mulmod_lazy(fin - x[k], (double)pinv, m);
            if (imod((i128)(long long)end, (long long)q) != imod((i128)(long long)(fin - x[k]) * (i128)pinv, (long long)q)) FAIL("end q=%llu", (unsigned long long)q);
        }
        (*count)++;
    }
    return 0;
}

int main(int argc, char** argv) {
    unsigned long long count = 0;
    for (int i = 1; i < argc; i++)
        if (check_prime(strtoull(argv[i], nullptr, 10), &count)) return 1;
    printf("OK %llu\n", count);
    return 0;
}
