// Host-side check of the integer butterflies and products of csrc/modarith.h (IntAr) against 128-bit integers, at the ends of the ranges
// that they accept: the negative modulus, the forward and inverse butterflies, the last inverse stage and the ends of a sum of products.
// Prints "OK <count>" or the first failure.
#include <stdio.h>
#include <stdlib.h>
#include "../../paper_2310_16530_amd/csrc/modarith.h"

static u64 rng_state = 0x9E3779B97F4A7C15ull;
static u64 rnd() { rng_state ^= rng_state << 13; rng_state ^= rng_state >> 7; rng_state ^= rng_state << 17; return rng_state; }
static u64 mulm(u64 a, u64 b, u64 q) { return (u64)((u128_t)a * b % q); }
static u64 shoup(u64 w, u64 q) { return (u64)(((u128_t)w << 64) / q); }
static u64 edge(u64 below) { const u64 r = rnd(); return r % 3 == 0 ? below - 1 - (r >> 8) % 3 : r % 3 == 1 ? (r >> 8) % 3 : rnd() % below; }
#define FAIL(what) return printf("%s q=%llu\n", what, (unsigned long long)q), 1

int main(int argc, char** argv) {
    unsigned long long count = 0;
    for (int i = 1; i < argc; i++) {
        const u64 q = strtoull(argv[i], 0, 10);
        PrimeConst p = {};
        u64 x = 1;
        for (int k = 0; k < 6; k++) x *= 2 - q * x;  // q^-1 modulo 2^64
        p.q = q, p.qneg = (u64)0 - x, p.r1 = (u64)(((u128_t)1 << 64) % q), p.r1_p = shoup(p.r1, q), p.r2 = mulm(p.r1, p.r1, q);
        const IntAr::Mod m = IntAr::mod(p);
        if (m.nq + q != 0) FAIL("negative modulus");
        for (int it = 0; it < 200000; it++) {
            const u64 w = edge(q), any = it & 1 ? rnd() : ~(u64)0 - rnd() % 3;
            const u64 r = mul_shoup_neg(any, w, shoup(w, q), m.nq);
            if (r >= 2 * q || r != mul_shoup_lazy(any, w, shoup(w, q), q) || r % q != mulm(any % q, w, q)) FAIL("product");
            const IntAr::Tw t = {w, shoup(w, q)};
            for (int red = 0; red < 2; red++) {
                u64 X = edge(red ? 8 * q : 6 * q), Y = edge(8 * q);
                const u64 x0 = X % q, y0 = mulm(Y % q, w, q);
                red ? IntAr::bfly_fwd<true>(X, Y, t, m) : IntAr::bfly_fwd<false>(X, Y, t, m);
                if (X >= 8 * q || Y >= 8 * q || X % q != (x0 + y0) % q || Y % q != (x0 + q - y0) % q) FAIL("forward butterfly");
            }
            const u64 a = edge(2 * q), b = edge(2 * q), d = (a % q + q - b % q) % q;
            u64 X = a, Y = b;
            IntAr::bfly_inv(X, Y, t, m);
            if (X >= 2 * q || Y >= 2 * q || X % q != (a + b) % q || Y % q != mulm(d, w, q)) FAIL("inverse butterfly");
            const u64 sy = edge(q);
            const InvScale s = {w, shoup(w, q), sy, shoup(sy, q), 0, 0};
            u64 ox, oy;
            X = a, Y = b;
            IntAr::bfly_inv_last(X, Y, s, m, SRC_CANON, ox, oy);
            if (ox != mulm((a + b) % q, w, q) || oy != mulm(d, sy, q)) FAIL("last inverse stage");
            const u64 f = IntAr::acc_finish(a, m), f2 = IntAr::acc_finish2(a, m);
            if (f >= 2 * q || f % q != mulm(a % q, p.r1, q) || f2 >= 2 * q || f2 % q != mulm(a % q, p.r2, q)) FAIL("end of a sum");
            count++;
        }
    }
    printf("OK %llu\n", count);
    return 0;
}
