// Host-side check of the unreduced sums of csrc/modarith.h (Wide: FpAr pairs of doubles, IntAr 128 bits) and of the
// recombination of a base conversion's digit sums (conv_recombine), against 128-bit integer arithmetic.  x86-64 FMA and
// CDNA4 FMA are both IEEE-754 binary64, so exactness shown here is exactness on the GPU.
// Arguments: moduli.  Prints "OK <count>" or the first failure.
#include <stdio.h>
#include <stdlib.h>
#include <math.h>
#include "../../paper_2310_16530_amd/csrc/modarith.h"

typedef __int128 i128;
typedef unsigned __int128 u128;
static u64 rng_state = 0x9E3779B97F4A7C15ull;
static u64 rnd() { rng_state ^= rng_state << 13; rng_state ^= rng_state >> 7; rng_state ^= rng_state << 17; return rng_state; }
static u64 imod(i128 x, u64 q) { i128 r = x % (i128)q; return (u64)(r < 0 ? r + q : r); }
static u64 pick(u64 q, int how) { return how == 0 ? q - 1 : how == 1 ? rnd() % 2 : how == 2 ? q - 1 - rnd() % 5 : rnd() % q; }
static void digits(long long v, int (&d)[8]) {  // v = sum d_g 256^g, d_g in [-128, 127]
    for (int g = 0; g < 8; g++) {
        int x = (int)(signed char)(v & 0xff);
        d[g] = x;
        v = (v - x) >> 8;
    }
}
static PrimeConst prime_const(u64 q) {
    PrimeConst p = {};
    p.q = q, p.qd = (double)q, p.qinv = 1.0 / (double)q, p.fp = q < CKKS_FP_PRIME_LIMIT;
    u64 x = q;
    for (int i = 0; i < 6; i++) x *= 2 - q * x;
    p.qneg = (u64)0 - x;
    p.r1 = (u64)(((u128)1 << 64) % q);
    return p;
}

int main(int argc, char** argv) {
    unsigned long long count = 0;
    for (int a = 1; a < argc; a++) {
        const u64 q = strtoull(argv[a], nullptr, 10);
        const PrimeConst pc = prime_const(q);
        for (int it = 0; it < 60000; it++) {
            // sums of every allowed number of products
            const u32 most = pc.fp ? FpAr::wide_terms : IntAr::wide_terms, n = 1 + rnd() % most;
            FpAr::Wide wf = FpAr::wide_zero();
            IntAr::Wide wi = IntAr::wide_zero();
            u64 want = 0;
            for (u32 k = 0; k < n; k++) {
                const u64 x = pick(q, it % 5), y = pick(q, (it / 5) % 5);
                want = (u64)((want + (u128)x * y) % q);
                if (pc.fp) FpAr::wide_mac(wf, x, y);
                else IntAr::wide_mac(wi, x, y);
            }
            if (pc.fp) {
                const double r = FpAr::wide_reduce(wf, FpAr::mod(pc));
                if (r != floor(r) || fabs(r) > 0.5 * (double)q + 1 || imod((i128)(long long)r, q) != want) {
                    printf("FpAr wide sum q=%llu n=%u r=%.0f\n", (unsigned long long)q, n, r); return 1; }
            } else {
                const u64 r = IntAr::wide_reduce(wi, IntAr::mod(pc));
                if (r >= 2 * q || (u64)((u128)r % q * pc.r1 % q) != want) {
                    printf("IntAr wide sum q=%llu n=%u\n", (unsigned long long)q, n); return 1; }
            }
            count++;
        }
        for (int it = 0; it < 20000; it++) {
            // a conversion from 1 .. 17 sources below 2^61
            const int ns = 1 + (int)(rnd() % 17);
            int s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            u64 want = 0;
            for (int i = 0; i < ns; i++) {
                const u64 y = it % 4 == 0 ? (1ull << 61) - 1 - rnd() % 3 : it % 4 == 1 ? 0x1f7f7f7f7f7f7f7full : rnd() >> 3, hat = pick(q, it % 5);
                int dy[8];
                digits((long long)y, dy);
                u64 c = hat;
                for (int b = 0; b < 8; b++) {
                    int dc[8];
                    digits(c > q / 2 ? (long long)c - (long long)q : (long long)c, dc);
                    for (int g = 0; g < 8; g++) s[g] += dc[g] * dy[b];
                    c = (u64)((u128)c * 256 % q);
                }
                want = (u64)((want + (u128)(y % q) * hat) % q);
            }
            v16i v = {s[0], s[1], s[2], s[3], s[4], s[5], s[6], s[7], s[0], s[1], s[2], s[3], s[4], s[5], s[6], s[7]};
            const int o = it & 1 ? 8 : 0;
            if (pc.fp) {
                const double r = conv_recombine(v, o, FpAr::mod(pc), pc);
                if (s[7] != 0 || r != floor(r) || fabs(r) > 0.51 * (double)q + 1 || imod((i128)(long long)r, q) != want) {
                    printf("FpAr recombination q=%llu ns=%d r=%.0f\n", (unsigned long long)q, ns, r); return 1; }
            } else {
                const u64 r = conv_recombine(v, o, IntAr::mod(pc), pc);
                if (5 * (u128)r <= 2 * (u128)q || 5 * (u128)r >= 8 * (u128)q || r % q != want) { printf("IntAr recombination q=%llu ns=%d\n", (unsigned long long)q, ns); return 1; }
            }
            count++;
        }
    }
    printf("OK %llu\n", count);
    return 0;
}
