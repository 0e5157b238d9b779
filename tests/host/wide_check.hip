// Host-side check of the unreduced sums of csrc/modarith.h (Wide: FpAr pairs of doubles, IntAr 128 bits), of longer sums joined from
// them that then meet plaintexts (join_part, acc_mac_wide), and of the recombination of a base conversion's digit sums
// (conv_recombine), against 128-bit integer arithmetic.  x86-64 FMA and
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
    p.r1 = (u64)(((u128)1 << 64) % q), p.r1_p = (u64)(((u128)p.r1 << 64) / q);
    return p;
}

// up to 32 rotations, each a sum of 1 .. 128 digit products times a plaintext, as dh_accum_kernel adds them for several giant steps.
// how = 0: operands at random; else every part of a sum ends at the same value near +q/2 (1, 2: the same for all
// rotations) or -q/2 (3), the farthest from zero that many parts can take the sum
template <class AR>
static bool joined_sums(const PrimeConst& pc, u32 terms, u32 rotations, int how) {
    const u64 q = pc.q;
    const typename AR::Mod m = AR::mod(pc);
    typename AR::T acc = AR::acc_zero();
    u64 want = 0;
    const u64 pt0 = rnd() % q;
    for (u32 r = 0; r < rotations; r++) {
        typename AR::T sum = AR::acc_zero();
        typename AR::Wide w = AR::wide_zero();
        u64 value = 0, part = 0;
        for (u32 j = 0, in_sum = 0; j < terms; j++) {
            const bool last = j + 1 == terms, ends = in_sum + 1 == AR::wide_terms || last;
            u64 x = pick(q, how ? 3 : (int)(rnd() % 4)), y = pick(q, how ? 3 : (int)(rnd() % 4));
            if (how && ends) {  // 1 * what is missing
                const u64 goal = how == 3 ? q - (q - 1) / 2 + rnd() % 3 : (q - 1) / 2 - rnd() % 3;
                x = 1, y = (goal + q - part) % q;
            }
            const u64 p = (u64)((u128)x * y % q);
            value = (value + p) % q, part = (part + p) % q;
            AR::wide_mac(w, x, y);
            if (++in_sum == AR::wide_terms || last) {
                join_part<AR>(sum, AR::wide_reduce(w, m), last, m);
                w = AR::wide_zero(), in_sum = 0, part = 0;
            }
        }
        if (AR::is_fp && fabs((double)sum) > (double)q + 2) return false;
        u64 pt = rnd() % q;
        if (how == 1) pt = pt0;
        for (int d = 0; how > 1 && d < 64; d++) {  // of 64, the one whose lazily reduced product is the largest
            const u64 other = rnd() % q;
            typename AR::T x = AR::acc_zero(), y = AR::acc_zero();
            AR::acc_mac_wide(x, sum, pt, m);
            AR::acc_mac_wide(y, sum, other, m);
            if (y > x) pt = other;
        }
        AR::acc_mac_wide(acc, sum, pt, m);
        want = (want + (u64)((u128)value * pt % q)) % q;
        if ((r & 7) == 7) acc = AR::acc_fold(acc, m);
    }
    // IntAr sums carry 2^-128 through the two reductions, acc_finish2 takes it off
    return AR::acc_canon(AR::acc_finish2(acc, m), m) == want;
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
        for (u32 terms = 1; terms <= 128; terms++)
            for (int it = 0; it < 60; it++, count++) {
                const u32 rotations = it < 40 ? 8 : 1 + (u32)(rnd() % 32);
                if (!(pc.fp ? joined_sums<FpAr>(pc, terms, rotations, it % 4) : joined_sums<IntAr>(pc, terms, rotations, it % 4))) {
                    printf("joined sum q=%llu terms=%u rotations=%u kind %d\n", (unsigned long long)q, terms, rotations, it % 4); return 1; }
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
