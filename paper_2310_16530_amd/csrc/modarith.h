// Modular arithmetic for the key-switch kernels, in two interchangeable "arithmetic policies".
//
// IntAr  -- 64-bit integer residues, any prime below 2^61:
//   * Shoup multiplication by a constant w with companion w' = floor(w*2^64/q):
//       x*w - floor(x*w'/2^64)*q  lies in [0, 2q) for every 64-bit x.
//   * Harvey-style lazy butterflies keeping values in [0, 4q) (forward) or [0, 2q) (inverse).
//   * Montgomery reduction of a 128-bit accumulator: acc * 2^-64 mod q in [0, 2q) for acc < q*2^64.
//
// FpAr   -- residues held as integer-valued doubles (possibly negative), primes below 3*2^48.
//   On CDNA4 an FP64 FMA issues at the rate of one 32-bit integer multiply (four cycles per wave), and a Shoup
//   product of 64-bit words needs ten of those, so for the ~50-bit ciphertext primes the butterflies run on the
//   FP64 pipe.  Everything is
//   exact: for integers a, w with |a| <= A*q (A <= 8), 0 <= w < q < 3*2^48,
//       h = fl(a*w), l = fma(a, w, -h)          (a*w = h + l exactly)
//       c = rint(fl(h * fl(1/q)))               (|c - a*w/q| <= 0.5 + 3A/8)
//       r = fma(-c, q, h) + l                   (both steps exact: integers below 2^53)
//   gives r = a*w (mod q) with |r| <= (0.5 + 3A/8) q.  Four forward stages started from |x| <= q
//   stay below 7q, four inverse stages started from |x| <= q/2 stay at or below 8q < 2^53; a
//   3-instruction reduction x - rint(x/q)*q brings values back to |x| <= q/2 between rounds of four stages.
//   Narrow primes, q <= 17*2^45: the quotient is off by 0.5 + 3A q/2^53 <= 0.5 + 0.2A, so a stage takes A to at most 1.2A + 0.5: eight
//   forward stages from |x| <= 0.51q end below 10.5q (1.12, 1.84, 2.71, 3.75, 5.0, 6.5, 8.3, 10.5), from canonical words below 12.6q,
//   and 2^53 is 15q.  What leaves such a pass unreduced makes products with residues of at most 2.6q.
//
// All functions are __host__ __device__ so that the same source is unit-tested on the CPU.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef uint64_t u64;
typedef uint32_t u32;
typedef unsigned __int128 u128_t;

#define HD __host__ __device__ __forceinline__

// primes strictly below this bound use FpAr
#define CKKS_FP_PRIME_LIMIT (3ull << 48)
// FpAr primes up to this bound (49 bits and a little) are narrow: a forward pass of eight stages reduces nothing on its way, see FpAr
#define CKKS_FP_NARROW_MAX (17ull << 45)

struct u128w {
    u64 lo, hi;
};

HD u64 mulhi64(u64 a, u64 b) { return (u64)(((u128_t)a * b) >> 64); }
HD u64 csub(u64 x, u64 q) { return x >= q ? x - q : x; }

HD u64 mul_shoup_lazy(u64 x, u64 w, u64 wp, u64 q) {
    u64 h = mulhi64(x, wp);
    return x * w - h * q;
}
// csub(x, c) for x < 2c < 2^63 with n = -c modulo 2^64: the sign of x - c makes the mask, so that no comparison leaves its result in a mask
// register.  The asm keeps the compiler from seeing a comparison in it again.  In the inverse butterflies 30 transforms of 2^15 words take
// 28.8 instead of 29.3 us; in the forward ones it gained nothing and cost 2 % in the passes at N = 2^15, so they keep the comparison.
HD u64 csub_sign(u64 x, u64 c, u64 n) {
    u64 t = x + n;
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+v"(t));
#endif
    return t + ((u64)((int64_t)t >> 63) & c);
}
// mul_shoup_lazy with nq = -q modulo 2^64: both products add up in multiply-adds, where a difference of two words takes a borrow through a
// mask register (on the device two idle wait states before it may be read).  Inverse strided pass at N = 2^16: 2297 vector instructions
// and 296 idle slots -> 2186 and 231; the integer inner product of a mult on 8 ciphertexts 124.6 -> 118.5 us.
HD u64 mul_shoup_neg(u64 x, u64 w, u64 wp, u64 nq) {
    u64 h = mulhi64(x, wp);
    return x * w + h * nq;
}
HD u64 mul_shoup(u64 x, u64 w, u64 wp, u64 q) { return csub(mul_shoup_lazy(x, w, wp, q), q); }
HD u64 addmod(u64 a, u64 b, u64 q) { return csub(a + b, q); }
HD u64 submod(u64 a, u64 b, u64 q) { return a >= b ? a - b : a + q - b; }

HD void mac128(u128w& acc, u64 a, u64 b) {
    u128_t p = (u128_t)a * b + (((u128_t)acc.hi << 64) | acc.lo);
    acc.lo = (u64)p;
    acc.hi = (u64)(p >> 64);
}

// acc * 2^-64 mod q in [0, 2q), for acc < q*2^64.  qneg = -q^-1 mod 2^64.
HD u64 redc_lazy(u128w acc, u64 q, u64 qneg) {
    u64 m = acc.lo * qneg;
    u64 t = mulhi64(m, q);
    return acc.hi + t + (acc.lo != 0 ? 1 : 0);
}
HD u64 redc(u128w acc, u64 q, u64 qneg) { return csub(redc_lazy(acc, q, qneg), q); }

// canonical residue of a 128-bit sum of products (acc < q*2^64): REDC, then REDC against 2^128 mod q
HD u64 reduce128(u128w acc, u64 q, u64 qneg, u64 r2) {
    u64 t = redc_lazy(acc, q, qneg);
    u128w p2 = {0, 0};
    mac128(p2, t, r2);
    return redc(p2, q, qneg);
}
HD u64 mulmod_var(u64 a, u64 b, u64 q, u64 qneg, u64 r2) {
    u128w p = {0, 0};
    mac128(p, a, b);
    return reduce128(p, q, qneg, r2);
}

// Word formats of base-conversion sources (the coefficients times the conversion pre-factor that the last
// inverse stage leaves for the conversion kernels):
//   SRC_CANON  canonical integer            SRC_F64  canonical integer as a double (FpAr primes only)
//   SRC_DIGITS eight signed base-256 digits d_k in [-128, 127], y = sum d_k 256^k, digit k stored in byte k as
//              d_k + 128 with the top bit flipped, i.e. as the two's-complement byte the matrix cores read:
//              word = (y + B) ^ B with B = 0x80 in every byte (y <= CKKS_DIGIT_MAX).
enum SrcFormat { SRC_CANON = 0, SRC_F64 = 1, SRC_DIGITS = 2 };
#define CKKS_DIGIT_BIAS 0x8080808080808080ull
#define CKKS_DIGIT_MAX 0x7f7f7f7f7f7f7f7full  // the largest word eight such digits can hold
HD u64 digits_encode(u64 y) { return (y + CKKS_DIGIT_BIAS) ^ CKKS_DIGIT_BIAS; }

// ------------------------------------------------------------------ per-prime constants
struct PrimeConst {
    u64 q;        // the prime
    u64 qneg;     // -q^-1 mod 2^64
    u64 r2;       // 2^128 mod q
    u64 r1;       // 2^64 mod q
    u64 r1_p;     // its Shoup companion
    double qd;    // q as a double (exact for FpAr primes)
    double qinv;  // fl(1/q)
    u32 fp;       // 1 if the prime uses FpAr
    u32 narrow;   // 1 if it is at most CKKS_FP_NARROW_MAX
};

// scaling constants of the last inverse-NTT stage: sx multiplies the sums, sy the differences
// (sy already includes the stage's twiddle); Shoup companions for IntAr, doubles for FpAr.
struct InvScale {
    u64 sx, sx_p, sy, sy_p;
    double sxd, syd;
};

// ------------------------------------------------------------------------------ IntAr
struct IntAr {
    typedef u64 T;
    static constexpr bool is_fp = false;

    struct Mod {
        u64 q, q2, qneg, r1, r1_p, nq;
    };
    struct Tw {
        u64 w, wp;
    };
    // nq = -q as (-q^-1) q q: written 0 - q, the compiler turns h * nq back into a subtraction of h * q
    static HD Mod mod(const PrimeConst& p) { return Mod{p.q, 2 * p.q, p.qneg, p.r1, p.r1_p, p.qneg * p.q * p.q}; }
    // tables: tw_int [prime][4][N] = fwd w, fwd w', inv w, inv w'
    static HD Tw tw(const u64* ti, const double*, u32 idx, u32 N, bool inverse) {
        const u64* b = ti + (inverse ? 2 * (size_t)N : 0);
        return Tw{b[idx], b[N + idx]};
    }
    static HD T from_canon(u64 v, const Mod&) { return v; }
    static HD T from_raw(u64 v) { return v; }
    static HD u64 to_raw(T v) { return v; }
    // product of two canonical residues, as a value the transforms accept
    static HD T mul_canon(u64 a, u64 b, const PrimeConst& p, const Mod&) { return mulmod_var(a, b, p.q, p.qneg, p.r2); }
    // forward: values in [0, 8q) (8q < 2^64 for primes below 2^61).  A stage adds less than 2q to its inputs
    // (the product is in [0, 2q) for any 64-bit Y), so inputs below 6q need no reduction; RED takes 4q off
    // inputs that may have reached 6q..8q first.  NttCore fixes per stage which of the two applies.
    template <bool RED>
    static HD void bfly_fwd(T& X, T& Y, const Tw& t, const Mod& m) {
        u64 x = X;
        if (RED) {
            const u64 q4 = m.q2 + m.q2;
            x = x >= q4 ? x - q4 : x;
        }
        u64 r = mul_shoup_neg(Y, t.w, t.wp, m.nq);
        X = x + r;
        Y = x - r + m.q2;
    }
    // inverse: values in [0, 2q)
    static HD void bfly_inv(T& X, T& Y, const Tw& t, const Mod& m) {
        u64 s = X + Y;
        u64 d = X - Y + m.q2;
        X = csub_sign(s, m.q2, 2 * m.nq);
        Y = mul_shoup_neg(d, t.w, t.wp, m.nq);
    }
    static HD T round_reduce(T v, const Mod&) { return v; }  // lazy ranges are invariants: nothing to do
    static HD bool narrow(const Mod&) { return true; }
    template <int W>
    static HD void mid_reduce(T (&)[W], const Mod&) {}
    static HD u64 canon_fwd(T v, const Mod& m) { return csub(csub(csub(v, m.q2 + m.q2), m.q2), m.q); }  // from [0, 8q)
    // last inverse stage with scaling, canonical results (fmt: SRC_CANON or SRC_DIGITS; SRC_F64 does not apply)
    static HD void bfly_inv_last(T& X, T& Y, const InvScale& s, const Mod& m, u32 fmt, u64& ox, u64& oy) {
        u64 a = X + Y, d = X - Y + m.q2;
        ox = csub(mul_shoup_neg(a, s.sx, s.sx_p, m.nq), m.q);
        oy = csub(mul_shoup_neg(d, s.sy, s.sy_p, m.nq), m.q);
        if (fmt == SRC_DIGITS) ox = digits_encode(ox), oy = digits_encode(oy);
    }
    // inner-product accumulation: acc holds sum of v*k*2^-64 in [0, 2q); v canonical or forward-lazy (any 64-bit word)
    static HD T acc_zero() { return 0; }
    static HD void acc_mac(T& acc, T v, u64 key, const Mod& m) {
        u128w p = {0, 0};
        mac128(p, v, key);  // v < 2^64, key < q: v*key < q*2^64
        u64 r = redc_lazy(p, m.q, m.qneg);
        u64 s = acc + r;
        acc = s >= m.q2 ? s - m.q2 : s;
    }
    static HD T acc_fold(T acc, const Mod&) { return acc; }  // already kept in [0, 2q)
    static HD T acc_finish(T acc, const Mod& m) {  // remove the 2^-64: result in [0, 2q), valid as inverse-lazy
        return mul_shoup_neg(acc, m.r1, m.r1_p, m.nq);
    }
    static HD u64 acc_canon(T fin, const Mod& m) { return csub(fin, m.q); }
    // unreduced sum of products of two canonical residues: at most 8 terms (8 q^2 < q * 2^64), then wide_reduce gives the
    // sum times 2^-64 in [0, 2q)
    typedef u128w Wide;
    static constexpr u32 wide_terms = 8;
    static HD Wide wide_zero() { return u128w{0, 0}; }
    static HD void wide_mac(Wide& w, u64 a, u64 b) { mac128(w, a, b); }
    static HD T wide_reduce(const Wide& w, const Mod& m) { return redc_lazy(w, m.q, m.qneg); }
    static HD T wide_join(T a, T b, const Mod& m) {  // sum of two such results, in [0, 2q)
        u64 s = a + b;
        return s >= m.q2 ? s - m.q2 : s;
    }
    // acc_mac of a wide_reduce result with a canonical residue: one more factor 2^-64 (acc_finish2 removes both)
    static HD void acc_mac_wide(T& acc, T v, u64 b, const Mod& m) { acc_mac(acc, v, b, m); }
    // finish of an accumulation whose operands came from wide_reduce: removes 2^-128
    static HD T acc_finish2(T acc, const Mod& m) {
        return mul_shoup_neg(mul_shoup_neg(acc, m.r1, m.r1_p, m.nq), m.r1, m.r1_p, m.nq);
    }
};

// ------------------------------------------------------------------------------- FpAr
// Conversions between residues and doubles through the bit pattern of 2^52 + x: for 0 <= x < 2^52 the
// double 2^52 + x has exponent 2^52 and x itself as its 52 mantissa bits (FpAr residues are below 2^50).
HD double u64_to_f64(u64 x) {  // exact for x < 2^52
    return __builtin_bit_cast(double, x | 0x4330000000000000ull) - 4503599627370496.0;
}
HD u64 f64_to_u64(double d) {  // exact for integer-valued 0 <= d < 2^52
    return __builtin_bit_cast(u64, d + 4503599627370496.0) & 0x000fffffffffffffull;
}

struct FpAr {
    typedef double T;
    static constexpr bool is_fp = true;
    struct Mod {
        double q, qinv;
        u32 narrow_;
    };
    struct Tw {
        double w;
    };
    static HD Mod mod(const PrimeConst& p) { return Mod{p.qd, p.qinv, p.narrow}; }
    // tables: tw_fp [prime][2][N] = fwd w, inv w (as doubles)
    static HD Tw tw(const u64*, const double* tf, u32 idx, u32 N, bool inverse) {
        return Tw{tf[(inverse ? (size_t)N : 0) + idx]};
    }
    static HD T mulmod_lazy(T a, T w, const Mod& m) {
        double h = a * w;
        double l = __builtin_fma(a, w, -h);
        double c = __builtin_rint(h * m.qinv);
        return __builtin_fma(-c, m.q, h) + l;
    }
    static HD T reduce(T x, const Mod& m) {  // |result| <= q/2 (+ rounding slack far below 1)
        double c = __builtin_rint(x * m.qinv);
        return __builtin_fma(-c, m.q, x);
    }
    // A word y < 2^61 given as ya + yl with ya = (y >> 30) * 2^30 (31 significant bits, an exact double) and
    // yl = y mod 2^30: an integer-valued double congruent to y modulo q with |result| <= (0.5 + 2^-4) q + 2^30.
    // q > 2N >= 2^13, so the quotient ya / q is below 2^48 and its estimate off by less than 2^-4 before rounding
    // (q >= 2^28: 2^-19); ya - c*q is an integer below 2^50 in magnitude, hence the fma and the sum are exact.  reduce()
    // of the result is again within q/2: the result over q is below 2^17 + 1.
    static HD T reduce_split(double ya, double yl, const Mod& m) {
        double c = __builtin_rint(ya * m.qinv);
        return __builtin_fma(-c, m.q, ya) + yl;
    }
    static HD T from_canon(u64 v, const Mod&) { return u64_to_f64(v); }
    static HD T from_raw(u64 v) { return __builtin_bit_cast(double, v); }
    static HD u64 to_raw(T v) { return __builtin_bit_cast(u64, v); }
    static HD T mul_canon(u64 a, u64 b, const PrimeConst&, const Mod& m) {
        return mulmod_lazy(u64_to_f64(a), u64_to_f64(b), m);  // |result| <= 0.875 q
    }
    template <bool RED>  // the reduction schedule of the integer arithmetic does not apply: ranges are restored per round of four stages, for
                         // narrow primes per pass
    static HD void bfly_fwd(T& X, T& Y, const Tw& t, const Mod& m) {
        double r = mulmod_lazy(Y, t.w, m);
        double x = X;
        X = x + r;
        Y = x - r;
    }
    static HD void bfly_inv(T& X, T& Y, const Tw& t, const Mod& m) {
        double s = X + Y, d = X - Y;
        X = s;
        Y = mulmod_lazy(d, t.w, m);
    }
    static HD T round_reduce(T v, const Mod& m) { return reduce(v, m); }
    static HD bool narrow(const Mod& m) { return m.narrow_ != 0; }
    // between the two halves of a forward pass, and where its results meet canonical factors: nothing for narrow primes.  Three of the
    // four reductions a word meets between a conversion and a key product, bound by issue (N = 2^16, 24 + 6 limbs, batch 8, just
    // above 2^49: conversion 116 -> 110 us, inner product 258 -> 248, ModDown conversion 74 -> 71; the whole HMult 707 -> 692, 17
    // hoisted rotations 1011 -> 998).  Wider primes pay a branch a half pass (18.75 * 2^45, the same shapes, before narrow primes were told apart /
    // now: HMult 708.0 / 707.0, HRot 673.6 / 671.7, one HMult 144.9 / 143.8, 32 double-hoisted rotations of 35 + 7 limbs 1601 / 1597;
    // rescales show it: 8 of 24 limbs 151.0 / 151.5, 12 of 6 limbs 80.8 / 81.6)
    template <int W>
    static HD void mid_reduce(T (&x)[W], const Mod& m) {
        if (!narrow(m)) {
#pragma unroll
            for (int k = 0; k < W; k++) x[k] = reduce(x[k], m);
        }
    }
    static HD u64 canon(T v, const Mod& m) {
        double r = reduce(v, m);
        r = r < 0.0 ? r + m.q : r;
        return f64_to_u64(r);
    }
    static HD u64 canon_fwd(T v, const Mod& m) { return canon(v, m); }
    static HD double canon_f64(T v, const Mod& m) {
        double r = reduce(v, m);
        return r < 0.0 ? r + m.q : r;
    }
    // fmt: SRC_F64 stores the canonical value as a double's bit pattern, SRC_DIGITS as signed digits
    static HD void bfly_inv_last(T& X, T& Y, const InvScale& s, const Mod& m, u32 fmt, u64& ox, u64& oy) {
        double a = X + Y, d = X - Y;
        double rx = canon_f64(mulmod_lazy(a, s.sxd, m), m), ry = canon_f64(mulmod_lazy(d, s.syd, m), m);
        ox = fmt == SRC_F64 ? to_raw(rx) : f64_to_u64(rx);
        oy = fmt == SRC_F64 ? to_raw(ry) : f64_to_u64(ry);
        if (fmt == SRC_DIGITS) ox = digits_encode(ox), oy = digits_encode(oy);
    }
    static HD T acc_zero() { return 0.0; }
    static HD void acc_mac(T& acc, T v, u64 key, const Mod& m) { acc += mulmod_lazy(v, u64_to_f64(key), m); }
    static HD T acc_fold(T acc, const Mod& m) { return reduce(acc, m); }
    static HD T acc_finish(T acc, const Mod& m) { return reduce(acc, m); }
    static HD u64 acc_canon(T fin, const Mod& m) {
        double r = fin < 0.0 ? fin + m.q : fin;
        return f64_to_u64(r);
    }
    static HD T premul(u64 a, u64 b, const Mod& m) { return mulmod_lazy(u64_to_f64(a), u64_to_f64(b), m); }  // <= 0.875 q
    // Unreduced sum of products of two residues, exact, in 4 instructions a term instead of the 7 of a reduced product and
    // an addition.  t starts at 2^102 and stays in [2^102, 2^103) for at most 6 terms below (3*2^48)^2 < 2^99.2, so it is
    // always a multiple of 2^50: the step n - t is exact, l collects a*b - (n - t), at most 2^49 a term and so exact.
    // wide_reduce: H = t - 2^102 exact, c = rint(H / q) off by less than 1.2 before rounding (c < 2^52.2), H - c*q an
    // integer below 1.7 q, plus |l| < 2^51.6: below 2^53, exact; reduced to at most q/2.
    struct Wide {
        double t, l;
    };
    static constexpr u32 wide_terms = 6;
    static HD Wide wide_zero() { return Wide{5070602400912917605986812821504.0, 0.0}; }
    static HD void wide_mac(Wide& w, u64 a, u64 b) {
        const double x = u64_to_f64(a), y = u64_to_f64(b), n = __builtin_fma(x, y, w.t), d = n - w.t;
        w.l += __builtin_fma(x, y, -d);
        w.t = n;
    }
    static HD T wide_reduce(const Wide& w, const Mod& m) {
        const double h = w.t - 5070602400912917605986812821504.0, c = __builtin_rint(h * m.qinv);
        return reduce(__builtin_fma(-c, m.q, h) + w.l, m);
    }
    static HD T wide_join(T a, T b, const Mod&) { return a + b; }
    static HD void acc_mac_wide(T& acc, T v, u64 b, const Mod& m) { acc += mulmod_lazy(v, u64_to_f64(b), m); }
    static HD T acc_finish2(T acc, const Mod& m) { return reduce(acc, m); }
};

// A sum of more products than wide_terms, from its parts: `part` is a wide_reduce result, `last` the final one of the sum.  FpAr parts
// are at most q/2 each and any number of them may come (128 terms are 22): what the next part joins is folded, so the sum that
// leaves stays within q and its product with a residue within 0.875 q, eight of which on a folded q/2 are below 2^53.
template <class AR>
HD void join_part(typename AR::T& sum, typename AR::T part, bool last, const typename AR::Mod& m) {
    sum = AR::wide_join(sum, part, m);
    if (!last) sum = AR::acc_fold(sum, m);
}

// ------------------------------------------- recombination of a base conversion's digit sums (see conv_mfma_body)
// s[o + g] = S_g, the sum over sources and source digits of (digit g of the folded constant) * (source digit);
// |S_g| <= 17 * 2^17, V = sum_g 256^g S_g, |V| <= 2^14 m.
typedef int v16i __attribute__((ext_vector_type(16)));
// V of an FpAr target reduced to |.| <= (0.5 + 2^-15) m, exactly: pairs of digits are joined as 32-bit integers (below
// 2^30), lo = digits 0..3 (below 2^46), hi = digits 4..6 times 2^32 (an integer multiple of 2^32 with 38 significant
// bits: exact); the quotient estimate of (hi + lo) / m is off by less than 2^-15 before rounding, hi - c*m is an integer
// below 2^53 in magnitude, so the fma and the sum are exact.
HD double conv_recombine(const v16i& s, int o, const FpAr::Mod& m, const PrimeConst&) {
    const int p0 = s[o + 0] + s[o + 1] * 256, p1 = s[o + 2] + s[o + 3] * 256, p2 = s[o + 4] + s[o + 5] * 256;
    const double lo = __builtin_fma((double)p1, 65536.0, (double)p0);
    const double hi = __builtin_fma((double)s[o + 6], 281474976710656.0, (double)p2 * 4294967296.0);
    const double c = __builtin_rint((hi + lo) * m.qinv);
    return __builtin_fma(-c, m.q, hi) + lo;
}
// V of an IntAr target (m >= 3*2^48) as a word in (0.4 m, 1.6 m): V = lo + 2^32 t with |lo| < 2^46, t = digits 4..7 exact
// in a double (below 2^47); z = 1 - rint(t * 2^32 / m) appears as the low bits of one fma onto 1.5*2^52, |lo| / m < 0.09
// is what the estimate leaves out, and V + z*m is formed modulo 2^64 with m = mh * 2^32 + (signed low half).  14
// instructions, where six 128-bit multiply-accumulates and a Montgomery reduction took 62.
HD u64 conv_recombine(const v16i& s, int o, const IntAr::Mod& m, const PrimeConst& pc) {
    const int p0 = s[o + 0] + s[o + 1] * 256, p1 = s[o + 2] + s[o + 3] * 256, p2 = s[o + 4] + s[o + 5] * 256, p3 = s[o + 6] + s[o + 7] * 256;
    const double t = __builtin_fma((double)p3, 65536.0, (double)p2);
    const int z = (int)(u32)__builtin_bit_cast(u64, __builtin_fma(t, pc.qinv * -4294967296.0, 6755399441055744.0 + 1.0));
    const int ml = (int)(u32)m.q;
    const u32 mh = (u32)(m.q >> 32) + (ml < 0 ? 1u : 0u);
    const u64 lo = (u64)((int64_t)p1 * 65536 + p0 + (int64_t)z * ml);
    return lo + ((u64)((u32)p2 + ((u32)p3 << 16) + (u32)z * mh) << 32);
}
