// Kernels of the key-switch path.  The paper (Section 2) names the NTT and the base conversion as
// the major, memory-bound kernels and fuses several jobs into each memory load; here every
// producer and consumer of a transform is fused into one of the two NTT passes:
//
//   inv_contig_kernel   load (copy | a1*a2 | sigma_g gather) -> first inverse pass (N <= 2^13: both)
//   inv_contig_rows_kernel  first inverse pass alone at N = 2^13 (few integer limbs)
//   inv_strided_kernel  second inverse pass -> scale by N^-1 (* base-conversion pre-factor)
//   conv_fwd_strided_kernel, conv_mfma_kernel, conv_int_kernel, conv_up_both_kernel
//                       base conversion from the digit / special limbs -> first forward pass of the targets
//   inv_conv_one_kernel, inv_whole_conv_one_kernel
//                       second, or both, inverse passes of a limb -> conversion from it -> first forward pass (small grids)
//   fwd_strided_kernel  load -> first forward pass
//   fwd_contig_kernel   second forward pass -> canonical store
//   fwd_whole_kernel    both forward passes, N <= 2^13
//   ks_inner_kernel     second forward pass of every extended digit -> key inner product accumulated over
//                       the digits in registers (+ P * tensor terms of HMult) -> special limbs: first inverse
//                       pass of ModDown; q-limbs, launched after the ModDown conversion: second forward pass
//                       of the converted special part -> (c' - .) * P^-1 (+ sigma_g(b)) -> result
//   ks_final_kernel     the same end of the ModDown from a stored c', for the calls whose inner product is
//                       not this kernel or is followed by a plaintext multiply-accumulate over rotations
//   dh_accum_kernel     double hoisting: plaintext products of all rotations accumulated in the extended basis (rows of 128
//                       words on integer chains and for few rotations, of 256 otherwise)
//   bsgs_mac_kernel     giant-step combinations of baby-step rotations kept in the extended basis (more than four giant steps;
//                       up to four are sums of dh_accum_kernel)
//   fwd_strided_cached_kernel, conv_one_cached_kernel, ks_final_cached_kernel
//                       the same with ordinary accesses to the words between two launches, where they fit the Infinity Cache
//   inv_strided_sum_kernel  second inverse pass of several instances, their words added as integers: one ModDown for a sum
//   modup_kernel / moddown_kernel / automorph kernels: the stand-alone coefficient-form entry points.
//
// Levels below L, rescale and the ModDown merged with a rescale reuse these kernels on per-level tables.
//
// Every limb has its arithmetic: FpAr for primes below 3*2^48, IntAr otherwise.
#pragma once
#include "ntt.h"

struct PinvConst {
    u64 w, wp;
    double d;
};

struct Tables {
    const u64* tw_int;         // [D][4][N]  fwd w, fwd w', inv w, inv w'
    const double* tw_fp;       // [D][2][N]  fwd w, inv w (FpAr primes only)
    const PrimeConst* pc;      // [D]
    const InvScale* sc_plain;  // [D]  N^-1
    const InvScale* sc_up;     // [L]  N^-1 * [(Q_j/q_i)^-1]_{q_i}
    const InvScale* sc_dn;     // [K]  N^-1 * [(P/p_k)^-1]_{p_k}
    const u64* up_hatinv;      // [L][2]  [(Q_j/q_i)^-1]_{q_i} and Shoup companion (stand-alone ModUp)
    const u64* dn_hatinv;      // [K][2]
    const u64* up_chat;        // [L][D]  (Q_j/q_i) * 2^64 mod m_t   (0 inside the digit; stand-alone ModUp)
    const u64* dn_chat;        // [K][L]  (P/p_k) * 2^64 mod q_i   (stand-alone ModDown)
    const PinvConst* pinv;     // [L]     P^-1 mod q_i
    const u64* pmod;           // [L]     P mod q_i
    u32 logN, L, K, dnum, alpha, D;
    u32 Lfull;  // q-limbs of the whole prime chain
    u32 Kfull;  // special limbs of the whole prime chain
    u32 Lq;     // limbs 0 .. Lq-1 of this basis are q-limbs of the chain, the rest its special limbs
    // A Tables value describes one level: the basis q_0..q_{L-1}, p_0..p_{K-1} with L <= Lfull active
    // q-limbs, dnum = ceil(L/alpha) digits (the last one possibly partial) and limb indices 0..D-1 over
    // that basis.  The per-prime tables (tw_int, tw_fp, pc, sc_plain) and switching keys are laid out
    // over the whole chain of Lfull + K primes: phys() maps a limb index of the level to them.  All
    // other tables are per level and indexed by the level's limb indices.
    // Three kinds of Tables exist: a level (L active q-limbs, K special limbs, Lq = L); a rescale step
    // (L targets, K = 1 source = q-limb L, Lq = L + 1); a ModDown merged with the rescale after it (L
    // targets, K sources = q-limb L followed by the special limbs, Lq = L + 1).
    __host__ __device__ __forceinline__ u32 phys(u32 i) const { return i < Lq ? i : i + (Lfull - Lq); }
};

// slot j of sigma_g(f) in evaluation form reads slot eval_perm(j) of f
__device__ __forceinline__ u32 eval_perm(u32 j, u32 g, u32 logN) {
    const u32 two_n_mask = (2u << logN) - 1;
    u32 e = (g * (2 * (__brev(j) >> (32 - logN)) + 1)) & two_n_mask;
    return __brev((e - 1) >> 1) >> (32 - logN);
}

// Limb addressing of the plain transform passes: instance `inst`, limb l of n_l:
//   word offset (inst*gs + first + l) * N, prime index prime_base + l.
struct LimbSel {
    u32 n_l, n_inst, gs, first, prime_base;
};
__device__ __forceinline__ size_t limb_offset(const LimbSel& s, u32 inst, u32 l) { return (size_t)inst * s.gs + s.first + l; }

// Layout CP of the 16 words of a lane in a 256-word row (lane e0 of the row's 16): register kk holds word
// (kk/2)*32 + e0*2 + kk%2, i.e. eight adjacent pairs: every global access of the inner product that does not feed a
// transform directly (keys, own-digit operands, results) is a 16-byte access per lane, half the memory
// instructions of the one-word-per-access layout CA.  The per-instruction cost of the address path, not the
// bytes, is what the kernel's memory side was bound by.
typedef u64 u64x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32 cp_word(u32 e0, int kk) { return (u32)(kk >> 1) * 32 + e0 * 2 + (u32)(kk & 1); }
template <bool NT>
__device__ __forceinline__ void load_row_cp(const u64* row, u32 e0, u64 (&o)[16]) {
#pragma unroll
    for (int k2 = 0; k2 < 8; k2++) {
        const u64x2* p = reinterpret_cast<const u64x2*>(row + k2 * 32 + e0 * 2);
        const u64x2 t = NT ? __builtin_nontemporal_load(p) : *p;
        o[2 * k2] = t.x, o[2 * k2 + 1] = t.y;
    }
}
template <bool NT = true>
__device__ __forceinline__ void store_row_cp(u64* row, u32 e0, const u64 (&v)[16]) {
#pragma unroll
    for (int k2 = 0; k2 < 8; k2++) {
        u64x2 t;
        t.x = v[2 * k2], t.y = v[2 * k2 + 1];
        u64x2* p = reinterpret_cast<u64x2*>(row + k2 * 32 + e0 * 2);
        if (NT) __builtin_nontemporal_store(t, p);
        else *p = t;
    }
}
// between the contiguous-pass layout CB (word e0*16 + k) and CP, through the row's LDS slice
template <class AR>
__device__ __forceinline__ void exchange_cb_to_cp(typename AR::T (&x)[16], u64* l, u32 e0) {
    row_sync();
#pragma unroll
    for (int k = 0; k < 16; k++) l[pad16(e0 * 16 + k)] = AR::to_raw(x[k]);
    row_sync();
#pragma unroll
    for (int kk = 0; kk < 16; kk++) x[kk] = AR::from_raw(l[pad16(cp_word(e0, kk))]);
}
template <class AR>
__device__ __forceinline__ void exchange_cp_to_cb(typename AR::T (&x)[16], u64* l, u32 e0) {
    row_sync();
#pragma unroll
    for (int kk = 0; kk < 16; kk++) l[pad16(cp_word(e0, kk))] = AR::to_raw(x[kk]);
    row_sync();
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = AR::from_raw(l[pad16(e0 * 16 + k)]);
}
// Row `row_off/256` of sigma_g(f) in layout CP.  In evaluation order the automorphism maps a 256-word row onto one
// source row (the row index is the bit-reversed low part of the exponent index, and multiplication by g keeps low
// parts among themselves), so the source row is loaded whole with 16-byte accesses, staged in the row's LDS
// slice and permuted there, instead of one scattered 8-byte global access per word.
__device__ __forceinline__ void gather_row_cp(const u64* limb, u32 row_off, u32 gal, u32 logN, u64* l, u32 e0, u64 (&o)[16]) {
    const u32 src_row = eval_perm(row_off, gal, logN) >> 8;
    load_row_cp<false>(limb + (size_t)src_row * 256, e0, o);
    row_sync();
#pragma unroll
    for (int kk = 0; kk < 16; kk++) l[pad16(cp_word(e0, kk))] = o[kk];
    row_sync();
#pragma unroll
    for (int kk = 0; kk < 16; kk++) o[kk] = l[pad16(eval_perm(row_off + cp_word(e0, kk), gal, logN) & 255)];
}

// Buffer access to memory from a uniform base: address = base + per-lane byte offset + scalar byte offset.  The strided
// passes step through rows 32 KiB (or 2 KiB) apart; with plain pointers every such access cost two 64-bit additions,
// six of the seventy vector instructions per output of the conversion kernels, here the step is scalar arithmetic.
typedef u32 u32x2 __attribute__((ext_vector_type(2)));
struct Buf {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ explicit Buf(const void* base) : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0xffffffffu, 0x00020000)) {}
    __device__ __forceinline__ u64 ld(u32 lane_bytes, u32 bytes) const {
        return __builtin_bit_cast(u64, __builtin_amdgcn_raw_buffer_load_b64(r, lane_bytes, bytes, 0));
    }
    __device__ __forceinline__ u64 ld_nt(u32 lane_bytes, u32 bytes) const {
        return __builtin_bit_cast(u64, __builtin_amdgcn_raw_buffer_load_b64(r, lane_bytes, bytes, 2));
    }
    __device__ __forceinline__ void st(u64 v, u32 lane_bytes, u32 bytes) const {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, lane_bytes, bytes, 0);
    }
    __device__ __forceinline__ void st_nt(u64 v, u32 lane_bytes, u32 bytes) const {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, lane_bytes, bytes, 2);
    }
};

// most rotations (each with its own key and Galois element) one launch can be given
#define CKKS_ROT_CHUNK 16
// ... and where it leaves one sum, or the special limbs of each alone
#define CKKS_DH_CHUNK 32

// ============================================================ inverse transform, first pass
enum InvLoad { INV_PLAIN = 0, INV_TENSOR = 1, INV_ROT = 2 };
struct InvContigArgs {
    const u64* src;   // PLAIN: canonical eval-form limbs addressed by sel; TENSOR: ct1; ROT: ct
    const u64* src2;  // TENSOR: ct2
    u64* dst;         // raw inverse-lazy words, addressed by dsel
    LimbSel sel, dsel;
    u32 galois[CKKS_ROT_CHUNK];  // ROT: [0], or one per instance when per_inst is set
    u32 per_inst;
    u32 scale, out_fmt;  // of the second pass, where the kernel runs it too (inv_one_kernel): InvScaleSel, SrcFormat
};
// N <= 2^13: a workgroup of N / 16 lanes holds the limb in its registers and the first inverse pass's kernel runs the
// second pass as well, fwd_whole_kernel both forward ones: the limb crosses LDS between the passes instead of HBM, one
// launch instead of two, half the traffic.  At N = 2^14 the one workgroup of a limb (1024 lanes) takes longer than two
// launches that spread it over four: ten limbs 14.8 us against 11.5.
constexpr bool inv_one_kernel(int A) { return A <= 5; }
enum InvScaleSel { SC_PLAIN = 0, SC_UP = 1, SC_DN = 2 };

// row r of limb l of instance `inst`, in layout CB
template <class AR, int LOAD>
__device__ __forceinline__ void inv_load_row(typename AR::T (&x)[16], const InvContigArgs& a, const Tables& tb, const PrimeConst& pc,
                                             u64* lrow, u32 l, u32 r, u32 e0, u32 inst) {
    const u32 N = 1u << tb.logN;
    const typename AR::Mod m = AR::mod(pc);
    // operands arrive in layout CP (16-byte accesses) and are brought into the pass's layout CB by the exchange
    // that the pass needs anyway; a rotation applies its permutation in that exchange
    if (LOAD == INV_PLAIN) {
        u64 w[16];
        load_row_cp<true>(a.src + limb_offset(a.sel, inst, l) * N + (size_t)r * 256, e0, w);
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = AR::round_reduce(AR::from_canon(w[k], m), m);
        exchange_cp_to_cb<AR>(x, lrow, e0);
    } else if (LOAD == INV_TENSOR) {  // d2 = a1 * a2 on limb l of pair `inst`
        const size_t off = (((size_t)inst * 2 + 1) * tb.L + l) * N + (size_t)r * 256;
        u64 w1[16], w2[16];
        load_row_cp<true>(a.src + off, e0, w1);
        load_row_cp<true>(a.src2 + off, e0, w2);
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = AR::round_reduce(AR::mul_canon(w1[k], w2[k], pc, m), m);
        exchange_cp_to_cb<AR>(x, lrow, e0);
    } else {  // sigma_g(a) on limb l of ciphertext `inst`: the source row, whole, permuted on its way through LDS
        const u32 gal = a.galois[a.per_inst ? inst : 0];
        const u64* p = a.src + (((size_t)inst * 2 + 1) * tb.L + l) * N;
        const u32 src_row = eval_perm(r * 256, gal, tb.logN) >> 8;
        u64 w[16];
        load_row_cp<false>(p + (size_t)src_row * 256, e0, w);
        row_sync();
#pragma unroll
        for (int kk = 0; kk < 16; kk++) lrow[pad16(cp_word(e0, kk))] = w[kk];
        row_sync();
#pragma unroll
        for (int k = 0; k < 16; k++)
            x[k] = AR::round_reduce(AR::from_canon(lrow[pad16(eval_perm(r * 256 + e0 * 16 + k, gal, tb.logN) & 255)], m), m);
    }
}

template <class AR, int A, int LOAD>
__device__ __forceinline__ void inv_contig_body(const InvContigArgs& a, const Tables& tb, u64* lds, u32 l, u32 tile,
                                                u32 inst) {
    const u32 N = 1u << tb.logN, tid = threadIdx.x, e0 = tid % 16, ch = tid / 16, r = tile * 16 + ch;
    const u32 pi = tb.phys(a.sel.prime_base + l);
    const PrimeConst pc = tb.pc[pi];
    const typename AR::Mod m = AR::mod(pc);
    const u64* ti = tb.tw_int + (size_t)pi * 4 * N;
    const double* tf = tb.tw_fp + (size_t)pi * 2 * N;
    u64* lrow = lds + ch * 272;
    typename AR::T x[16];
    inv_load_row<AR, LOAD>(x, a, tb, pc, lrow, l, r, e0, inst);
    NttCore<AR, A>::template inv_contig<true>(x, lrow, e0, r, ti, tf, N, m);
    u64* o = a.dst + limb_offset(a.dsel, inst, l) * N + (size_t)r * 256;
#pragma unroll
    for (int k = 0; k < 16; k++) o[k * 16 + e0] = AR::to_raw(AR::round_reduce(x[k], m));
}

// Every transform kernel is compiled once per arithmetic and launched on a run of consecutive
// limbs [run.first, run.first + run.count) whose primes all use that arithmetic.  The plain passes exist for AR = AnyAr
// too, where a workgroup picks the arithmetic of its limb: a range that mixes both is then one launch, whose
// memory-bound FP64 workgroups and instruction-bound integer ones share the chip instead of taking turns.
struct LimbRun {
    u32 first, count;
};
struct AnyAr {};
#define CKKS_BY_ARITHMETIC(AR, prime, CALL)                                              \
    if constexpr (!__is_same(AR, AnyAr)) { typedef AR AR_; CALL; }                       \
    else if (tb.pc[tb.phys(prime)].fp) { typedef FpAr AR_; CALL; }                       \
    else { typedef IntAr AR_; CALL; }

// both passes of limb l of instance inst: put(k, word) for the lane's sixteen words, in layout SA of its tile, as they come (kept for a
// loop of stores after them, three limbs of 2^13 words take 9.1 instead of 8.9 us)
template <class AR, int A, int LOAD, class PUT>
__device__ __forceinline__ void inv_whole_words(const InvContigArgs& a, const Tables& tb, u64* lds, u32 l, u32 inst, PUT put) {
    typedef NttCore<AR, A> C;
    const u32 N = 1u << tb.logN, tid = threadIdx.x, e0 = tid % 16, r = tid / 16;
    const u32 vi = a.sel.prime_base + l, pi = tb.phys(vi);
    const PrimeConst pc = tb.pc[pi];
    const typename AR::Mod m = AR::mod(pc);
    const u64* ti = tb.tw_int + (size_t)pi * 4 * N;
    const double* tf = tb.tw_fp + (size_t)pi * 2 * N;
    u64* lrow = lds + r * 272;
    typename AR::T x[16];
    inv_load_row<AR, LOAD>(x, a, tb, pc, lrow, l, r, e0, inst);
    C::inv_contig(x, lrow, e0, r, ti, tf, N, m);
    row_sync();
#pragma unroll
    for (int k = 0; k < 16; k++) lrow[pad16(k * 16 + e0)] = AR::to_raw(AR::round_reduce(x[k], m));
    __syncthreads();
    const u32 g = tid >> 8, t = tid & 255, c = t % C::TC, r0 = t / C::TC, col = g * C::TC + c;
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = AR::from_raw(lds[(A > 4 ? r0 * 16 + k : k) * 272 + pad16(col)]);
    if (A > 4) __syncthreads();  // the pass exchanges through the same memory
    C::inv_strided_but_last(x, lds + g * 4096, t, ti, tf, N, m);
    const InvScale sc = a.scale == SC_PLAIN ? tb.sc_plain[pi] : a.scale == SC_UP ? tb.sc_up[vi] : tb.sc_dn[vi - tb.L];
#pragma unroll
    for (int k = 0; k < 8; k++) {
        u64 ox, oy;
        AR::bfly_inv_last(x[k], x[k + 8], sc, m, a.out_fmt, ox, oy);
        put(k, ox), put(k + 8, oy);
    }
}
template <class AR, int A, int LOAD>
__device__ __forceinline__ void inv_whole_body(const InvContigArgs& a, const Tables& tb, u64* lds, u32 l, u32 inst) {
    typedef NttCore<AR, A> C;
    const u32 t = threadIdx.x & 255, r0 = t / C::TC, col = (threadIdx.x >> 8) * C::TC + t % C::TC;
    u64* base = a.dst + (limb_offset(a.dsel, inst, l) << tb.logN) + (size_t)r0 * 256 + col;
    inv_whole_words<AR, A, LOAD>(a, tb, lds, l, inst, [=](int k, u64 w) __attribute__((always_inline)) { base[(size_t)k * C::RB * 256] = w; });
}
template <class AR, int A, int LOAD>
__global__ __launch_bounds__(inv_one_kernel(A) ? 16 << A : 256) void inv_contig_kernel(InvContigArgs a, Tables tb, LimbRun run) {
    constexpr bool ONE = inv_one_kernel(A);
    __shared__ u64 lds[ONE ? (1 << A) * 272 : NTT_LDS_WORDS];
    constexpr u32 TILES = ONE ? 1 : (1u << A) / 16;
    u32 group, inst;
    if (ONE ? !whole_decode(blockIdx.x, a.sel.n_inst, run.count, group, inst) : !xcd_decode(blockIdx.x, a.sel.n_inst, run.count * TILES, group, inst)) return;
    const u32 l = run.first + group / TILES;
    if constexpr (ONE) { CKKS_BY_ARITHMETIC(AR, a.sel.prime_base + l, (inv_whole_body<AR_, A, LOAD>(a, tb, lds, l, inst))) }
    else { CKKS_BY_ARITHMETIC(AR, a.sel.prime_base + l, (inv_contig_body<AR_, A, LOAD>(a, tb, lds, l, group % TILES, inst))) }
}

// the first pass alone where inv_contig_kernel would run both (spread_limbs on the host)
template <class AR, int A, int LOAD>
__global__ __launch_bounds__(256) void inv_contig_rows_kernel(InvContigArgs a, Tables tb, LimbRun run) {
    __shared__ u64 lds[NTT_LDS_WORDS];
    constexpr u32 TILES = (1u << A) / 16;
    u32 group, inst;
    if (!xcd_decode(blockIdx.x, a.sel.n_inst, run.count * TILES, group, inst)) return;
    inv_contig_body<AR, A, LOAD>(a, tb, lds, run.first + group / TILES, group % TILES, inst);
}

// =========================================================== inverse transform, second pass
struct InvStridedArgs {
    u64* data;  // in place: raw inverse-lazy words in, canonical coefficients (times the scale) out
    LimbSel sel;
    u32 scale;   // InvScaleSel
    u32 out_fmt;  // SrcFormat of the stored words: SRC_F64 applies to limbs of FpAr primes only (others stay canonical)
};

// the pass on a tile of limb vi at `base`: put(k, word) for the lane's sixteen words as they come
template <class AR, int A, class PUT>
__device__ __forceinline__ void inv_strided_words(const u64* base, const Tables& tb, u64* lds, u32 vi, u32 tile, u32 scale, u32 out_fmt, PUT put) {
    typedef typename AR::T T;
    typedef NttCore<AR, A> C;
    const u32 N = 1u << tb.logN, tid = threadIdx.x, pi = tb.phys(vi);
    const typename AR::Mod m = AR::mod(tb.pc[pi]);
    const u64* ti = tb.tw_int + (size_t)pi * 4 * N;
    const double* tf = tb.tw_fp + (size_t)pi * 2 * N;
    const InvScale sc = scale == SC_PLAIN ? tb.sc_plain[pi] : scale == SC_UP ? tb.sc_up[vi] : tb.sc_dn[vi - tb.L];
    const u32 c = tid % C::TC, r0 = tid / C::TC, col = tile * C::TC + c;
    T x[16];
    if constexpr (A > 4) {
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = AR::from_raw(base[(size_t)(r0 * 16 + k) * 256 + col]);
    } else {
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = AR::from_raw(base[(size_t)(k * C::RB + r0) * 256 + col]);
    }
    C::inv_strided_but_last(x, lds, tid, ti, tf, N, m);
#pragma unroll
    for (int k = 0; k < 8; k++) {
        u64 ox, oy;
        AR::bfly_inv_last(x[k], x[k + 8], sc, m, out_fmt, ox, oy);
        put(k, ox), put(k + 8, oy);
    }
}
template <class AR, int A>
__device__ __forceinline__ void inv_strided_body(const InvStridedArgs& a, const Tables& tb, u64* lds, u32 l, u32 tile,
                                                 u32 inst) {
    typedef NttCore<AR, A> C;
    u64* base = a.data + (limb_offset(a.sel, inst, l) << tb.logN);
    const u32 c = threadIdx.x % C::TC, r0 = threadIdx.x / C::TC, col = tile * C::TC + c;
    inv_strided_words<AR, A>(base, tb, lds, a.sel.prime_base + l, tile, a.scale, a.out_fmt,
                             [=](int k, u64 w) __attribute__((always_inline)) { base[(size_t)(k * C::RB + r0) * 256 + col] = w; });
}

#ifndef CKKS_INV_STRIDED_WAVES
#define CKKS_INV_STRIDED_WAVES 6
#endif
template <class AR, int A>
__global__ __launch_bounds__(256, (A == 8 && INV_STRIDED_HALF_EXCHANGE && !__is_same(AR, AnyAr)) ? CKKS_INV_STRIDED_WAVES : 4) void inv_strided_kernel(InvStridedArgs a, Tables tb, LimbRun run) {
    __shared__ u64 lds[(A == 8 && INV_STRIDED_HALF_EXCHANGE) ? 2048 : 4096];
    constexpr u32 TILES = (1u << A) / 16;
    u32 group, inst;
    if (!xcd_decode(blockIdx.x, a.sel.n_inst, run.count * TILES, group, inst)) return;
    const u32 l = run.first + group / TILES;
    CKKS_BY_ARITHMETIC(AR, a.sel.prime_base + l, (inv_strided_body<AR_, A>(a, tb, lds, l, group % TILES, inst)))
}

// The same pass on several instances of a limb at once: what is stored, as digits, is the sum of the instances' canonical words as
// an integer.  A conversion is linear over the integers, so the ModDowns of ciphertexts that are only ever added need one
// conversion of that sum.  A workgroup holds the same columns of four instances, 256 lanes each, and takes further ones in turn;
// the sums are joined in LDS.  The caller sees to it that n_sum primes fit the digit format (CKKS_DIGIT_MAX).
struct InvStridedSumArgs {
    u64* data;  // [n_sum][sel.n_inst][sel.gs][N]; the sums replace instance 0
    LimbSel sel;
    u32 scale, n_sum;
};
template <class AR, int A>
__global__ __launch_bounds__(1024) void inv_strided_sum_kernel(InvStridedSumArgs a, Tables tb, LimbRun run) {
    typedef NttCore<AR, A> C;
    __shared__ u64 all[4 * 4096];  // of each part: its exchange, then its sums
    constexpr u32 TILES = (1u << A) / 16;
    const u32 N = 1u << tb.logN, tid = threadIdx.x & 255, part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    u32 group, inst;
    if (!xcd_decode(blockIdx.x, a.sel.n_inst, run.count * TILES, group, inst)) return;
    const u32 l = run.first + group / TILES, vi = a.sel.prime_base + l, pi = tb.phys(vi);
    const typename AR::Mod m = AR::mod(tb.pc[pi]);
    const u64* ti = tb.tw_int + (size_t)pi * 4 * N;
    const double* tf = tb.tw_fp + (size_t)pi * 2 * N;
    const InvScale sc = a.scale == SC_PLAIN ? tb.sc_plain[pi] : a.scale == SC_UP ? tb.sc_up[vi] : tb.sc_dn[vi - tb.L];
    const u32 c = tid % C::TC, r0 = tid / C::TC, col = (group % TILES) * C::TC + c;
    const size_t step = (size_t)a.sel.n_inst * a.sel.gs * N;
    u64* limb = a.data + limb_offset(a.sel, inst, l) * N;
    u64* lds = all + part * 4096;
    u64 sum[16];
#pragma unroll
    for (int k = 0; k < 16; k++) sum[k] = 0;
    for (u32 g0 = 0; g0 < a.n_sum; g0 += 4) {  // the same barriers in every part: one that has no instance repeats the first
        const bool has = g0 + part < a.n_sum;
        const u64* base = limb + (has ? g0 + part : 0) * step;
        typename AR::T x[16];
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = AR::from_raw(base[(size_t)(A > 4 ? r0 * 16 + k : k * C::RB + r0) * 256 + col]);
        if (g0) __syncthreads();  // the previous exchange has been read
        C::inv_strided_but_last(x, lds, tid, ti, tf, N, m);
#pragma unroll
        for (int k = 0; k < 8; k++) {
            u64 ox, oy;
            AR::bfly_inv_last(x[k], x[k + 8], sc, m, SRC_CANON, ox, oy);
            if (has) sum[k] += ox, sum[k + 8] += oy;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; k++) lds[k * 256 + tid] = sum[k];
    __syncthreads();
#pragma unroll
    for (u32 k4 = 0; k4 < 4; k4++) {
        const u32 k = part * 4 + k4;
        u64 y = 0;
#pragma unroll
        for (u32 v = 0; v < 4; v++) y += all[v * 4096 + k * 256 + tid];
        limb[(size_t)(k * C::RB + r0) * 256 + col] = digits_encode(y);
    }
}

// ============================================================ forward transform, first pass
struct FwdStridedArgs {
    const u64* src;  // canonical coefficients addressed by sel
    u64* dst;        // raw forward-lazy words, same addressing (in place when dst == src)
    LimbSel sel;
};

// stages + store; x in layout SA.  CACHED: ordinary stores (stores_cached), in kernels of their own (see ks_final_cached_kernel)
template <class AR, int A, bool CACHED>
__device__ __forceinline__ void fwd_strided_finish(typename AR::T (&x)[16], const Tables& tb, u64* lds, u32 vi,
                                                   u64* dst, u32 tile) {
    typedef NttCore<AR, A> C;
    const u32 N = 1u << tb.logN, pi = tb.phys(vi);
    const u32 tid = threadIdx.x;
    const typename AR::Mod m = AR::mod(tb.pc[pi]);
    const u64* ti = tb.tw_int + (size_t)pi * 4 * N;
    const double* tf = tb.tw_fp + (size_t)pi * 2 * N;
    const u32 c = tid % C::TC, r0 = tid / C::TC, col = tile * C::TC + c;
    C::fwd_strided(x, lds, tid, ti, tf, N, m);
    if constexpr (A > 4) {
#pragma unroll
        for (int k = 0; k < 16; k++) {
            u64* const o = &dst[(size_t)(r0 * 16 + k) * 256 + col];
            if constexpr (CACHED) *o = AR::to_raw(AR::round_reduce(x[k], m));
            else __builtin_nontemporal_store(AR::to_raw(AR::round_reduce(x[k], m)), o);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 16; k++)
            dst[(size_t)(k * C::RB + r0) * 256 + col] = AR::to_raw(AR::round_reduce(x[k], m));
    }
}

template <class AR, int A, bool CACHED>
__device__ __forceinline__ void fwd_strided_body(const FwdStridedArgs& a, const Tables& tb, u64* lds, u32 l, u32 tile, u32 inst) {
    typedef NttCore<AR, A> C;
    const u32 N = 1u << tb.logN, tid = threadIdx.x, pi = a.sel.prime_base + l;
    const size_t off = limb_offset(a.sel, inst, l) * N;
    const typename AR::Mod m = AR::mod(tb.pc[tb.phys(pi)]);
    const u32 c = tid % C::TC, r0 = tid / C::TC, col = tile * C::TC + c;
    typename AR::T x[16];
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = AR::from_canon(a.src[off + (size_t)(k * C::RB + r0) * 256 + col], m);
    fwd_strided_finish<AR, A, CACHED>(x, tb, lds, pi, a.dst + off, tile);
}
template <class AR, int A, bool CACHED>
__device__ __forceinline__ void fwd_strided_workgroup(const FwdStridedArgs& a, const Tables& tb, const LimbRun run, u64* lds) {
    constexpr u32 TILES = (1u << A) / 16;
    u32 group, inst;
    if (!xcd_decode(blockIdx.x, a.sel.n_inst, run.count * TILES, group, inst)) return;
    const u32 l = run.first + group / TILES;
    CKKS_BY_ARITHMETIC(AR, a.sel.prime_base + l, (fwd_strided_body<AR_, A, CACHED>(a, tb, lds, l, group % TILES, inst)))
}
template <class AR, int A>
__global__ __launch_bounds__(256) void fwd_strided_kernel(FwdStridedArgs a, Tables tb, LimbRun run) {
    __shared__ u64 lds[4096];
    fwd_strided_workgroup<AR, A, false>(a, tb, run, lds);
}
template <class AR, int A>
__global__ __launch_bounds__(256) void fwd_strided_cached_kernel(FwdStridedArgs a, Tables tb, LimbRun run) {
    __shared__ u64 lds[4096];
    fwd_strided_workgroup<AR, A, true>(a, tb, run, lds);
}

// ============================== base conversion fused into the first forward pass of its targets
// CONV_UP: group = (b, digit j, tile); sources y [b][L][N] = coefficients times [(Q_j/q_i)^-1]; targets = the primes
//          outside digit j; dst dt [b][dnum][D][N].
// CONV_DN: group = (g, tile); sources y = special limbs [g][K][N]; targets = q-limbs; dst cv [g][L][N].
// Two or more sources convert on the matrix cores (conv_mfma_body), a single one is reduced directly (conv_one_body).
enum ConvDir { CONV_UP = 1, CONV_DN = 2 };
struct ConvArgs {
    const u64* src;       // CONV_UP [b][L][N], CONV_DN [g][K][N], in the format that conv_src_fmt names
    u64* dst;             // raw forward-lazy words after the first pass: CONV_UP dt [b][dnum][D][N], CONV_DN cv [g][L][N]
    u32 groups_outer;     // CONV_UP: batch; CONV_DN: number of g
    u32 blocks;           // workgroups per (group, tile): the run's targets in blocks
    // matrix cores: constant operands [digit][prime of the chain][KS][2 lane halves][8 digit rows][2 words], and the same
    // of a shorter last digit, [limb of the level]; digits from n_full on use the latter
    const u64* aop;
    const u64* aop_part;
    u32 n_full;
    u32 inverse;  // CONV_DN from a single source, one target per workgroup: src holds the words of the first inverse pass, the second is
                  // done here
};

// Twiddles of the strided pass of one target, W[0 .. R1) of its table, staged in LDS before the pass: a global load
// issued after the stores of an earlier target waits for those stores (one counter covers both), and with two or three
// targets per workgroup those waits were a quarter of the conversion kernels' time.  IntAr keeps w and its Shoup
// companion side by side (one 16-byte LDS read).
template <class AR, int A>
struct StridedTw {
    static constexpr u32 R1 = 1u << A, WORDS = AR::is_fp ? R1 : 2 * R1;
    static __device__ __forceinline__ void fill(u64* blk, u32 tid, const Tables& tb, u32 pi) {
        const u32 N = 1u << tb.logN;
        if (tid < R1) {
            if constexpr (AR::is_fp) {
                blk[tid] = __builtin_bit_cast(u64, tb.tw_fp[(size_t)pi * 2 * N + tid]);
            } else {
                blk[2 * tid] = tb.tw_int[(size_t)pi * 4 * N + tid];
                blk[2 * tid + 1] = tb.tw_int[(size_t)pi * 4 * N + N + tid];
            }
        }
    }
    static __device__ __forceinline__ typename AR::Tw get(const u64* blk, u32 idx) {
        if constexpr (AR::is_fp) return typename AR::Tw{__builtin_bit_cast(double, blk[idx])};
        else {
            const u64x2 t = *reinterpret_cast<const u64x2*>(blk + 2 * idx);
            return typename AR::Tw{t.x, t.y};
        }
    }
};
// stages 0-3 of the strided pass on the 16 words of layout SA; integer inputs below 2q leave below 6q
template <class AR, int A>
__device__ __forceinline__ void strided_stages_lo(typename AR::T (&x)[16], const u64* tw, const typename AR::Mod& m) {
#pragma unroll
    for (int s = 0; s < 4; s++) {
        const int d = 8 >> s;
#pragma unroll
        for (int k = 0; k < 16; k++) {
            if (k & d) continue;
            const typename AR::Tw w = StridedTw<AR, A>::get(tw, (1u << s) + (k >> (4 - s)));
            if (s == 3) AR::template bfly_fwd<true>(x[k], x[k + d], w, m);  // below 4q, 6q, 8q before stages 1, 2, 3
            else AR::template bfly_fwd<false>(x[k], x[k + d], w, m);
        }
    }
}
// stages 4 .. A-1 on layout SB (row r1*16 + k)
template <class AR, int A>
__device__ __forceinline__ void strided_stages_hi(typename AR::T (&x)[16], const u64* tw, u32 r1, const typename AR::Mod& m) {
#pragma unroll
    for (int s = 4; s < A; s++) {
        const int d = 1 << (A - s - 1);
#pragma unroll
        for (int k = 0; k < 16; k++) {
            if (k & d) continue;
            const typename AR::Tw w = StridedTw<AR, A>::get(tw, (1u << s) + ((r1 * 16 + k) >> (A - s)));
            if (s & 1) AR::template bfly_fwd<true>(x[k], x[k + d], w, m);  // below 6q after stage 3: odd stages reduce
            else AR::template bfly_fwd<false>(x[k], x[k + d], w, m);
        }
    }
}

// ---- a single source (digits of one limb, one special prime, the rescale): out_t = y mod m_t, the conversion constant is 1.
// A workgroup keeps the words of one load and reduces them to TB targets in turn: 4 FP64 targets share a load where the
// launch fills the chip (rescale of 8 ciphertexts at N = 2^16, 23 limbs: 63 -> 53 us against three targets converted before
// the first is transformed), 1 where it does not and the time is that of one workgroup; integer targets always 1 (launch_conv).
// CACHED: see fwd_strided_finish.
// One target of a source whose words y are in layout SA: reduced, first forward pass, stored to `limb`.  src_fp: the words of an FpAr
// source, doubles for FpAr targets, integers for IntAr ones.  tid: lane of the 256 that share the tile; again: lds still holds words.
template <class AR, int A, bool MANY, bool CACHED>
__device__ __forceinline__ void conv_one_target(u64 (&y)[16], bool src_fp, const PrimeConst& pc, const u64* tw, u64* lds, u64* limb, u32 tid, u32 tile, bool again) {
    typedef NttCore<AR, A> C;
    const typename AR::Mod m = AR::mod(pc);
    const u32 c = tid % C::TC, r0 = tid / C::TC, col = tile * C::TC + c;
    typename AR::T x[16];
    if constexpr (AR::is_fp) {
        if (src_fp) {
#pragma unroll
            for (int k = 0; k < 16; k++) x[k] = FpAr::reduce(FpAr::from_raw(y[k]), m);
        } else {
            // a 61-bit word is first brought below the target, which leaves it at most 0.6 q + 2^30
#pragma unroll
            for (int k = 0; k < 16; k++) {
                if (MANY) asm volatile("" : "+v"(y[k]));  // split here, not once for all targets (64 registers)
                x[k] = FpAr::reduce(FpAr::reduce_split((double)(u32)(y[k] >> 30) * 1073741824.0, (double)(u32)(y[k] & 0x3fffffffu), m), m);
            }
        }
    } else if (src_fp) {  // every FpAr prime is below every IntAr prime: the source is canonical already
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = y[k];
    } else {
#pragma unroll
        for (int k = 0; k < 16; k++) {
            u128w p = {0, 0};
            mac128(p, y[k], pc.r1);
            x[k] = redc(p, pc.q, pc.qneg);
        }
    }
    strided_stages_lo<AR, A>(x, tw, m);
    if constexpr (A > 4) {
        const Buf dst(limb);
        if (again) __syncthreads();  // the previous exchange has been read
        AR::mid_reduce(x, m);
#pragma unroll
        for (int k = 0; k < 16; k++) lds[k * 256 + tid] = AR::to_raw(x[k]);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 16; k++) x[k] = AR::from_raw(lds[(r0 * 16 + k) * C::TC + c]);
        strided_stages_hi<AR, A>(x, tw, r0, m);
#pragma unroll
        for (int k = 0; k < 16; k++) {
            if constexpr (CACHED) dst.st(AR::to_raw(AR::round_reduce(x[k], m)), 8 * (r0 * 16 * 256 + col), 8 * 256 * k);
            else dst.st_nt(AR::to_raw(AR::round_reduce(x[k], m)), 8 * (r0 * 16 * 256 + col), 8 * 256 * k);
        }
    } else {
        u64* dst = limb;
#pragma unroll
        for (int k = 0; k < 16; k++) dst[(size_t)(k * C::RB + r0) * 256 + col] = AR::to_raw(AR::round_reduce(x[k], m));
    }
}
template <class AR, int A, int DIR, int TB, bool CACHED = false>
__device__ __forceinline__ void conv_one_body(const ConvArgs& a, const Tables& tb, const LimbRun run) {
    typedef NttCore<AR, A> C;
    typedef StridedTw<AR, A> TW;
    constexpr u32 TILES = (1u << A) / 16;
    __shared__ u64 lds[A > 4 ? 4096 : 1];
    __shared__ __align__(16) u64 tws[TB * TW::WORDS];
    const u32 N = 1u << tb.logN, tid = threadIdx.x;
    u32 group, inst, own = 0xffffffffu, src_prime;
    const u64* src;
    u64* dst0;  // limb 0 of the destination group
    if (DIR == CONV_UP) {
        if (!xcd_decode(blockIdx.x, a.blocks, a.groups_outer * tb.dnum * TILES, group, inst)) return;
        const u32 bj = group / TILES, j = bj % tb.dnum, b = bj / tb.dnum;
        src = a.src + ((size_t)b * tb.L + j) * N;
        dst0 = a.dst + ((size_t)b * tb.dnum + j) * tb.D * N;
        own = src_prime = j;
    } else {
        if (!xcd_decode(blockIdx.x, a.blocks, a.groups_outer * TILES, group, inst)) return;
        const u32 g = group / TILES;
        src = a.src + (size_t)g * N;
        dst0 = a.dst + (size_t)g * tb.L * N;
        src_prime = tb.L;
    }
    const u32 tile = group % TILES, first = run.first + inst * TB, end = run.first + run.count;
    if (TB == 1 && first == own) return;
    const u32 c = tid % C::TC, r0 = tid / C::TC, col = tile * C::TC + c;
    const bool src_fp = tb.pc[tb.phys(src_prime)].fp;
    const Buf sb(src);
    u64 y[16];
    if (DIR == CONV_DN && TB == 1 && !CACHED && a.inverse) {  // CACHED: sources that are coefficients already
        auto keep = [&y](int k, u64 w) __attribute__((always_inline)) { y[k] = w; };
        if (src_fp) inv_strided_words<FpAr, A>(src, tb, lds, src_prime, tile, SC_DN, SRC_CANON, keep);
        else inv_strided_words<IntAr, A>(src, tb, lds, src_prime, tile, SC_DN, SRC_CANON, keep);
    } else {
#pragma unroll
        for (int k = 0; k < 16; k++) y[k] = sb.ld(8 * (r0 * 256 + col), 8 * 256 * C::RB * k);
    }
#pragma unroll
    for (int t = 0; t < TB; t++)
        if (first + t < end) TW::fill(tws + t * TW::WORDS, tid, tb, tb.phys(first + t));
    // a source of an FpAr prime, below 2^50: a double for FpAr targets (ModUp stores it so), an integer for IntAr ones
    if (src_fp && AR::is_fp == (DIR == CONV_DN)) {
#pragma unroll
        for (int k = 0; k < 16; k++) y[k] = AR::is_fp ? FpAr::to_raw(u64_to_f64(y[k])) : f64_to_u64(FpAr::from_raw(y[k]));
    }
    __syncthreads();
    bool again = false;
    for (int t = 0; t < TB; t++) {
        const u32 vi = first + t;
        if (vi >= end) break;
        if (vi == own) continue;
        conv_one_target<AR, A, (TB > 1), CACHED>(y, src_fp, tb.pc[tb.phys(vi)], tws + t * TW::WORDS, lds, dst0 + (size_t)vi * N, tid, tile, again);
        again = true;
    }
}

// ---- the same with the inverse transform of the source, repeated by the workgroup of every target (up_with_inverse and dn_with_inverse
// on the host): targets of either arithmetic in one launch.
// words of an FpAr source as conv_one_target takes them
__device__ __forceinline__ void conv_one_words(u64 (&y)[16], bool src_fp, bool dst_fp) {
    if (src_fp && dst_fp) {
#pragma unroll
        for (int k = 0; k < 16; k++) y[k] = FpAr::to_raw(u64_to_f64(y[k]));
    }
}
// ModUp, N >= 2^14: the second inverse pass; a.src holds the words of the first
template <int A>
__global__ __launch_bounds__(256) void inv_conv_one_kernel(ConvArgs a, Tables tb) {
    constexpr u32 TILES = (1u << A) / 16;
    __shared__ u64 lds[4096];
    __shared__ __align__(16) u64 tws[2u << A];
    u32 group, vi;
    if (!xcd_decode(blockIdx.x, tb.D, a.groups_outer * tb.dnum * TILES, group, vi)) return;
    const u32 of = group / TILES, tile = group % TILES, src = of % tb.dnum;
    if (vi == src) return;  // a digit's own limb
    const PrimeConst &ps = tb.pc[tb.phys(src)], &pt = tb.pc[tb.phys(vi)];
    const u64* limb = a.src + ((size_t)of << tb.logN);
    u64 y[16];
    auto keep = [&y](int k, u64 w) __attribute__((always_inline)) { y[k] = w; };
    if (ps.fp) inv_strided_words<FpAr, A>(limb, tb, lds, src, tile, SC_UP, SRC_CANON, keep);
    else inv_strided_words<IntAr, A>(limb, tb, lds, src, tile, SC_UP, SRC_CANON, keep);
    conv_one_words(y, ps.fp, pt.fp);
    CKKS_BY_ARITHMETIC(AnyAr, vi, (StridedTw<AR_, A>::fill(tws, threadIdx.x, tb, tb.phys(vi))))
    __syncthreads();
    u64* to = a.dst + (((size_t)of * tb.D + vi) << tb.logN);
    CKKS_BY_ARITHMETIC(AnyAr, vi, (conv_one_target<AR_, A, false, false>(y, ps.fp, pt, tws, lds, to, threadIdx.x, tile, false)))
}
// both inverse passes, N <= 2^13: of limb l of instance inst onto the level's limbs but itself (ModUp), or of the one
// limb after the targets (rescale)
template <int A, int LOAD, int DIR>
__global__ __launch_bounds__(16 << A) void inv_whole_conv_one_kernel(InvContigArgs a, u64* dst, Tables tb) {
    __shared__ u64 lds[(1 << A) * 272];
    __shared__ __align__(16) u64 tws[2u << A];
    u32 group, vi;
    const u32 targets = DIR == CONV_UP ? tb.D : tb.L;
    if (!xcd_decode(blockIdx.x, targets, a.sel.n_inst * a.sel.n_l, group, vi)) return;
    const u32 inst = group / a.sel.n_l, l = group % a.sel.n_l, src = a.sel.prime_base + l;
    if (vi == src) return;  // a digit's own limb
    const PrimeConst &ps = tb.pc[tb.phys(src)], &pt = tb.pc[tb.phys(vi)];
    u64 y[16];
    auto keep = [&y](int k, u64 w) __attribute__((always_inline)) { y[k] = w; };
    if (ps.fp) inv_whole_words<FpAr, A, LOAD>(a, tb, lds, l, inst, keep);
    else inv_whole_words<IntAr, A, LOAD>(a, tb, lds, l, inst, keep);
    conv_one_words(y, ps.fp, pt.fp);
    const u32 tid = threadIdx.x & 255, tile = threadIdx.x >> 8;
    CKKS_BY_ARITHMETIC(AnyAr, vi, (StridedTw<AR_, A>::fill(tws, threadIdx.x, tb, tb.phys(vi))))
    __syncthreads();
    u64* to = dst + (((size_t)group * targets + vi) << tb.logN);
    CKKS_BY_ARITHMETIC(AnyAr, vi, (conv_one_target<AR_, A, false, false>(y, ps.fp, pt, tws, lds + tile * 4096, to, tid, tile, false)))
}

// ---- several sources, on the matrix cores.
// out_t = sum_i y_i * chat_{i,t} mod m_t as an 8-bit integer matrix product.  Every source word arrives as eight
// signed base-256 digits (SRC_DIGITS), y_i = sum_b d_{i,b} 256^b; the digit weight is folded into the constant,
// C_{(i,b),t} = centred (chat_{i,t} * 256^b mod m_t), itself cut into signed digits C = sum_g c_g 256^g (seven for FpAr
// targets, eight for IntAr ones).  Then
//   S_{t,g}[n] = sum_{(i,b)} c_g(C_{(i,b),t}) * d_{i,b}(y_i[n])          (v_mfma_i32_32x32x32_i8, |S| <= 17 * 2^17)
//   out_t[n]  == V = sum_g 256^g S_{t,g}[n]  (mod m_t),  |V| <= 2^14 m_t
// recombined exactly (conv_recombine).  One 32x32x32 product handles 32 coefficients (columns) and 32 rows = four
// targets x 8 digits, over 32 values of (i,b) = four sources (lane half h holds the digit words of sources 4*ks + h and
// 4*ks + 2 + h in its 16 operand bytes, the constant operand the matching bytes); KS = ceil(ns/4) products accumulate
// all sources.  Row m of the constant operand sits in accumulator a = (m/8)*4 + m%4 of lane half (m/4)%2: a lane of half h
// gets the digits of target slot h in accumulators 0..7 and of slot 2 + h in accumulators 8..15.
//
// A lane keeps NTT x 16 converted words, x[u][k], k the coefficient's row block: rows k*RB + r0 of column c, the inputs of the
// first four forward stages, which therefore run in the lane that converted them; (r0, c) from a position pp = wave*32 + lane%32
// of the tile as tid maps to (r0, c) in layout SA.  A workgroup has 512 lanes (SETS = 1) and 2*NTT targets, u = target slot 2*u + h.
// What bounds it: the source words come from L2, and that traffic (7.3 TB/s with two targets at batch 8, N = 2^16, six sources;
// all loads from one cached row: 121 -> 78 us per launch) is the limit rather than the arithmetic, so four targets share a
// load where the registers allow it: FpAr targets need 128 (four waves per SIMD): 121 -> 111 us ModUp, 84 -> 71 us
// ModDown.  IntAr targets do not fit 128 with NTT = 2 (spills, 61 -> 66 us) and take NTT = 1: in workgroups of 256 lanes that kept
// twice the words each they needed 144 registers and, with their long butterflies, were the time of every small launch (one
// ciphertext at N = 2^16: conv_up_both_kernel 37 -> 25 us, at level 13 27 -> 22, one HMult 153 -> 140).
// Source i travels in word (i / 2) % 2 of lane half i % 2, so that six sources take three loads a lane half and not four (NW; both
// conversions of a batch of 8 108 -> 105 and 71 -> 68 us with the second batch of loads in flight, AHEAD).
typedef int v4i __attribute__((ext_vector_type(4)));
// SETS = 2: workgroups of 256 lanes that keep two positions each, pp = wave*64 + 32*set + lane%32, 32 words (IntAr targets of large
// launches).
template <class AR, int A, int KS, int DIR, int NTT, int NW, int AHEAD, int SETS = 1>
__device__ __forceinline__ void conv_mfma_body(const ConvArgs& a, const Tables& tb, const LimbRun run, u64* lds, u64* tws, const u32 tid,
                                               const u32 group, const u32 inst) {
    typedef NttCore<AR, A> C;
    typedef StridedTw<AR, A> TW;
    typedef typename AR::T T;
    static_assert(SETS == 1 || NTT == 1, "two targets or two positions a lane");
    static_assert(SETS == 1 || !AR::is_fp, "two positions a lane are for integers, whose sums go to the exchange unreduced");
    constexpr u32 TILES = (1u << A) / 16, TPW = 2 * NTT;  // targets per workgroup
    const u32 N = 1u << tb.logN, lane = tid & 63, wave = tid >> 6, n = lane & 31, h = lane >> 5;
    const u32 tile = group % TILES;
    u32 j = 0, ns, skip_lo = 0, skip_n = 0;
    const u64* src;
    u64* dst0;
    if (DIR == CONV_UP) {
        const u32 bj = group / TILES, b = bj / tb.dnum;
        j = bj % tb.dnum;
        // the last digit of a level may hold fewer than alpha limbs
        const u32 own_lo = j * tb.alpha, own_hi = (j + 1) * tb.alpha < tb.L ? (j + 1) * tb.alpha : tb.L;
        ns = own_hi - own_lo;
        src = a.src + ((size_t)b * tb.L + own_lo) * N;
        dst0 = a.dst + ((size_t)b * tb.dnum + j) * tb.D * N;
        // the digit's own limbs that lie in the run are no targets
        skip_lo = own_lo > run.first ? own_lo : run.first;
        const u32 hi = own_hi < run.first + run.count ? own_hi : run.first + run.count;
        skip_n = hi > skip_lo ? hi - skip_lo : 0;
    } else {
        const u32 g = group / TILES;
        ns = tb.K;
        src = a.src + (size_t)g * tb.K * N;
        dst0 = a.dst + (size_t)g * tb.L * N;
    }
    const u32 left = run.count - skip_n;
    if (inst * TPW >= left) return;  // digits with fewer targets leave their last blocks unused (uniform per workgroup)
    const u32 nt = left - inst * TPW < TPW ? left - inst * TPW : TPW;
    // limb of target slot sl (slots from nt on repeat the first: converted, never stored)
    auto limb_of = [&](u32 sl) {
        const u32 t = run.first + inst * TPW + (sl < nt ? sl : 0);
        return skip_n && t >= skip_lo ? t + skip_n : t;
    };
    bool narrow = true;  // of every target of the workgroup, so that the lane halves agree
    if constexpr (AR::is_fp) {
#pragma unroll
        for (u32 sl = 0; sl < TPW; sl++) narrow &= tb.pc[tb.phys(limb_of(sl))].narrow != 0;
    }
    v4i aop[KS];
    {
        const u32 sl = (NTT == 2 ? (n >> 4) * 2 : 0) + ((n >> 2) & 1), dg = ((n >> 3) & 1) * 4 + (n & 3), t = limb_of(sl);
        const u64* base = j < a.n_full ? a.aop + ((size_t)j * (tb.Lfull + tb.Kfull) + tb.phys(t)) * KS * 32 : a.aop_part + (size_t)t * KS * 32;
#pragma unroll
        for (int ks = 0; ks < KS; ks++) aop[ks] = *reinterpret_cast<const v4i*>(base + ks * 32 + h * 16 + dg * 2);
    }
#pragma unroll
    for (u32 tt = 0; tt < NTT * SETS; tt++) {
        const u32 sl = SETS == 2 ? tt : 2 * tt + (tid >> 8);  // 256 lanes fill one slot's twiddles
        if (sl < nt) TW::fill(tws + sl * TW::WORDS, tid & 255, tb, tb.phys(limb_of(sl)));
    }
    T x[NTT * SETS][16];
    {
        const PrimeConst pc0 = tb.pc[tb.phys(limb_of(h))], pc1 = tb.pc[tb.phys(limb_of(NTT == 2 ? 2 + h : h))];
        const typename AR::Mod m0 = AR::mod(pc0), m1 = AR::mod(pc1);
        // word q of this lane half: the digits of source 4*(q/2) + 2*(q%2) + h; beyond the last source any valid word will do (the
        // constant rows of those sources are zero)
        const Buf sb(src);
        u32 so[NW];
        const u32 pp0 = wave * (32 * SETS) + n;
#pragma unroll
        for (int q = 0; q < NW; q++) {
            const u32 i = 4 * (q >> 1) + 2 * (q & 1) + h;
            so[q] = 8 * ((i < ns ? i : ns - 1) * N + tile * C::TC + (pp0 / C::TC) * 256 + pp0 % C::TC);
        }
        // the second set is 32 positions on: 32 / TC rows down, or 32 columns on where a row holds more
        constexpr u32 SET = C::TC >= 64 ? 32 : (32 / C::TC) * 256;
        auto src_off = [&](int g) { return 8 * (u32)((g & 15) * C::RB * 256 + (g >> 4) * SET); };
        // one row block (32 coefficients a wave) at a time; the source words of the next AHEAD ones are requested before its products
        // are issued; scheduling barriers keep the compiler from hoisting every load of the unrolled loop (which would spill)
        u64 bw[AHEAD + 1][NW];
#pragma unroll
        for (int f = 0; f < AHEAD; f++)
#pragma unroll
            for (int q = 0; q < NW; q++) bw[f][q] = sb.ld(so[q], src_off(f));
#pragma unroll
        for (int g = 0; g < 16 * SETS; g++) {
            const int k = g & 15;
            if (g + AHEAD < 16 * SETS) {
#pragma unroll
                for (int q = 0; q < NW; q++) bw[(g + AHEAD) % (AHEAD + 1)][q] = sb.ld(so[q], src_off(g + AHEAD));
            }
            const u64* w = bw[g % (AHEAD + 1)];
            v16i acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < KS; ks++) {
                const u64 w0 = w[2 * ks], w1 = 2 * ks + 1 < NW ? w[2 * ks + 1 < NW ? 2 * ks + 1 : 0] : 0;
                const v4i bop = {(int)(u32)w0, (int)(u32)(w0 >> 32), (int)(u32)w1, (int)(u32)(w1 >> 32)};
                acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(aop[ks], bop, acc, 0, 0, 0);
            }
            // the empty statements keep a recombination here: sunk to a conditional use it would keep the sums alive
            x[g >> 4][k] = conv_recombine(acc, 0, m0, pc0);
            asm volatile("" : "+v"(x[g >> 4][k]));
            if constexpr (NTT == 2) {
                x[1][k] = conv_recombine(acc, 8, m1, pc1);
                asm volatile("" : "+v"(x[1][k]));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();  // the twiddles are in LDS
        // first four forward stages, in place (FP64: |x| <= 0.51 q on entry, below 7 q after, narrow primes 3.75 q)
        strided_stages_lo<AR, A>(x[0], tws + h * TW::WORDS, m0);
        if constexpr (NTT == 2)
            if (nt > 2) strided_stages_lo<AR, A>(x[1], tws + (2 + h) * TW::WORDS, m1);
        if constexpr (SETS == 2) strided_stages_lo<AR, A>(x[1], tws + h * TW::WORDS, m0);
    }
    if constexpr (SETS == 2) {  // one target after the other through half the memory
#pragma unroll
        for (u32 u = 0; u < 2; u++) {
            if constexpr (A > 4) {
                if (u >= nt) break;
                if (u) __syncthreads();  // the first exchange has been read
                const u32 t = limb_of(u), c = tid % C::TC, r1 = tid / C::TC;
                const typename AR::Mod m = AR::mod(tb.pc[tb.phys(t)]);
                if (h == u) {
#pragma unroll
                    for (u32 v = 0; v < 2; v++)
#pragma unroll
                        for (int k = 0; k < 16; k++) lds[k * 256 + wave * 64 + v * 32 + n] = AR::to_raw(x[v][k]);  // integers: no reduction
                }
                __syncthreads();
                T y[16];
#pragma unroll
                for (int k = 0; k < 16; k++) y[k] = AR::from_raw(lds[(r1 * 16 + k) * C::TC + c]);
                strided_stages_hi<AR, A>(y, tws + u * TW::WORDS, r1, m);
                u64* dst = dst0 + (size_t)t * N + (size_t)r1 * 16 * 256 + tile * C::TC + c;
#pragma unroll
                for (int k = 0; k < 16; k++) __builtin_nontemporal_store(AR::to_raw(AR::round_reduce(y[k], m)), &dst[k * 256]);
            } else if (h < nt) {
                const u32 t = limb_of(h), pp = wave * 64 + u * 32 + n;
                const typename AR::Mod m = AR::mod(tb.pc[tb.phys(t)]);
                u64* dst = dst0 + (size_t)t * N + (pp / C::TC) * 256 + tile * C::TC + pp % C::TC;
#pragma unroll
                for (int k = 0; k < 16; k++) dst[k * C::RB * 256] = AR::to_raw(AR::round_reduce(x[u][k], m));
            }
        }
        return;
    }
#pragma unroll
    for (u32 u = 0; u < NTT; u++) {  // slots 2u and 2u + 1
        if (2 * u >= nt) break;
        if constexpr (A > 4) {
            if (u) __syncthreads();  // the first exchange has been read
            if (AR::is_fp && !narrow) {
                const typename AR::Mod mx = AR::mod(tb.pc[tb.phys(limb_of(2 * u + h))]);
#pragma unroll
                for (int k = 0; k < 16; k++) x[u][k] = AR::round_reduce(x[u][k], mx);
            }
#pragma unroll
            for (int k = 0; k < 16; k++) lds[h * 4096 + k * 256 + wave * 32 + n] = AR::to_raw(x[u][k]);
            __syncthreads();
            const u32 half = tid >> 8, sl = 2 * u + half, st = tid & 255, c = st % C::TC, r1 = st / C::TC;
            if (sl < nt) {  // uniform per wave
                const u32 t = limb_of(sl);
                const typename AR::Mod m = AR::mod(tb.pc[tb.phys(t)]);
                T y[16];
#pragma unroll
                for (int k = 0; k < 16; k++) y[k] = AR::from_raw(lds[half * 4096 + (r1 * 16 + k) * C::TC + c]);
                strided_stages_hi<AR, A>(y, tws + sl * TW::WORDS, r1, m);
                u64* dst = dst0 + (size_t)t * N + (size_t)r1 * 16 * 256 + tile * C::TC + c;
#pragma unroll
                for (int k = 0; k < 16; k++) __builtin_nontemporal_store(AR::to_raw(AR::round_reduce(y[k], m)), &dst[k * 256]);
            }
        } else {
            const u32 sl = 2 * u + h, pp = wave * 32 + n;
            if (sl < nt) {
                const u32 t = limb_of(sl);
                const typename AR::Mod m = AR::mod(tb.pc[tb.phys(t)]);
                u64* dst = dst0 + (size_t)t * N + (pp / C::TC) * 256 + tile * C::TC + pp % C::TC;
#pragma unroll
                for (int k = 0; k < 16; k++) dst[k * C::RB * 256] = AR::to_raw(AR::round_reduce(x[u][k], m));
            }
        }
    }
}

// IntAr targets in workgroups of 256 lanes
template <int A, int KS, int DIR, int NW>
__device__ __forceinline__ void conv_int_workgroup(const ConvArgs& a, const Tables& tb, const LimbRun run) {
    constexpr u32 EXCH = A > 4 ? 4096 : 2, TW = 2 * StridedTw<IntAr, A>::WORDS;
    __shared__ __align__(16) u64 lds[EXCH + TW];
    u32 group, inst;
    if (!xcd_decode(blockIdx.x, a.blocks, a.groups_outer * (DIR == CONV_UP ? tb.dnum : 1) * ((1u << A) / 16), group, inst)) return;
    conv_mfma_body<IntAr, A, KS, DIR, 1, NW, KS <= 2 ? 2 : 1, 2>(a, tb, run, lds, lds + EXCH, threadIdx.x, group, inst);
}
template <int A, int KS, int DIR, int NW>
__global__ __launch_bounds__(256, 3) void conv_int_kernel(ConvArgs a, Tables tb, LimbRun run) { conv_int_workgroup<A, KS, DIR, NW>(a, tb, run); }

// row blocks whose source words are requested ahead: two where the registers allow it
constexpr int conv_ahead(int KS, int NW) { return KS <= 2 && NW <= 3 ? 2 : 1; }
// LDS words of conv_mfma_body: the exchange, and the twiddles of its targets
template <class AR, int A, int NTT>
struct ConvLds {
    static constexpr u32 exch = A > 4 ? 2 * 4096 : 2, tw = 2 * NTT * StridedTw<AR, A>::WORDS;
};
template <class AR, int A, int KS, int DIR, int NTT, int NW>
__device__ __forceinline__ void conv_mfma_workgroup(const ConvArgs& a, const Tables& tb, const LimbRun run) {
    __shared__ __align__(16) u64 lds[ConvLds<AR, A, NTT>::exch + ConvLds<AR, A, NTT>::tw];
    u32 group, inst;
    if (!xcd_decode(blockIdx.x, a.blocks, a.groups_outer * (DIR == CONV_UP ? tb.dnum : 1) * ((1u << A) / 16), group, inst)) return;
    conv_mfma_body<AR, A, KS, DIR, NTT, NW, conv_ahead(KS, NW)>(a, tb, run, lds, lds + ConvLds<AR, A, NTT>::exch, threadIdx.x, group, inst);
}

// targets per lane of the matrix-core form, for every number of sources from two on: with 9 to 16 sources it is 1.1 to 1.9
// times as fast as conversions on the vector units (HMult, N = 2^16, L = 30, K = 15, dnum 2, batch 4: 582 -> 469 us; L = 36,
// K = 12, dnum 3, batch 2: 396 -> 358; a rotation, L = 27, K = 9, dnum 3: 205 -> 168)
template <class AR>
constexpr int conv_mfma_ntt() { return AR::is_fp ? 2 : 1; }
// ONE: a single source, P targets per workgroup.  Else the matrix-core form, P = products per coefficient group + targets
// per lane.  NW: source words a lane half loads per coefficient where that is one fewer than the products take (six sources three words
// instead of four, two sources one instead of two), overloads so that the argument is in their names and only there.
template <class AR, int A, int DIR, int P, bool ONE>
__global__ __launch_bounds__(ONE ? 256 : 512, ONE ? (AR::is_fp ? 4 : 3) : !AR::is_fp ? 4 : P <= 4 ? 4 : 2)
void conv_fwd_strided_kernel(ConvArgs a, Tables tb, LimbRun run) {
    constexpr int NTT = conv_mfma_ntt<AR>();
    if constexpr (ONE) conv_one_body<AR, A, DIR, P>(a, tb, run);
    else conv_mfma_workgroup<AR, A, P - NTT, DIR, NTT, 2 * (P - NTT)>(a, tb, run);
}
template <class AR, int A, int DIR, int P, bool ONE, int NW>
__global__ __launch_bounds__(512, !AR::is_fp || P <= 4 ? 4 : 2) void conv_fwd_strided_kernel(ConvArgs a, Tables tb, LimbRun run) {
    static_assert(!ONE, "a single source is one word");
    constexpr int NTT = conv_mfma_ntt<AR>();
    conv_mfma_workgroup<AR, A, P - NTT, DIR, NTT, NW>(a, tb, run);
}
// ModDown from a single source with ordinary stores
template <class AR, int A, int P>
__global__ __launch_bounds__(256, AR::is_fp ? 4 : 3) void conv_one_cached_kernel(ConvArgs a, Tables tb, LimbRun run) {
    conv_one_body<AR, A, CONV_DN, P, true>(a, tb, run);
}
// ModDown onto FpAr targets, KS products per coefficient group, NTT targets per lane: a name of its own, so that profiles tell
// it from ModUp
template <int A, int KS, int DIR, int NTT>
__global__ __launch_bounds__(512, KS <= 2 ? 4 : 2) void conv_mfma_kernel(ConvArgs a, Tables tb, LimbRun run) {
    static_assert(DIR == CONV_DN, "the other conversions are conv_fwd_strided_kernel");
    conv_mfma_workgroup<FpAr, A, KS, DIR, NTT, 2 * KS>(a, tb, run);
}
template <int A, int KS, int DIR, int NTT, int NW>
__global__ __launch_bounds__(512, KS <= 2 ? 4 : 2) void conv_mfma_kernel(ConvArgs a, Tables tb, LimbRun run) {
    static_assert(DIR == CONV_DN, "the other conversions are conv_fwd_strided_kernel");
    conv_mfma_workgroup<FpAr, A, KS, DIR, NTT, NW>(a, tb, run);
}
// ModUp onto both classes of targets in one launch: the first workgroups convert to the IntAr run, the longer ones, the others to
// the FpAr run; bound by instructions and by source words from L2, they share the compute units (conv_up_both has the figures).
struct ConvBothArgs {
    ConvArgs fp, in;  // differ in `blocks`
    LimbRun run_fp, run_in;
    u32 grid_in;  // workgroups of the IntAr part, a multiple of 8
};
template <int A, int KS, int NW>
__device__ __forceinline__ void conv_up_both_workgroup(const ConvBothArgs& a, const Tables& tb) {
    constexpr u32 EXCH = ConvLds<FpAr, A, 2>::exch, TWF = ConvLds<FpAr, A, 2>::tw, TWI = ConvLds<IntAr, A, 1>::tw, TILES = (1u << A) / 16;
    __shared__ __align__(16) u64 lds[EXCH + (TWF > TWI ? TWF : TWI)];
    u32 group, inst;
    if (blockIdx.x >= a.grid_in) {
        if (!xcd_decode(blockIdx.x - a.grid_in, a.fp.blocks, a.fp.groups_outer * tb.dnum * TILES, group, inst)) return;
        conv_mfma_body<FpAr, A, KS, CONV_UP, 2, NW, 1>(a.fp, tb, a.run_fp, lds, lds + EXCH, threadIdx.x, group, inst);
    } else {
        if (!xcd_decode(blockIdx.x, a.in.blocks, a.in.groups_outer * tb.dnum * TILES, group, inst)) return;
        conv_mfma_body<IntAr, A, KS, CONV_UP, 1, NW, 1>(a.in, tb, a.run_in, lds, lds + EXCH, threadIdx.x, group, inst);
    }
}
template <int A, int KS>
__global__ __launch_bounds__(512, 4) void conv_up_both_kernel(ConvBothArgs a, Tables tb) { conv_up_both_workgroup<A, KS, 2 * KS>(a, tb); }
template <int A, int KS, int NW>
__global__ __launch_bounds__(512, 4) void conv_up_both_kernel(ConvBothArgs a, Tables tb) { conv_up_both_workgroup<A, KS, NW>(a, tb); }

// =========================================================== forward transform, second pass
struct FwdContigArgs {
    u64* data;  // in place: raw forward-lazy words in, canonical evaluation form out
    LimbSel sel;
    u32 own_alpha, own_L;  // own_alpha != 0: instances are digits, limb l < own_L has nothing to do in digit l / own_alpha
};

template <class AR, int A>
__device__ __forceinline__ void fwd_contig_body(const FwdContigArgs& a, const Tables& tb, u64* lds, u32 l, u32 tile,
                                                u32 inst) {
    typedef typename AR::T T;
    const u32 N = 1u << tb.logN, tid = threadIdx.x, e0 = tid % 16, ch = tid / 16, r = tile * 16 + ch;
    const u32 pi = tb.phys(a.sel.prime_base + l);
    const typename AR::Mod m = AR::mod(tb.pc[pi]);
    const u64* ti = tb.tw_int + (size_t)pi * 4 * N;
    const double* tf = tb.tw_fp + (size_t)pi * 2 * N;
    u64* lrow = lds + ch * 272;
    u64* p = a.data + limb_offset(a.sel, inst, l) * N + (size_t)r * 256;
    T x[16];
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = AR::from_raw(p[k * 16 + e0]);
    NttCore<AR, A>::template fwd_contig<!AR::is_fp>(x, lrow, e0, r, ti, tf, N, m);
    row_sync();
#pragma unroll
    for (int k = 0; k < 16; k++) lrow[pad16(e0 * 16 + k)] = AR::canon_fwd(x[k], m);
    row_sync();
    u64 res[16];  // stored in layout CP: 16 bytes per access; cacheable, the caller's next call reads it
#pragma unroll
    for (int kk = 0; kk < 16; kk++) res[kk] = lrow[pad16(cp_word(e0, kk))];
    store_row_cp<false>(p, e0, res);
}

// AnyAr: four waves per SIMD, as LDS allows; two registers above 128 made it three (transforms of mixed limbs, N = 2^14 .. 2^16: 31.3 -> 28.9 us,
// 41.9 -> 40.6, 55.4 -> 54.1; those of one round of workgroups within 0.5 %)
template <class AR, int A>
__global__ __launch_bounds__(256, __is_same(AR, AnyAr) ? 4 : 1) void fwd_contig_kernel(FwdContigArgs a, Tables tb, LimbRun run) {
    __shared__ u64 lds[NTT_LDS_WORDS];
    constexpr u32 TILES = (1u << A) / 16;
    u32 group, inst;
    if (!xcd_decode(blockIdx.x, a.sel.n_inst, run.count * TILES, group, inst)) return;
    const u32 l = run.first + group / TILES;
    if (a.own_alpha && l < a.own_L && l / a.own_alpha == inst) return;
    CKKS_BY_ARITHMETIC(AR, a.sel.prime_base + l, (fwd_contig_body<AR_, A>(a, tb, lds, l, group % TILES, inst)))
}

// ============================================== forward transform of a limb that one workgroup holds
template <class AR, int A>
__device__ __forceinline__ void fwd_whole_body(const FwdContigArgs& a, const Tables& tb, u64* lds, u32 l, u32 inst) {
    typedef NttCore<AR, A> C;
    const u32 N = 1u << tb.logN, tid = threadIdx.x, pi = tb.phys(a.sel.prime_base + l);
    const typename AR::Mod m = AR::mod(tb.pc[pi]);
    const u64* ti = tb.tw_int + (size_t)pi * 4 * N;
    const double* tf = tb.tw_fp + (size_t)pi * 2 * N;
    const u32 g = tid >> 8, t = tid & 255, c = t % C::TC, r0 = t / C::TC, col = g * C::TC + c;
    u64* limb = a.data + limb_offset(a.sel, inst, l) * N;
    typename AR::T x[16];
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = AR::from_canon(limb[(size_t)(k * C::RB + r0) * 256 + col], m);
    C::fwd_strided(x, lds + g * 4096, t, ti, tf, N, m);
    if (A > 4) __syncthreads();  // the pass's exchange has been read
#pragma unroll
    for (int k = 0; k < 16; k++) lds[(A > 4 ? r0 * 16 + k : k) * 272 + pad16(col)] = AR::to_raw(AR::round_reduce(x[k], m));
    __syncthreads();
    const u32 e0 = tid % 16, r = tid / 16;
    u64* lrow = lds + r * 272;
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = AR::from_raw(lrow[pad16(k * 16 + e0)]);
    row_sync();
    C::fwd_contig(x, lrow, e0, r, ti, tf, N, m);
    row_sync();
#pragma unroll
    for (int k = 0; k < 16; k++) lrow[pad16(e0 * 16 + k)] = AR::canon_fwd(x[k], m);
    row_sync();
    u64 res[16];
#pragma unroll
    for (int kk = 0; kk < 16; kk++) res[kk] = lrow[pad16(cp_word(e0, kk))];
    store_row_cp<false>(limb + (size_t)r * 256, e0, res);
}
template <int A>
__global__ __launch_bounds__(16 << A) void fwd_whole_kernel(FwdContigArgs a, Tables tb, LimbRun run) {
    __shared__ u64 lds[(1 << A) * 272];
    u32 group, inst;
    if (!whole_decode(blockIdx.x, a.sel.n_inst, run.count, group, inst)) return;
    const u32 l = run.first + group;
    CKKS_BY_ARITHMETIC(AnyAr, a.sel.prime_base + l, (fwd_whole_body<AR_, A>(a, tb, lds, l, inst)))
}

// ==================================================================== key inner product
// Work item = (limb i of D, tile, instance).  For every digit j the evaluation-form value of the
// extended digit on limb i is produced in registers -- the second forward pass of dt[.][j][i]
// (NTT_INSIDE), or a gather from the already transformed digits (hoisted rotations), or, on the
// digit's own limbs, the switched polynomial itself (copy | a1*a2 | sigma_g(a)) -- multiplied by
// the two key components and accumulated.  q-limbs: c' is stored canonical.  Special limbs: the
// first inverse pass of ModDown runs on the accumulators and raw words are stored.
// OWN_ROT_SUM: the rotations of n_sum ciphertexts, added: everything after the ModDowns' conversions is linear, so the sum over the
// digits runs over all instances' and ends in one ModDown (of the sum of the special parts, see inv_strided_sum_kernel).
enum OwnLoad { OWN_COPY = 0, OWN_TENSOR = 1, OWN_ROT = 2, OWN_ROT_SUM = 3 };
struct InnerArgs {
    const u64* dt;    // [inst or 1][dnum][D][N]: raw forward-lazy (NTT_INSIDE) or canonical eval (hoisted)
    const u64* own;   // COPY: d [inst][L][N]; TENSOR: ct1; ROT: ct ([inst][2][L][N]); hoisted: ct [2][L][N]
    const u64* own2;  // TENSOR: ct2
    const u64* key[CKKS_DH_CHUNK];  // one shared key (index 0) or one per instance (hoisted: at most CKKS_DH_CHUNK)
    u32 galois[CKKS_DH_CHUNK];      // ROT: [0]; hoisted: per instance
    u64* cq;                         // [inst][2][L][N] canonical
    u64* cp;                         // [inst][2][D - split][N] raw inverse-lazy after the first inverse pass
    u32 n_inst;
    u32 split;    // limbs below split are stored to cq ([inst][2][split][N]), the others continue to cp: the number
                  // of q-limbs, or one less when the ModDown that follows also divides by the last q-limb
    u32 per_inst;    // not hoisted: every instance has its own key and Galois element (at most CKKS_ROT_CHUNK instances)
    u32 n_sum;       // OWN_ROT_SUM: instances added (n_inst is 1)
    // FUSED (limbs below split only, launched after the ModDown conversion): the kernel also ends the ModDown
    const u64* cv;              // [inst][2][split][N] converted special part, first forward pass done
    u64* out;                   // [inst][2][split][N]
    const PinvConst* fin_pinv;  // [split] inverse of the product of the ModDown's source primes
    // 1: a workgroup owns 16 rows.  2, 4: it owns 8 or 4, and a team of two or four wavefronts works on four of them, each on every
    // second or fourth digit; the sums are joined in LDS and the first two wavefronts of a team end a component each.  For grids
    // that leave the chip idle, where the time is that of one wavefront and its dnum + 2 passes run one after the other
    // (inner_ways).
    u32 ways;
};

// Twiddles of one row's second forward pass, kept in LDS for kernels that run that pass several times on the same
// row of the same limb (the inner product: once per digit and twice more when it ends the ModDown).  FP64 limbs
// only: 255 doubles per row.  Words [0, 15): stages 0-3, whose 2^u twiddles are the same for the row's 16 lanes
// (stage u from offset 2^u - 1); then 15 words per lane: stages 4-7, 2^(u-4) twiddles each.  The lane blocks are
// 15 words apart, so the 16 lanes of a row read 16 different bank pairs.  Loaded from the tables once per
// workgroup: the 30 global loads per lane and pass were 14 % of the fused kernel's time.
#define CKKS_ROW_TW_WORDS 256
template <int A>
__device__ __forceinline__ void fill_row_tw(u64* blk, u32 e0, u32 r, const double* tf) {
    if (e0 < 15) {
        const u32 u = 31 - __clz(e0 + 1), off = e0 + 1 - (1u << u);
        blk[e0] = __builtin_bit_cast(u64, tf[(1u << (A + u)) + (r << u) + off]);
    }
#pragma unroll
    for (int u = 4; u < 8; u++) {
#pragma unroll
        for (int t = 0; t < (1 << (u - 4)); t++)
            blk[15 + e0 * 15 + (1 << (u - 4)) - 1 + t] = __builtin_bit_cast(u64, tf[(1u << (A + u)) + (r << u) + (e0 << (u - 4)) + t]);
    }
    row_sync();
}
struct RowTwLds {
    const u64* blk;
    u32 e0;
    __device__ __forceinline__ FpAr::Tw get(int u, u32 w) const {
        const u32 t = w >> (8 - u);
        const u32 at = u < 4 ? (1u << u) - 1 + t : 15 + e0 * 15 + (1u << (u - 4)) - 1 + (t - (e0 << (u - 4)));
        return FpAr::Tw{__builtin_bit_cast(double, blk[at])};
    }
};

template <class AR, int A, int OWN, bool HOISTED, bool FUSED>
__device__ __forceinline__ void ks_inner_body(const InnerArgs& a, const Tables& tb, u64* lds, u32 i, u32 tile,
                                              u32 inst) {
    typedef typename AR::T T;
    const u32 ways = HOISTED ? 1 : a.ways, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the `ways` (1, 2 or 4) wavefronts of a team share four rows; by shifts: chosen by comparisons they cost branches
    const u32 lg = ways >> 1, part = wave & (ways - 1);
    const u32 N = 1u << tb.logN, tid = threadIdx.x, e0 = tid % 16, ch = tid / 16, r0 = (tile * (4 >> lg) + (wave >> lg)) * 4, r = r0 + (ch & 3);
    const u32 L = tb.L, D = tb.D;
    const u32 pi = tb.phys(i), Dkey = tb.Lfull + tb.K;  // keys are laid out over the whole chain
    const PrimeConst pc = tb.pc[pi];
    const typename AR::Mod m = AR::mod(pc);
    const u64* ti = tb.tw_int + (size_t)pi * 4 * N;
    const double* tf = tb.tw_fp + (size_t)pi * 2 * N;
    u64* lrow = lds + ch * 272;
    const u32 row_off = r * 256;
    constexpr bool SUM = OWN == OWN_ROT_SUM;
    const u32 kidx = (HOISTED || a.per_inst) ? inst : 0;
    const u64* key = SUM ? nullptr : a.key[kidx] + (size_t)pi * N + row_off;
    u32 gal = SUM ? 0 : a.galois[kidx];
    const u32 own_digit = i < L ? i / tb.alpha : 0xffffffffu;
    constexpr bool TWL = AR::is_fp && !HOISTED;  // the row's forward twiddles live in LDS
    u64* twblk = lds + NTT_LDS_WORDS + ch * CKKS_ROW_TW_WORDS;
    if constexpr (TWL) fill_row_tw<A>(twblk, e0, r, tf);
    T acc0[16], acc1[16];  // layout CP
#pragma unroll
    for (int k = 0; k < 16; k++) acc0[k] = AR::acc_zero(), acc1[k] = AR::acc_zero();
    // FpAr sums at most 8 lazily reduced products (0.69 q each) between reductions; narrow primes five of digits that were not reduced
    // (2.6 q each: 13.5 q with what is left of the sum before)
    u32 since = 0;
    const u32 fold_at = AR::is_fp && AR::narrow(m) ? 5 : 8;
    for (u32 jj = part; jj < (SUM ? a.n_sum : 1) * tb.dnum; jj += ways) {
        u32 j = jj, src = inst;
        if constexpr (SUM) {  // digits in rotated order: the cheap own digits spread over the wavefronts that share the row
            src = jj / tb.dnum, j = (jj + src) % tb.dnum;
            key = a.key[src] + (size_t)pi * N + row_off, gal = a.galois[src];
        }
        const u64* k0 = key + ((size_t)j * 2 + 0) * Dkey * N;
        const u64* k1 = key + ((size_t)j * 2 + 1) * Dkey * N;
        u64 kv0[16], kv1[16];
        // FpAr issues key loads before the transform so that they are in flight meanwhile: both components
        // where the registers allow it (measured per variant), else the first one only; IntAr has no
        // registers to spare and loads the key at its use
        constexpr bool EARLY0 = AR::is_fp, EARLY1 = AR::is_fp && OWN == OWN_TENSOR;
        if constexpr (EARLY0) load_row_cp<false>(k0, e0, kv0);
        if constexpr (EARLY1) load_row_cp<false>(k1, e0, kv1);
        T v[16];  // the digit on this limb, evaluation form, layout CP
        if (j == own_digit) {
            if (HOISTED) {
                u64 w[16];
                gather_row_cp(a.own + ((size_t)L + i) * N, row_off, gal, tb.logN, lrow, e0, w);
#pragma unroll
                for (int k = 0; k < 16; k++) v[k] = AR::round_reduce(AR::from_canon(w[k], m), m);
            } else if (OWN == OWN_COPY) {
                u64 w[16];
                load_row_cp<false>(a.own + ((size_t)inst * L + i) * N + row_off, e0, w);
#pragma unroll
                for (int k = 0; k < 16; k++) v[k] = AR::round_reduce(AR::from_canon(w[k], m), m);
            } else if (OWN == OWN_TENSOR) {
                // the tensor terms d0 = b1*b2 and d1 = a1*b2 + a2*b1 join c' here as P * d, where a1 and a2 are
                // loaded anyway: (c' + P*d - conv) * P^-1 = (c' - conv) * P^-1 + d, so the kernel that ends the
                // ModDown adds nothing, also when it divides by the last q-limb as well.  One more product
                // between folds: at most 9 * 0.69 q < 2^53, still exact.
                const size_t off = (((size_t)inst * 2 + 1) * L + i) * N + row_off, offb = off - (size_t)L * N;
                const u64 pmod = tb.pmod[i];
#pragma unroll
                for (int k2 = 0; k2 < 8; k2++) {
                    const u32 w = k2 * 32 + e0 * 2;
                    const u64x2 a1 = __builtin_nontemporal_load(reinterpret_cast<const u64x2*>(a.own + off + w));
                    const u64x2 a2 = __builtin_nontemporal_load(reinterpret_cast<const u64x2*>(a.own2 + off + w));
                    const u64x2 b1 = __builtin_nontemporal_load(reinterpret_cast<const u64x2*>(a.own + offb + w));
                    const u64x2 b2 = __builtin_nontemporal_load(reinterpret_cast<const u64x2*>(a.own2 + offb + w));
#pragma unroll
                    for (int b = 0; b < 2; b++) {
                        const int k = 2 * k2 + b;
                        v[k] = AR::round_reduce(AR::mul_canon(a1[b], a2[b], pc, m), m);
                        AR::acc_mac(acc0[k], AR::mul_canon(b1[b], b2[b], pc, m), pmod, m);
                        AR::acc_mac(acc1[k], AR::mul_canon(a1[b], b2[b], pc, m) + AR::mul_canon(a2[b], b1[b], pc, m), pmod, m);
                    }
                }
            } else {
                u64 w[16];
                gather_row_cp(a.own + (((size_t)src * 2 + 1) * L + i) * N, row_off, gal, tb.logN, lrow, e0, w);
#pragma unroll
                for (int k = 0; k < 16; k++) v[k] = AR::round_reduce(AR::from_canon(w[k], m), m);
            }
        } else if (HOISTED) {
            u64 w[16];
            gather_row_cp(a.dt + ((size_t)j * D + i) * N, row_off, gal, tb.logN, lrow, e0, w);
#pragma unroll
            for (int k = 0; k < 16; k++) v[k] = AR::round_reduce(AR::from_canon(w[k], m), m);
        } else {
            const u64* p = a.dt + (((size_t)src * tb.dnum + j) * D + i) * N + row_off;
#pragma unroll
            for (int k = 0; k < 16; k++) v[k] = AR::from_raw(__builtin_nontemporal_load(&p[k * 16 + e0]));
            if constexpr (TWL) NttCore<AR, A>::fwd_contig_with(v, lrow, e0, RowTwLds{twblk, e0}, m);
            else NttCore<AR, A>::fwd_contig(v, lrow, e0, r, ti, tf, N, m);
            AR::mid_reduce(v, m);
            exchange_cb_to_cp<AR>(v, lrow, e0);
        }
        if constexpr (!EARLY0) load_row_cp<false>(k0, e0, kv0);
#pragma unroll
        for (int k = 0; k < 16; k++) AR::acc_mac(acc0[k], v[k], kv0[k], m);
        if constexpr (!EARLY1) load_row_cp<false>(k1, e0, kv1);
#pragma unroll
        for (int k = 0; k < 16; k++) AR::acc_mac(acc1[k], v[k], kv1[k], m);
        if (++since == fold_at) {
            since = 0;
#pragma unroll
            for (int k = 0; k < 16; k++) acc0[k] = AR::acc_fold(acc0[k], m), acc1[k] = AR::acc_fold(acc1[k], m);
        }
    }
    if (!HOISTED && ways != 1) {
        // The wavefronts of a team join their sums, the first two end with a component each: the other two of a team of four add
        // theirs to those of the first, which then exchange a component with one another as a team of two does.
        auto put = [&](u32 at, const T (&acc)[16]) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 16; k++) lds[at * 1024 + k * 64 + (tid & 63)] = AR::to_raw(acc[k]);
        };
        auto join = [&](u32 at, T (&acc)[16]) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 16; k++) acc[k] = AR::wide_join(acc[k], AR::from_raw(lds[at * 1024 + k * 64 + (tid & 63)]), m);
        };
#pragma unroll
        for (int k = 0; k < 16; k++) acc0[k] = AR::acc_fold(acc0[k], m), acc1[k] = AR::acc_fold(acc1[k], m);
        __syncthreads();  // the exchanges of the transforms have been read
        if (ways == 4) {
            if (wave > 1) put(wave - 2, acc0), put(wave, acc1);
            __syncthreads();
            if (wave < 2) join(wave, acc0), join(wave + 2, acc1);
        }
        if (part == 0) put(wave, acc1);  // block `wave` has been read by this wavefront alone
        else if (part == 1) put(wave, acc0);
        __syncthreads();
        if (part == 0) join(wave ^ 1, acc0);
        else if (part == 1) join(wave ^ 1, acc1);
        __syncthreads();
        if (part > 1) return;
    }
    // An opaque copy of the lane's row, and of its other coordinates below: every address of what follows is derived from them, so none
    // of it is computed before the accumulation loop, which has no registers to spare (both arithmetics, HMult with the merged rescale: 12 bytes of scratch without).
    u32 chl = ch;
    if (!FUSED) asm volatile("" : "+v"(chl));
    const u32 rl = r0 + (chl & 3);
    if (FUSED) {
        // c' stays in registers: out = (c' - second forward pass of the converted special part) * P^-1
        // (+ sigma_g(b) on the first component of a rotation; adding it as P * sigma_g(b) where sigma_g(a) is
        // gathered measured slower: the accumulation loop has no registers for it).  FP64 magnitudes in units
        // of q: c' <= 0.5, v <= 5.2 (narrow primes 10.5), the product with P^-1 <= 2.9; canonicalised before the store.
        u32 e0f = e0, chf = ch, gal_fin = gal;
        asm volatile("" : "+v"(e0f), "+v"(chf), "+s"(gal_fin));
        const PinvConst pinv = a.fin_pinv[i];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            if (ways != 1 && part != (u32)t) continue;
            // IntAr, whose twiddles come from memory: opaque for each component again, or the addresses of all of them are computed once for
            // both and wait in scratch memory (348 to 480 bytes), a reload before every twiddle.
            if constexpr (!TWL) asm volatile("" : "+v"(e0f), "+v"(chf));
            const u32 rf = r0 + (chf & 3), row_off_f = rf * 256;
            u64* lrow_f = lds + chf * 272;
            T v[16];
            const u64* p = a.cv + (((size_t)inst * 2 + t) * a.split + i) * N + row_off_f;
#pragma unroll
            for (int k = 0; k < 16; k++) v[k] = AR::from_raw(__builtin_nontemporal_load(&p[k * 16 + e0f]));
            if constexpr (TWL) NttCore<AR, A>::fwd_contig_with(v, lrow_f, e0f, RowTwLds{lds + NTT_LDS_WORDS + chf * CKKS_ROW_TW_WORDS, e0f}, m);
            else NttCore<AR, A>::fwd_contig(v, lrow_f, e0f, rf, ti, tf, N, m);
            exchange_cb_to_cp<AR>(v, lrow_f, e0f);
            u64 res[16];
#pragma unroll
            for (int k = 0; k < 16; k++) {
                const T fin = AR::acc_finish(t ? acc1[k] : acc0[k], m);
                if constexpr (AR::is_fp) res[k] = AR::to_raw(FpAr::mulmod_lazy(fin - v[k], pinv.d, FpAr::mod(pc)));
                else res[k] = mul_shoup(submod(AR::acc_canon(fin, m), AR::canon_fwd(v[k], m), pc.q), pinv.w, pinv.wp, pc.q);
            }
            if (SUM && t == 0) {
                for (u32 g = 0; g < a.n_sum; g++) {
                    u64 bw[16];
                    gather_row_cp(a.own + ((size_t)g * 2 * L + i) * N, row_off_f, a.galois[g], tb.logN, lrow_f, e0f, bw);
#pragma unroll
                    for (int k = 0; k < 16; k++) {  // FP64: at most 2.9 q + 1, then 1.5 q
                        if constexpr (AR::is_fp) res[k] = AR::to_raw(FpAr::reduce(AR::from_raw(res[k]) + u64_to_f64(bw[k]), FpAr::mod(pc)));
                        else res[k] = addmod(res[k], bw[k], pc.q);
                    }
                }
            }
            if (OWN == OWN_ROT && t == 0) {
                u64 bw[16];
                gather_row_cp(a.own + ((size_t)inst * 2 * L + i) * N, row_off_f, gal_fin, tb.logN, lrow_f, e0f, bw);
#pragma unroll
                for (int k = 0; k < 16; k++) {
                    if constexpr (AR::is_fp) res[k] = AR::to_raw(AR::from_raw(res[k]) + u64_to_f64(bw[k]));
                    else res[k] = addmod(res[k], bw[k], pc.q);
                }
            }
            if constexpr (AR::is_fp) {
#pragma unroll
                for (int k = 0; k < 16; k++) res[k] = FpAr::canon(AR::from_raw(res[k]), FpAr::mod(pc));
            }
            store_row_cp(a.out + (((size_t)inst * 2 + t) * a.split + i) * N + row_off_f, e0f, res);
        }
    } else if (i < a.split) {
        u64 res[16];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            if (ways != 1 && part != (u32)t) continue;
#pragma unroll
            for (int k = 0; k < 16; k++) res[k] = AR::acc_canon(AR::acc_finish(t ? acc1[k] : acc0[k], m), m);
            store_row_cp(a.cq + (((size_t)inst * 2 + t) * a.split + i) * N + rl * 256, e0, res);
        }
    } else {
#pragma unroll
        for (int t = 0; t < 2; t++) {
            if (ways != 1 && part != (u32)t) continue;
            T x[16];
#pragma unroll
            for (int k = 0; k < 16; k++) x[k] = AR::acc_finish(t ? acc1[k] : acc0[k], m);
            exchange_cp_to_cb<AR>(x, lrow, e0);
            NttCore<AR, A>::inv_contig(x, lrow, e0, rl, ti, tf, N, m);
            u64* o = a.cp + (((size_t)inst * 2 + t) * (D - a.split) + (i - a.split)) * N + rl * 256;
#pragma unroll
            for (int k = 0; k < 16; k++) o[k * 16 + e0] = AR::to_raw(AR::round_reduce(x[k], m));
        }
    }
}

template <class AR, int A, int OWN, bool HOISTED, bool FUSED>
__global__ __launch_bounds__(256, 2) void ks_inner_kernel(InnerArgs a, Tables tb, LimbRun run) {
    constexpr bool ANY = __is_same(AR, AnyAr), TWL = !HOISTED && !__is_same(AR, IntAr);
    __shared__ u64 lds[NTT_LDS_WORDS + (TWL ? 16 * CKKS_ROW_TW_WORDS : 0)];
    const u32 TILES = (1u << A) / 16 * (HOISTED ? 1 : a.ways);
    u32 group, inst;
    if (!xcd_decode(blockIdx.x, a.n_inst, run.count * TILES, group, inst)) return;
    // both arithmetics in one launch: the special limbs, the longer workgroups, first
    const u32 i = ANY ? run.first + run.count - 1 - group / TILES : run.first + group / TILES;
    CKKS_BY_ARITHMETIC(AR, i, (ks_inner_body<AR_, A, OWN, HOISTED, FUSED>(a, tb, lds, i, group % TILES, inst)))
}

// ===================================================== double-hoisted rotate-multiply-accumulate
// Over the rotations r of the launch and the digits j, on every limb i of the extended basis:
//   C_t[i] += pt_r[i] * (sum_j sigma_{g_r}(Dh_j)[i] * rk_r[j][t][i]),   t = 0, 1,
// with Dh_j the transformed digits (the polynomial's own limb on the digit that owns limb i).  On q-limbs sigma_{g_r}(b) * P
// joins the sum of t = 0: ModDown divides it by P exactly, which gives the same words as adding pt_r * sigma_{g_r}(b) after
// ModDown.  C_t is stored canonical, evaluation form: q-limbs in cq, special limbs in cp (ModDown follows).
//
// No transform is involved; keys and plaintexts stream from HBM once and bound the kernel.  What it spent besides: a
// 64-lane gather per digit word (64 cache lines an instruction), digits re-read through the fabric for every rotation, and
// on IntAr limbs two reduced products per digit.  Hence a wavefront owns one 256-word row (lane l: words 2l, 2l+1, 128+2l,
// 128+2l+1), loads the source row whole with 16-byte accesses and permutes it in LDS (sigma_g maps rows onto rows, see
// gather_row_cp); the sum over the digits stays unreduced and meets the plaintext once per rotation; the words of the next
// term are requested before this one is worked on; each XCD takes a contiguous range of rows, limb after limb, and the
// four wavefronts of a workgroup share a row (each takes every fourth rotation), so that one limb at a time is in flight
// per XCD and its digits stay in the L2; and both arithmetics share one launch.  32 rotations at N = 2^16, L + K = 42,
// dnum = 5 (7.8 GB of keys and plaintexts): 1673 us in two launches -> 1414 us, 5.5 TB/s; without the shared rows 1623 us,
// without the early requests 1730 us, with the digit reads removed 1386 us.
#define CKKS_DH_SUMS 4
struct DhInnerArgs {
    const u64* dt;   // [dnum][D][N] canonical evaluation form
    const u64* ct;   // [2][L][N]
    const u64* pt;   // [n_rot][pt_limbs][N] canonical evaluation form; null = the constant 1
    u32 pt_limbs;    // D: extended basis; L: q-limbs, for a launch on those alone
    const u64* key[CKKS_DH_CHUNK];
    u32 galois[CKKS_DH_CHUNK];
    u64* cq;         // [2][L][N]
    u64* cp;         // [2][K][N]  (evaluation form here; the inverse transform is a separate launch)
    u32 n_rot;
    u32 accumulate;  // add to what cq / cp already hold (a call with more rotations than one launch takes)
    u32 split;       // limbs below split go to cq ([2][split][N]), the others to cp ([2][D - split][N])
    u32 waves;       // wavefronts of a workgroup that share a row, each taking every waves-th rotation: 1 (four rows) or 4
    u32 first, count;  // limbs of this launch
    u32 each;        // rotations are not summed: rotation r's result goes to cq + r*2*split*N, cp + r*2*(D - split)*N
    u32 sums;        // G > 1: G; sum g takes the plaintexts pt[g][n_rot][pt_limbs][N] and goes to cq + g*2*split*N, cp likewise
};
// Wavefronts that share a row of 128 words where several sums are formed (DhInnerArgs::waves): four where four rows a workgroup leave
// the chip half empty, counted by the wavefronts that have a rotation; one rotation is nothing to share.  Whole transforms (the
// kernel), not shared / shared, both arithmetics and integers alone, two and four sums, N = 2^12 .. 2^16: 1 baby step 0.96 to 1.00 (0.68 to 0.98) at
// every size; 2: 256 to 768 rows 1.00 to 1.01 (0.99 to 1.17), 960 and 1024 1.00 (0.94 to 1.02), 1536 0.97 to 0.99 (0.76 to 0.84); 3: 256 to
// 1024 1.00 to 1.03 (0.97 to 1.41), 1536 0.98 to 1.00 (0.87 to 1.01); 4 to 6: 768 to 1344 0.99 to 1.03 (0.94 to 1.34), 1536 to 1792 0.98 to 1.02 (0.88 to
// 1.11); 7 to 13: 768 to 1600 1.00 to 1.08 (0.99 to 1.52), 1728 and 1792 0.99 to 1.02 (0.96 to 1.09).
HD u32 sums_waves(u32 rows, u32 n_rot) { return n_rot > 1 && rows * 4 < 1792 * (n_rot < 4 ? n_rot : 4) ? 4 : 1; }

// Sum over the rotations of (unreduced digit sum, reduced) * plaintext, at most 8 terms between folds
template <class AR, int W>
struct DhSum {
    typename AR::T s;
    __device__ __forceinline__ DhSum() : s(AR::acc_zero()) {}
    __device__ __forceinline__ void add(typename AR::T v, u64 b, const typename AR::Mod& m) { AR::acc_mac_wide(s, v, b, m); }
    __device__ __forceinline__ void fold(const typename AR::Mod& m) { s = AR::acc_fold(s, m); }
    __device__ __forceinline__ typename AR::T get(const typename AR::Mod&) const { return s; }
};
// 128 bits where the registers allow it: one reduction at the end instead of one per term.  v < 2q and b < q < 2^61 make a term
// less than q * 2^62, eight of them on hi < q less than 3q * 2^64; multiples of q * 2^64 are taken off by hi alone.
template <>
struct DhSum<IntAr, 2> {
    u128w s;
    __device__ __forceinline__ DhSum() : s{0, 0} {}
    __device__ __forceinline__ void add(u64 v, u64 b, const IntAr::Mod&) { mac128(s, v, b); }
    __device__ __forceinline__ void fold(const IntAr::Mod& m) { s.hi = csub(csub(s.hi, m.q2), m.q); }
    __device__ __forceinline__ u64 get(const IntAr::Mod& m) const { return redc_lazy(u128w{s.lo, csub(csub(s.hi, m.q2), m.q)}, m.q, m.qneg); }
};

// an address that is the same in every lane, in scalar registers
template <class P>
__device__ __forceinline__ P uniform_ptr(P p) {
    const u64 v = (u64)p;
    return (P)((u64)(u32)__builtin_amdgcn_readfirstlane((int)(u32)v) | (u64)(u32)__builtin_amdgcn_readfirstlane((int)(u32)(v >> 32)) << 32);
}

// G > 1: up to G sums of the same rotations, each with plaintexts of its own (the giant steps of a transform): the rotations, kept
// in the extended basis, meet all of them in registers instead of making a round trip through memory.
template <class AR, int W, int G>
__device__ __forceinline__ void dh_accum_body(const DhInnerArgs& a, const Tables& tb, const PrimeConst& pc, u64* lds, u32 i, u32 row, u32 wave) {
    typedef typename AR::T T;
    typedef typename AR::Wide Wide;
    constexpr u32 ROW = 64 * W;
    const u32 logN = tb.logN, N = 1u << logN, lane = threadIdx.x & 63, L = tb.L, D = tb.D;
    const u32 pi = tb.phys(i), Dkey = tb.Lfull + tb.K;
    const bool is_q = i < L;
    const typename AR::Mod m = AR::mod(pc);
    const u32 own_digit = is_q ? i / tb.alpha : 0xffffffffu, row_off = row * ROW;
    const u64 pmod = is_q ? tb.pmod[i] : 0;
    u64* stage = lds + wave * ROW;
    auto load = [&](const u64* p, u64 (&o)[W], bool nt) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < W / 2; h++) {
            const u64x2* q = reinterpret_cast<const u64x2*>(p + h * 128 + lane * 2);
            const u64x2 t = nt ? __builtin_nontemporal_load(q) : *q;
            o[2 * h] = t.x, o[2 * h + 1] = t.y;
        }
    };
    const u32 sp = a.split;
    auto out = [&](u32 rr, int t) {
        u64* base = i < sp ? a.cq + ((size_t)t * sp + i) * N : a.cp + ((size_t)t * (D - sp) + (i - sp)) * N;
        return base + (a.each || G > 1 ? (size_t)rr * 2 * (i < sp ? sp : D - sp) * N : 0) + row_off;
    };
    auto store = [&](const T (&acc)[W], u64* o) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < W / 2; h++) {
            u64x2* q = reinterpret_cast<u64x2*>(o + h * 128 + lane * 2);
            u64x2 r;
            r.x = AR::acc_canon(AR::acc_finish2(acc[2 * h], m), m), r.y = AR::acc_canon(AR::acc_finish2(acc[2 * h + 1], m), m);
            if (a.accumulate) {
                const u64x2 p = *q;
                r.x = addmod(r.x, p.x, pc.q), r.y = addmod(r.y, p.y, pc.q);
            }
            *q = r;
        }
    };
    typedef DhSum<AR, G == 1 ? W : 0> Sum;  // G > 1: no registers for 128-bit sums
    Sum acc0[G][W], acc1[G][W];
    typedef const u64 __attribute__((address_space(1))) * Global;  // known to be global behind an opaque selection
    const u64 *ct = a.ct, *dt = a.dt;
    const size_t pt_step = (size_t)a.pt_limbs * N;
    u64 sv[W], kv0[W], kv1[W];  // the term worked on: row of the digit or of b, both components of the key
    Wide w0[W], w1[W];
#pragma unroll
    for (int k = 0; k < W; k++) w0[k] = w1[k] = AR::wide_zero();
    u32 folds = 0, in_sum = 0, rr = a.waves == 1 ? 0 : wave, idx[W];
    auto permutation = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < W; k++) idx[k] = eval_perm(row_off + (k >> 1) * 128 + lane * 2 + (k & 1), a.galois[rr], logN) & (ROW - 1);
    };
    auto permute = [&]() __attribute__((always_inline)) {
        row_sync();  // the previous term's words have been read
#pragma unroll
        for (int h = 0; h < W / 2; h++) {
            u64x2 t;
            t.x = sv[2 * h], t.y = sv[2 * h + 1];
            *reinterpret_cast<u64x2*>(stage + h * 128 + lane * 2) = t;
        }
        row_sync();
#pragma unroll
        for (int k = 0; k < W; k++) sv[k] = stage[idx[k]];
    };
    if constexpr (G > 1) {
        // Terms of a rotation: digits 0 .. dnum - 1, then one for every two plaintexts, the first of which also brings b (times P, on
        // q-limbs).  The words of the next term, also across rotations, are requested before this one is worked on, and no request
        // depends on a branch: behind one that may skip a load, the compiler waits for all of them before the previous term's words
        // are used.  The digits end before the plaintexts come, so that no register holds a plaintext meanwhile: 104 registers and
        // four waves per SIMD with four sums where a loop over all terms took 168 and three (8 x 4 transform at N = 2^16, 24 + 6
        // limbs: 387 -> 354 us, 1.6 GB).
        constexpr u32 PT = (G + 1) / 2;
        u64 sn[W], kn0[W], kn1[W];
        auto source = [&](u32 r) { return eval_perm(row_off, a.galois[r], logN) & ~(ROW - 1); };
        auto request_digit = [&](u32 r, u32 j, u64 (&s)[W], u64 (&k0)[W], u64 (&k1)[W]) __attribute__((always_inline)) {
            const u64* key = a.key[r] + ((size_t)j * 2 * Dkey + pi) * N + row_off;
            Global row = uniform_ptr((Global)((j == own_digit ? ct + ((size_t)L + i) * N : dt + ((size_t)j * D + i) * N) + source(r)));
            asm volatile("" : "+s"(row));  // the address is selected, not the load skipped
            load((const u64*)row, s, false);
            load(key, k0, true);
            load(key + (size_t)Dkey * N, k1, true);
        };
        // plaintexts 2u and 2u + 1; u = 0: and b, or, on special limbs, a row that is not used
        auto request_pt = [&](u32 r, u32 u, u64 (&s)[W], u64 (&k0)[W], u64 (&k1)[W]) __attribute__((always_inline)) {
            const u64* pt = a.pt + ((size_t)(2 * u) * a.n_rot + r) * pt_step + (size_t)i * N + row_off;
            Global row = uniform_ptr((Global)((is_q ? ct : dt) + (size_t)i * N + source(r)));
            asm volatile("" : "+s"(row));
            if (u == 0) load((const u64*)row, s, false);
            load(pt, k0, true);
            if (2 * u + 1 < G) load(pt + (size_t)a.n_rot * pt_step, k1, true);
        };
        if (rr < a.n_rot) request_digit(rr, 0, sv, kv0, kv1);
        while (rr < a.n_rot) {
            permutation();
            T d0[W], d1[W];  // the rotation's digit sums
#pragma unroll
            for (int k = 0; k < W; k++) d0[k] = d1[k] = AR::acc_zero();
            auto join = [&](bool last) __attribute__((always_inline)) {
#pragma unroll
                for (int k = 0; k < W; k++) {
                    join_part<AR>(d0[k], AR::wide_reduce(w0[k], m), last, m);
                    join_part<AR>(d1[k], AR::wide_reduce(w1[k], m), last, m);
                    w0[k] = w1[k] = AR::wide_zero();
                }
                in_sum = 0;
            };
            auto advance = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int k = 0; k < W; k++) sv[k] = sn[k], kv0[k] = kn0[k], kv1[k] = kn1[k];
            };
            auto digit = [&]() __attribute__((always_inline)) {
                permute();
#pragma unroll
                for (int k = 0; k < W; k++) AR::wide_mac(w0[k], sv[k], kv0[k]), AR::wide_mac(w1[k], sv[k], kv1[k]);
                if (++in_sum == AR::wide_terms) join(false);
                advance();
            };
            for (u32 j = 1; j < tb.dnum; j++) {
                request_digit(rr, j, sn, kn0, kn1);
                digit();
            }
            request_pt(rr, 0, sn, kn0, kn1);
            digit();
            ++folds;  // FP64: at most 8 products (0.875 q each, join_part) between reductions
            const u32 next = rr + a.waves < a.n_rot ? rr + a.waves : rr;  // at the end a term once more, unused
#pragma unroll
            for (u32 u = 0; u < PT; u++) {
                if (u + 1 < PT) request_pt(rr, u + 1, sn, kn0, kn1);
                else request_digit(next, 0, sn, kn0, kn1);
                if (u == 0) {
                    if (is_q) {
                        permute();
#pragma unroll
                        for (int k = 0; k < W; k++) AR::wide_mac(w0[k], sv[k], pmod);
                    }
                    join(true);
                }
#pragma unroll
                for (u32 g = 2 * u; g < (u32)G && g < 2 * u + 2; g++) {
#pragma unroll
                    for (int k = 0; k < W; k++) {
                        acc0[g][k].add(d0[k], g & 1 ? kv1[k] : kv0[k], m);
                        acc1[g][k].add(d1[k], g & 1 ? kv1[k] : kv0[k], m);
                        if ((folds & 7) == 0) acc0[g][k].fold(m), acc1[g][k].fold(m);
                        __builtin_amdgcn_sched_barrier(0);  // one product's temporaries at a time
                    }
                }
                advance();
            }
            rr += a.waves;
        }
    } else {
        // terms of a rotation: digits 0 .. dnum - 1, then (q-limbs) b times P.  The words of the next term, also across
        // rotations, are requested before this one is worked on: a wavefront of the wide form has 12 KiB in flight.
        const u32 n_terms = tb.dnum + (is_q ? 1 : 0);
        u64 ptv[W];
#pragma unroll
        for (int k = 0; k < W; k++) ptv[k] = 1;
        // EVEN: every request is the same number of loads, and what a term does not need is the source row once more (L2): behind
        // a branch that may skip some, the compiler waits for all of them before the previous term's words are used.  The narrow
        // form gains (18 rotations, L + K = 12 + 4, dnum = 3: 360 -> 354 us), the wide one loses by the extra loads (24 + 6: 672 -> 684).
        constexpr bool EVEN = W == 2;
        auto request = [&](u32 r, u32 j, u64 (&s)[W], u64 (&k0)[W], u64 (&k1)[W], u64 (&p)[W]) __attribute__((always_inline)) {
            const u32 src_off = eval_perm(row_off, a.galois[r], logN) & ~(ROW - 1);
            const bool is_b = j == tb.dnum;
            const u64* src = (is_b ? ct + (size_t)i * N : j == own_digit ? ct + ((size_t)L + i) * N : dt + ((size_t)j * D + i) * N) + src_off;
            const u64* key = a.key[r] + ((size_t)j * 2 * Dkey + pi) * N + row_off;
            const u64* pt = a.pt + r * pt_step + (size_t)i * N + row_off;
            if constexpr (EVEN) {
                Global kp = (Global)(is_b ? src : key), kp1 = (Global)(is_b ? src : key + (size_t)Dkey * N), pp = (Global)(j == 0 && a.pt ? pt : src);
                asm volatile("" : "+s"(kp), "+s"(kp1), "+s"(pp));  // addresses selected, not loads skipped
                load(src, s, false);
                load((const u64*)kp, k0, true);
                load((const u64*)kp1, k1, true);
                load((const u64*)pp, p, true);
            } else {
                load(src, s, false);
                if (!is_b) {
                    load(key, k0, true);
                    load(key + (size_t)Dkey * N, k1, true);
                }
                if (j == 0 && a.pt) load(pt, p, true);
            }
        };
        u32 j = 0;
        if (rr < a.n_rot) request(rr, 0, sv, kv0, kv1, ptv);
        while (rr < a.n_rot) {
            permutation();
            for (; j < n_terms; j++) {
                const bool last = j + 1 == n_terms;
                const bool more = !last || rr + a.waves < a.n_rot;  // else (EVEN) this term once more, unused
                u64 sn[W], kn0[W], kn1[W], pn[W];
#pragma unroll
                for (int k = 0; k < W; k++) pn[k] = 1;
                if (EVEN || more) request(more && last ? rr + a.waves : rr, !more ? j : last ? 0 : j + 1, sn, kn0, kn1, pn);
                permute();
                if (j == tb.dnum) {
#pragma unroll
                    for (int k = 0; k < W; k++) AR::wide_mac(w0[k], sv[k], pmod);
                } else {
#pragma unroll
                    for (int k = 0; k < W; k++) AR::wide_mac(w0[k], sv[k], kv0[k]), AR::wide_mac(w1[k], sv[k], kv1[k]);
                }
                if (++in_sum == AR::wide_terms || last) {
                    in_sum = 0;
#pragma unroll
                    for (int k = 0; k < W; k++) {
                        const u64 ptk = EVEN && !a.pt ? 1 : ptv[k];
                        acc0[0][k].add(AR::wide_reduce(w0[k], m), ptk, m);
                        acc1[0][k].add(AR::wide_reduce(w1[k], m), ptk, m);
                        w0[k] = w1[k] = AR::wide_zero();
                    }
                    if ((++folds & 7) == 0) {  // FP64: at most 8 products (0.69 q each) between reductions
#pragma unroll
                        for (int k = 0; k < W; k++) acc0[0][k].fold(m), acc1[0][k].fold(m);
                    }
                }
#pragma unroll
                for (int k = 0; k < W; k++) {
                    sv[k] = sn[k], kv0[k] = kn0[k], kv1[k] = kn1[k];
                    if (last) ptv[k] = pn[k];
                }
            }
            if (a.each) {
                T t0[W], t1[W];
#pragma unroll
                for (int k = 0; k < W; k++) t0[k] = acc0[0][k].get(m), t1[k] = acc1[0][k].get(m), acc0[0][k] = acc1[0][k] = Sum();
                store(t0, out(rr, 0));
                store(t1, out(rr, 1));
                folds = 0;
            }
            j = 0, rr += a.waves;
        }
    }
    if (G == 1 && a.each) return;
#pragma unroll
    for (int g = 0; g < G; g++) {
        T t0[W], t1[W];
#pragma unroll
        for (int k = 0; k < W; k++) t0[k] = acc0[g][k].get(m), t1[k] = acc1[g][k].get(m);
        if (a.waves > 1) {  // the first of the row's four wavefronts joins their sums
#pragma unroll
            for (int k = 0; k < W; k++) t0[k] = AR::acc_fold(t0[k], m), t1[k] = AR::acc_fold(t1[k], m);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < W; k++) {
                lds[(wave * 2 + 0) * ROW + k * 64 + lane] = AR::to_raw(t0[k]);
                lds[(wave * 2 + 1) * ROW + k * 64 + lane] = AR::to_raw(t1[k]);
            }
            __syncthreads();
            if (wave == 0) {
#pragma unroll
                for (int k = 0; k < W; k++)
#pragma unroll
                    for (int v = 1; v < 4; v++) {
                        t0[k] = AR::wide_join(t0[k], AR::from_raw(lds[(v * 2 + 0) * ROW + k * 64 + lane]), m);
                        t1[k] = AR::wide_join(t1[k], AR::from_raw(lds[(v * 2 + 1) * ROW + k * 64 + lane]), m);
                    }
            }
        }
        if (a.waves == 1 || wave == 0) {
            store(t0, out(g, 0));
            store(t1, out(g, 1));
        }
    }
}

// W words per lane; a row, a wavefront's share, is 64 times that (sigma_g maps every aligned block of 2^m slots onto one).
// AnyAr, FP64 and integer limbs in one launch: rows of 256 words, 12 KiB in flight per wavefront and three waves per SIMD, or
// of 128 and five.  IntAr, for chains of integer primes alone: rows of 128 words.  launch_dh_accum has the rule.
template <class AR, int W, int G>
__device__ __forceinline__ void dh_accum_workgroup(const DhInnerArgs& a, const Tables& tb) {
    __shared__ __align__(16) u64 lds[512 * W];  // a row per wavefront to permute it in; eight to join four pairs of sums
    const u32 rows_wg = 4 / a.waves, per_limb = ((1u << tb.logN) / (64 * W)) / rows_wg, total = a.count * per_limb, per = (total + 7) / 8;
    const u32 pos = blockIdx.x >> 3, q = (blockIdx.x & 7) * per + pos;  // workgroups go to the XCDs round-robin
    if (pos >= per || q >= total) return;
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // uniform: addresses stay in scalar registers
    const u32 i = a.first + q / per_limb, row = (q % per_limb) * rows_wg + (a.waves == 1 ? wave : 0);
    const PrimeConst pc = tb.pc[tb.phys(i)];
    CKKS_BY_ARITHMETIC(AR, i, (dh_accum_body<AR_, W, G>(a, tb, pc, lds, i, row, wave)))
}
// one sum, or G of them
template <class AR, int W>
__global__ __launch_bounds__(256, W == 4 ? 3 : 5) void dh_accum_kernel(DhInnerArgs a, Tables tb) { dh_accum_workgroup<AR, W, 1>(a, tb); }
template <class AR, int W, int G>
__global__ __launch_bounds__(256, 4) void dh_accum_kernel(DhInnerArgs a, Tables tb) { dh_accum_workgroup<AR, W, G>(a, tb); }

// ==================================================== baby-step giant-step accumulation and sums
// C[g][t][i] = sum_b pt[g][b][i] * R[b][t][i] on every limb i of the extended basis: the giant-step
// combinations of the baby-step rotations R_b (kept in the extended basis, times P).  Element-parallel;
// one workgroup per 256 * EPT slots of (limb, giant step).
struct BsgsMacArgs {
    const u64* rq;  // [n1][2][L][N]  q-limbs of R_b
    const u64* rp;  // [n1][2][K][N]  special limbs of R_b
    const u64* pt;  // [n2][n1][D][N]
    u64* cq;        // [n2][2][L][N]
    u64* cp;        // [n2][2][K][N]
    u32 n1, n2;
};

template <class AR, int EPT>
__global__ __launch_bounds__(256) void bsgs_mac_kernel(BsgsMacArgs a, Tables tb, LimbRun run) {
    typedef typename AR::T T;
    const u32 N = 1u << tb.logN, tid = threadIdx.x, L = tb.L, K = tb.K, D = tb.D;
    const u32 chunks = N / (256 * EPT);
    // the giant steps of one (limb, slot range) share the R_b they read: adjacent on one XCD
    u32 rest, g;
    if (!xcd_decode(blockIdx.x, a.n2, run.count * chunks, rest, g)) return;
    const u32 i = run.first + rest / chunks, base = (rest % chunks) * (256 * EPT) + tid;
    const PrimeConst pc = tb.pc[tb.phys(i)];
    const typename AR::Mod m = AR::mod(pc);
    const bool is_q = i < L;
    T acc0[EPT], acc1[EPT];
    u128w w0[EPT], w1[EPT];
#pragma unroll
    for (int k = 0; k < EPT; k++) acc0[k] = AR::acc_zero(), acc1[k] = AR::acc_zero(), w0[k] = u128w{0, 0}, w1[k] = u128w{0, 0};
    for (u32 b = 0; b < a.n1; b++) {
        const u64* r0 = (is_q ? a.rq + (((size_t)b * 2 + 0) * L + i) * N : a.rp + (((size_t)b * 2 + 0) * K + (i - L)) * N) + base;
        const u64* r1 = (is_q ? a.rq + (((size_t)b * 2 + 1) * L + i) * N : a.rp + (((size_t)b * 2 + 1) * K + (i - L)) * N) + base;
        const u64* pp = a.pt + (((size_t)g * a.n1 + b) * D + i) * N + base;
#pragma unroll
        for (int k = 0; k < EPT; k++) {
            const u64 pv = __builtin_nontemporal_load(&pp[k * 256]);
            if constexpr (AR::is_fp) {
                acc0[k] += AR::premul(r0[k * 256], pv, m);
                acc1[k] += AR::premul(r1[k * 256], pv, m);
            } else {  // at most 64 products below 2^122 fit the 128-bit accumulator
                mac128(w0[k], r0[k * 256], pv);
                mac128(w1[k], r1[k * 256], pv);
            }
        }
        if constexpr (AR::is_fp) {
            if ((b & 7) == 7) {
#pragma unroll
                for (int k = 0; k < EPT; k++) acc0[k] = AR::acc_fold(acc0[k], m), acc1[k] = AR::acc_fold(acc1[k], m);
            }
        }
    }
    u64* o0 = (is_q ? a.cq + (((size_t)g * 2 + 0) * L + i) * N : a.cp + (((size_t)g * 2 + 0) * K + (i - L)) * N) + base;
    u64* o1 = (is_q ? a.cq + (((size_t)g * 2 + 1) * L + i) * N : a.cp + (((size_t)g * 2 + 1) * K + (i - L)) * N) + base;
#pragma unroll
    for (int k = 0; k < EPT; k++) {
        if constexpr (AR::is_fp) {
            o0[k * 256] = AR::acc_canon(AR::acc_finish(acc0[k], m), m);
            o1[k * 256] = AR::acc_canon(AR::acc_finish(acc1[k], m), m);
        } else {
            o0[k * 256] = reduce128(w0[k], pc.q, pc.qneg, pc.r2);
            o1[k * 256] = reduce128(w1[k], pc.q, pc.qneg, pc.r2);
        }
    }
}

// out[l][n] = sum_g in[g][l][n] mod q_l over n_limbs limbs per item (limb l uses prime l % L).
__global__ __launch_bounds__(256) void sum_instances_kernel(const u64* __restrict__ in, u64* __restrict__ out,
                                                            const PrimeConst* pcs, u32 logN, u32 L, u32 n_limbs, u32 n_g) {
    const u32 N = 1u << logN;
    const u32 n = blockIdx.x * 256 + threadIdx.x, l = blockIdx.y;
    const u64 q = pcs[l % L].q;
    u64 acc = 0;
    for (u32 g = 0; g < n_g; g++) acc = addmod(acc, in[((size_t)g * n_limbs + l) * N + n], q);
    out[(size_t)l * N + n] = acc;
}

// ======================================================================== final combine
// ks_t[i] = (c'_t[i] - NTT(conv_t)[i]) * P^-1 mod q_i, the NTT's second pass done here, then
//   FIN_KS     : out[inst / 2][t][i] = ks, t = inst % 2: a workgroup per component, the two adjacent on one XCD (with both in one
//                workgroup, one after the other: rescale of one ciphertext at N = 2^16, 24 limbs 38.4 us, so 35.5; 8 of 35 limbs 240, 235)
//   FIN_HOISTED: out[t][i] (+)= sum_r pt_r[i] * (ks_r + (t == 0 ? sigma_{g_r}(b) : 0)); work item (i, tile, t)
//   FIN_SUMMED : the same words as (C_t - sum_r pt_r * NTT(conv_{r,t})) * P^-1 with C_t = sum_r pt_r * (c'_{r,t} + P * (t == 0 ?
//                sigma_{g_r}(b) : 0)), which dh_accum_kernel has left in cq: on a q-limb everything after the conversions is linear,
//                so neither c' nor sigma_{g_r}(b) of a single rotation reaches memory; work item (i, tile, t)
// (HMult, HRot and the plain key switch end inside the inner-product kernel, which also adds the tensor
// terms or sigma_g(b).)  The numbering keeps kernel names stable.
enum FinalMode { FIN_KS = 0, FIN_HOISTED = 3, FIN_SUMMED = 4 };
struct FinalArgs {
    const u64* cq;   // [g][2][L][N] canonical; SUMMED: C [2][L][N]
    const u64* cv;   // [g][2][L][N] raw forward-lazy (first pass done)
    const u64* ct1;  // HOISTED: ct
    const u64* pt;   // HOISTED, SUMMED: plaintexts of this chunk [n_rot][L][N]
    u64* out;
    u32 galois[CKKS_ROT_CHUNK];  // HOISTED
    u32 n_inst;      // KS: 2 * batch; HOISTED, SUMMED: 2, the component t
    u32 n_rot;       // HOISTED, SUMMED
    u32 accumulate;  // HOISTED, SUMMED: add to what out already holds
    u32 cq_L;        // limbs per component of cq (L, or L + 1 when cq is a ciphertext about to lose its last limb)
};

// CACHED (KS): ordinary loads of cv (loads_cached)
template <class AR, int A, int MODE, bool CACHED = false>
__device__ __forceinline__ void ks_final_body(const FinalArgs& a, const Tables& tb, u64* lds, u32 i, u32 tile, u32 inst) {
    typedef typename AR::T T;
    const u32 N = 1u << tb.logN, tid = threadIdx.x, e0 = tid % 16, ch = tid / 16, r = tile * 16 + ch;
    const u32 L = tb.L;
    const PrimeConst pc = tb.pc[i];
    const typename AR::Mod m = AR::mod(pc);
    const PinvConst pinv = tb.pinv[i];
    const u64* ti = tb.tw_int + (size_t)i * 4 * N;
    const double* tf = tb.tw_fp + (size_t)i * 2 * N;
    u64* lrow = lds + ch * 272;
    const u32 row_off = r * 256;
    const u64 q = pc.q;
    // The converted part leaves its second forward pass in layout CP: c', plaintexts and results move with 16-byte
    // accesses, and sigma_g(b) comes as a whole source row permuted in LDS (gather_row_cp).
    // FP64 pipe (magnitudes in units of q): v <= 5.2, c' - v <= 6.2, ks = (c' - v) * P^-1 <= 2.9 (narrow primes 10.5, 11.5, 2.8),
    // every added product of canonical operands <= 0.875; everything is canonicalised before the store.
    if (MODE == FIN_HOISTED) {
        const u32 t = inst;
        double facc[AR::is_fp ? 16 : 1];
        u128w iacc[AR::is_fp ? 1 : 16];
#pragma unroll
        for (int k = 0; k < 16; k++) {
            if constexpr (AR::is_fp) facc[k] = 0.0;
            else iacc[k] = u128w{0, 0};
        }
        for (u32 rr = 0; rr < a.n_rot; rr++) {
            T v[16];
            const u64* p = a.cv + (((size_t)rr * 2 + t) * L + i) * N + row_off;
#pragma unroll
            for (int k = 0; k < 16; k++) v[k] = AR::from_raw(__builtin_nontemporal_load(&p[k * 16 + e0]));
            NttCore<AR, A>::fwd_contig(v, lrow, e0, r, ti, tf, N, m);
            exchange_cb_to_cp<AR>(v, lrow, e0);
            // one operand stream at a time: c', then sigma_g(b), then the plaintext (16 words each)
            T ks[16];
            {
                u64 c[16];
                load_row_cp<true>(a.cq + (((size_t)rr * 2 + t) * L + i) * N + row_off, e0, c);
#pragma unroll
                for (int k = 0; k < 16; k++) {
                    if constexpr (AR::is_fp) ks[k] = FpAr::mulmod_lazy(u64_to_f64(c[k]) - v[k], pinv.d, FpAr::mod(pc));
                    else ks[k] = mul_shoup(submod(c[k], AR::canon_fwd(v[k], m), q), pinv.w, pinv.wp, q);
                }
            }
            if (t == 0) {
                u64 bw[16];
                gather_row_cp(a.ct1 + (size_t)i * N, row_off, a.galois[rr], tb.logN, lrow, e0, bw);
#pragma unroll
                for (int k = 0; k < 16; k++) {
                    if constexpr (AR::is_fp) ks[k] += u64_to_f64(bw[k]);
                    else ks[k] = addmod(ks[k], bw[k], q);
                }
            }
            {
                u64 ptw[16];
                load_row_cp<true>(a.pt + ((size_t)rr * L + i) * N + row_off, e0, ptw);
                AR::mid_reduce(ks, m);
#pragma unroll
                for (int k = 0; k < 16; k++) {
                    // FP64: ks reduced to <= q/2, so that the at most 8 products accumulated between folds stay below 6 q; narrow primes:
                    // ks <= 3.8 q, 1.3 q a product
                    if constexpr (AR::is_fp) facc[k] += FpAr::mulmod_lazy(ks[k], u64_to_f64(ptw[k]), FpAr::mod(pc));
                    else mac128(iacc[k], ks[k], ptw[k]);
                }
            }
            if constexpr (AR::is_fp) {
                if ((rr & 7) == 7) {
#pragma unroll
                    for (int k = 0; k < 16; k++) facc[k] = FpAr::reduce(facc[k], FpAr::mod(pc));
                }
            }
        }
        u64* o = a.out + ((size_t)t * L + i) * N + row_off;
        u64 prev[16], res[16];
        if (a.accumulate) load_row_cp<false>(o, e0, prev);
#pragma unroll
        for (int k = 0; k < 16; k++) {
            if constexpr (AR::is_fp) {
                double x = facc[k];
                if (a.accumulate) x += u64_to_f64(prev[k]);
                res[k] = FpAr::canon(x, FpAr::mod(pc));
            } else {
                res[k] = reduce128(iacc[k], q, pc.qneg, pc.r2);
                if (a.accumulate) res[k] = addmod(res[k], prev[k], q);
            }
        }
        store_row_cp(o, e0, res);
        return;
    }
    if (MODE == FIN_SUMMED) {
        const u32 t = inst, fold_at = AR::is_fp && AR::narrow(m) ? 5 : 8;
        u32 since = 0;
        double facc[AR::is_fp ? 16 : 1];
        u128w iacc[AR::is_fp ? 1 : 16];
#pragma unroll
        for (int k = 0; k < 16; k++) {
            if constexpr (AR::is_fp) facc[k] = 0.0;
            else iacc[k] = u128w{0, 0};
        }
        for (u32 rr = 0; rr < a.n_rot; rr++) {
            T v[16];
            const u64* p = a.cv + (((size_t)rr * 2 + t) * L + i) * N + row_off;
#pragma unroll
            for (int k = 0; k < 16; k++) v[k] = AR::from_raw(__builtin_nontemporal_load(&p[k * 16 + e0]));
            u64 ptw[16];
            load_row_cp<true>(a.pt + ((size_t)rr * L + i) * N + row_off, e0, ptw);
            NttCore<AR, A>::fwd_contig(v, lrow, e0, r, ti, tf, N, m);
            exchange_cb_to_cp<AR>(v, lrow, e0);
            AR::mid_reduce(v, m);
#pragma unroll
            for (int k = 0; k < 16; k++) {
                // FP64: reduced to <= q/2 so that the at most 8 products accumulated between folds stay below 6 q; narrow primes: not
                // reduced, 2.6 q a product, five between folds.  Integers: a term below 2q * q < q * 2^62, eight of them on hi < q below
                // 3q * 2^64; hi alone takes multiples of q * 2^64 off
                if constexpr (AR::is_fp) facc[k] += FpAr::mulmod_lazy(v[k], u64_to_f64(ptw[k]), FpAr::mod(pc));
                else mac128(iacc[k], csub(csub(v[k], 4 * q), 2 * q), ptw[k]);
            }
            if (++since == fold_at) {
                since = 0;
#pragma unroll
                for (int k = 0; k < 16; k++) {
                    if constexpr (AR::is_fp) facc[k] = FpAr::reduce(facc[k], FpAr::mod(pc));
                    else iacc[k].hi = csub(csub(iacc[k].hi, 2 * q), q);
                }
            }
        }
        u64* o = a.out + ((size_t)t * L + i) * N + row_off;
        u64 c[16], prev[16], res[16];
        load_row_cp<true>(a.cq + ((size_t)t * L + i) * N + row_off, e0, c);
        if (a.accumulate) load_row_cp<false>(o, e0, prev);
#pragma unroll
        for (int k = 0; k < 16; k++) {
            if constexpr (AR::is_fp) {
                const FpAr::Mod fm = FpAr::mod(pc);
                double x = FpAr::mulmod_lazy(u64_to_f64(c[k]) - FpAr::reduce(facc[k], fm), pinv.d, fm);
                if (a.accumulate) x += u64_to_f64(prev[k]);
                res[k] = FpAr::canon(x, fm);
            } else {
                res[k] = mul_shoup(submod(c[k], reduce128(iacc[k], q, pc.qneg, pc.r2), q), pinv.w, pinv.wp, q);
                if (a.accumulate) res[k] = addmod(res[k], prev[k], q);
            }
        }
        store_row_cp(o, e0, res);
        return;
    }
    T v[16];
    const u64* p = a.cv + ((size_t)inst * L + i) * N + row_off;
#pragma unroll
    for (int k = 0; k < 16; k++) {
        if constexpr (CACHED) v[k] = AR::from_raw(p[k * 16 + e0]);
        else v[k] = AR::from_raw(__builtin_nontemporal_load(&p[k * 16 + e0]));
    }
    NttCore<AR, A>::template fwd_contig<true>(v, lrow, e0, r, ti, tf, N, m);
    exchange_cb_to_cp<AR>(v, lrow, e0);
    u64 c[16], res[16];
    load_row_cp<true>(a.cq + ((size_t)inst * a.cq_L + i) * N + row_off, e0, c);
#pragma unroll
    for (int k = 0; k < 16; k++) {
        if constexpr (AR::is_fp) {
            const FpAr::Mod fm = FpAr::mod(pc);
            res[k] = FpAr::canon(FpAr::mulmod_lazy(u64_to_f64(c[k]) - v[k], pinv.d, fm), fm);
        } else {
            res[k] = mul_shoup(submod(c[k], AR::canon_fwd(v[k], m), q), pinv.w, pinv.wp, q);
        }
    }
    store_row_cp(a.out + ((size_t)inst * L + i) * N + row_off, e0, res);
}

template <class AR, int A, int MODE>
__global__ __launch_bounds__(256, MODE >= FIN_HOISTED ? (AR::is_fp ? 3 : 2) : 4) void ks_final_kernel(FinalArgs a, Tables tb, LimbRun run) {
    __shared__ u64 lds[NTT_LDS_WORDS];
    constexpr u32 TILES = (1u << A) / 16;
    u32 group, inst;
    if (!xcd_decode(blockIdx.x, a.n_inst, run.count * TILES, group, inst)) return;
    ks_final_body<AR, A, MODE>(a, tb, lds, run.first + group / TILES, group % TILES, inst);
}
// MODE 0 with ordinary loads of the converted part.  A kernel of its own: of two loads behind a condition, one of them nontemporal, the compiler
// makes a single ordinary one, and the conversion of the next call writes more slowly over lines that such loads have left in the
// caches (rescale of ten ciphertexts, 13 limbs, N = 2^14: conversion 10.9 -> 14.0 us)
template <class AR, int A>
__global__ __launch_bounds__(256, 4) void ks_final_cached_kernel(FinalArgs a, Tables tb, LimbRun run) {
    __shared__ u64 lds[NTT_LDS_WORDS];
    constexpr u32 TILES = (1u << A) / 16;
    u32 group, inst;
    if (!xcd_decode(blockIdx.x, a.n_inst, run.count * TILES, group, inst)) return;
    ks_final_body<AR, A, FIN_KS, true>(a, tb, lds, run.first + group / TILES, group % TILES, inst);
}

// ================================================== stand-alone coefficient-form base conversions
// in [b][L][N] coeff -> out [b][dnum][D][N].  grid (N/256, dnum, batch).
template <int ALPHA>
__global__ __launch_bounds__(256) void modup_kernel(const u64* __restrict__ in, u64* __restrict__ out, Tables tb) {
    const u32 N = 1u << tb.logN, L = tb.L, D = tb.D;
    const u32 n = blockIdx.x * 256 + threadIdx.x, j = blockIdx.y, b = blockIdx.z;
    const u64* src = in + ((size_t)b * L + (size_t)j * ALPHA) * N + n;
    u64* dst = out + ((size_t)b * tb.dnum + j) * D * N + n;
    const u32 ns = (j + 1) * ALPHA <= L ? ALPHA : L - j * ALPHA;  // the last digit may be shorter
    u64 y[ALPHA];
#pragma unroll
    for (int ii = 0; ii < ALPHA; ii++) {
        y[ii] = 0;
        if ((u32)ii < ns) {
            const u32 i = j * ALPHA + ii;
            const u64 x = src[(size_t)ii * N];
            dst[(size_t)i * N] = x;
            y[ii] = mul_shoup(x, tb.up_hatinv[2 * i], tb.up_hatinv[2 * i + 1], tb.pc[i].q);
        }
    }
    const u64* chat = tb.up_chat + (size_t)j * ALPHA * D;
    for (u32 t = 0; t < D; t++) {
        if (t >= j * ALPHA && t < j * ALPHA + ns) continue;
        u128w acc = {0, 0};
        const PrimeConst pc = tb.pc[t];
#pragma unroll
        for (int ii = 0; ii < ALPHA; ii++) {
            if ((u32)ii < ns) mac128(acc, y[ii], chat[(size_t)ii * D + t]);
            if (ALPHA > 8 && ((ii & 7) == 7 || ii + 1 == ALPHA)) acc.hi = csub(acc.hi, pc.q);  // keeps acc < q * 2^64
        }
        dst[(size_t)t * N] = redc(acc, pc.q, pc.qneg);
    }
}

// in [g][D][N] coeff -> out [g][L][N] = (in_i - conv_i) * P^-1.  grid (N/256, groups).
template <int KK>
__global__ __launch_bounds__(256) void moddown_kernel(const u64* __restrict__ in, u64* __restrict__ out, Tables tb) {
    const u32 N = 1u << tb.logN, L = tb.L, D = tb.D;
    const u32 n = blockIdx.x * 256 + threadIdx.x, g = blockIdx.y;
    const u64* src = in + (size_t)g * D * N + n;
    u64* dst = out + (size_t)g * L * N + n;
    u64 y[KK];
#pragma unroll
    for (int k = 0; k < KK; k++)
        y[k] = mul_shoup(src[(size_t)(L + k) * N], tb.dn_hatinv[2 * k], tb.dn_hatinv[2 * k + 1], tb.pc[L + k].q);
    for (u32 i = 0; i < L; i++) {
        u128w acc = {0, 0};
        const PrimeConst pc = tb.pc[i];
#pragma unroll
        for (int k = 0; k < KK; k++) {
            mac128(acc, y[k], tb.dn_chat[(size_t)k * L + i]);
            if (KK > 8 && ((k & 7) == 7 || k + 1 == KK)) acc.hi = csub(acc.hi, pc.q);  // keeps acc < q * 2^64
        }
        const u64 conv = redc(acc, pc.q, pc.qneg);
        const PinvConst pi = tb.pinv[i];
        dst[(size_t)i * N] = mul_shoup(submod(src[(size_t)i * N], conv, pc.q), pi.w, pi.wp, pc.q);
    }
}

// ------------------------------------------------------------------------ automorphism
__global__ __launch_bounds__(256) void automorph_eval_kernel(const u64* __restrict__ in, u64* __restrict__ out, u32 logN,
                                                             u32 n_limbs, u32 galois) {
    const u32 N = 1u << logN;
    const u32 n = blockIdx.x * 256 + threadIdx.x;
    const size_t limb = ((size_t)blockIdx.z * n_limbs + blockIdx.y) * N;
    out[limb + n] = in[limb + eval_perm(n, galois, logN)];
}

// coefficient form, as a gather: out[u] = +-in[t] with t*g = u (mod 2N) or t*g = u + N (mod 2N)
__global__ __launch_bounds__(256) void automorph_coeff_kernel(const u64* __restrict__ in, u64* __restrict__ out,
                                                              const PrimeConst* pcs, u32 logN, u32 n_limbs,
                                                              u32 prime_first, u32 galois_inv) {
    const u32 N = 1u << logN;
    const u32 u = blockIdx.x * 256 + threadIdx.x;
    const size_t limb = ((size_t)blockIdx.z * n_limbs + blockIdx.y) * N;
    const u64 q = pcs[prime_first + blockIdx.y].q;
    const u32 tp = (u * galois_inv) & (2 * N - 1);
    u64 v;
    if (tp < N) {
        v = in[limb + tp];
    } else {
        v = in[limb + tp - N];
        v = v ? q - v : 0;
    }
    out[limb + u] = v;
}

// -------------------------------------------------------------------- limb-wise arithmetic
// out[g][l][n] = a[g][l][n] (op) b[g % b_period][l][n] mod prime (prime_first + l); two words per lane
// (16-byte accesses).  out may be a or b themselves: every lane reads its words before it writes them.
enum PointwiseOp { PW_ADD = 0, PW_SUB = 1, PW_MUL = 2, PW_MAC = 3 };
template <int OP>
__global__ __launch_bounds__(256) void pointwise_kernel(const u64* a, const u64* b, u64* out, const PrimeConst* pcs,
                                                        u32 logN, u32 n_limbs, u32 prime_first, u32 b_period) {
    const u32 N = 1u << logN;
    const u32 n = (blockIdx.x * 256 + threadIdx.x) * 2;
    const size_t la = ((size_t)blockIdx.z * n_limbs + blockIdx.y) * N + n;
    const size_t lb = ((size_t)(blockIdx.z % b_period) * n_limbs + blockIdx.y) * N + n;
    const PrimeConst pc = pcs[prime_first + blockIdx.y];
    const ulonglong2 av = *reinterpret_cast<const ulonglong2*>(a + la);
    const ulonglong2 bv = *reinterpret_cast<const ulonglong2*>(b + lb);
    ulonglong2 r;
    if (OP == PW_ADD) {
        r.x = addmod(av.x, bv.x, pc.q), r.y = addmod(av.y, bv.y, pc.q);
    } else if (OP == PW_SUB) {
        r.x = submod(av.x, bv.x, pc.q), r.y = submod(av.y, bv.y, pc.q);
    } else {
        r.x = mulmod_var(av.x, bv.x, pc.q, pc.qneg, pc.r2), r.y = mulmod_var(av.y, bv.y, pc.q, pc.qneg, pc.r2);
        if (OP == PW_MAC) {
            const ulonglong2 ov = *reinterpret_cast<const ulonglong2*>(out + la);
            r.x = addmod(r.x, ov.x, pc.q), r.y = addmod(r.y, ov.y, pc.q);
        }
    }
    *reinterpret_cast<ulonglong2*>(out + la) = r;
}
