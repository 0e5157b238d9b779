// Host side of the C ABI declared in include/ckks_mi355x.h: context creation (table
// generation on the host, one upload), argument validation, workspace carving and kernel
// launches.  No device memory is allocated here.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <string>
#include <vector>

#include "../../include/ckks_mi355x.h"
#include "kernels.h"

typedef unsigned __int128 u128;
static_assert(CKKS_ROT_CHUNK == CKKS_ROTATIONS_PER_LAUNCH, "the public constant must match the kernels' argument arrays");

// ------------------------------------------------------------------ host modular helpers
static inline u64 h_mulmod(u64 a, u64 b, u64 m) { return (u64)(((u128)a * b) % m); }
static u64 h_powmod(u64 b, u64 e, u64 m) {
    u64 r = 1 % m;
    b %= m;
    while (e) {
        if (e & 1) r = h_mulmod(r, b, m);
        b = h_mulmod(b, b, m);
        e >>= 1;
    }
    return r;
}
static inline u64 h_invmod(u64 a, u64 m) { return h_powmod(a % m, m - 2, m); }
static inline u64 h_shoup(u64 w, u64 m) { return (u64)(((u128)w << 64) / m); }
static inline u64 h_mont(u64 w, u64 m) { return (u64)(((u128)w << 64) % m); }
static u64 h_neg_inv64(u64 q) {  // -q^-1 mod 2^64 by Newton iteration
    u64 x = q;                    // correct to 3 bits (q odd)
    for (int i = 0; i < 6; i++) x *= 2 - q * x;
    return (u64)0 - x;
}
static u32 h_bitrev(u32 x, u32 bits) {
    u32 r = 0;
    for (u32 i = 0; i < bits; i++) r |= ((x >> i) & 1u) << (bits - 1 - i);
    return r;
}
static bool h_is_prime(u64 n) {
    if (n < 2) return false;
    static const u64 bases[] = {2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37};
    for (u64 p : bases) {
        if (n % p == 0) return n == p;
    }
    u64 d = n - 1;
    int r = 0;
    while ((d & 1) == 0) {
        d >>= 1;
        r++;
    }
    for (u64 a : bases) {
        u64 x = h_powmod(a, d, n);
        if (x == 1 || x == n - 1) continue;
        bool comp = true;
        for (int i = 1; i < r; i++) {
            x = h_mulmod(x, x, n);
            if (x == n - 1) {
                comp = false;
                break;
            }
        }
        if (comp) return false;
    }
    return true;
}
// smallest primitive 2N-th root of unity: minimum over the odd powers of any one of them
static u64 h_min_root(u64 m, u32 logN) {
    const u64 N = 1ull << logN;
    u64 root = 0;
    for (u64 x = 2; x < m && !root; x++) {
        u64 y = h_powmod(x, (m - 1) / (2 * N), m);
        if (h_powmod(y, N, m) == m - 1) root = y;
    }
    u64 sq = h_mulmod(root, root, m), cur = root, best = root;
    for (u64 k = 1; k < N; k++) {
        cur = h_mulmod(cur, sq, m);
        if (cur < best) best = cur;
    }
    return best;
}

static inline u32 u8_of(u64 z, u32 k) { return (u32)(z >> (8 * k)) & 0xffu; }

// ------------------------------------------------------------------------------ context
static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// The caller's table buffer holds one block shared by every level (per-prime twiddles and
// constants over the whole chain), one block of conversion constants per level ell = 1..L (basis
// q_0..q_{ell-1}, p_0..p_{K-1}) and one small block per rescale step ell -> ell-1 (ell = 2..L).
struct SharedLayout {
    size_t tw_int, tw_fp, pc, sc_plain, sc_dn, dn_hatinv, up_aop, dn_aop, end;
};
struct LevelLayout {
    size_t sc_up, up_hatinv, up_chat, dn_chat, pinv, pmod, up_aop, end;
};

// Conversion from `sources` limbs on the matrix cores: products per coefficient group (few values, so that few kernels are
// built; 5 = the merged rescale of a 16-prime special basis).  Two sources are enough for it to pay: a batch of 8 rotations
// at N = 2^16, L = 12 with digits of two / three limbs takes 409 / 366 us, with direct multiply-accumulates 427 / 393 us.
static inline u32 mfma_ks(u32 sources) { return sources < 2 ? 0 : sources <= 4 ? 1 : sources <= 8 ? 2 : sources <= 16 ? 4 : 5; }
static inline size_t aop_words(u32 ks) { return (size_t)ks * 32; }  // constant operands of one (digit, target)
struct RescaleLayout {
    size_t sc_dn, pinv, end;
};

struct Taker {
    size_t o;
    size_t take(size_t bytes) {
        size_t at = o;
        o += align256(bytes);
        return at;
    }
};

static SharedLayout shared_layout(u32 logN, u32 L, u32 K, u32 alpha) {
    const size_t N = (size_t)1 << logN, D = L + K, K1 = K ? K : 1;
    Taker t{0};
    SharedLayout l;
    l.tw_int = t.take(D * 4 * N * sizeof(u64));
    l.tw_fp = t.take(D * 2 * N * sizeof(double));
    l.pc = t.take(D * sizeof(PrimeConst));
    l.sc_plain = t.take(D * sizeof(InvScale));
    l.sc_dn = t.take(K1 * sizeof(InvScale));
    l.dn_hatinv = t.take(K1 * 2 * sizeof(u64));
    l.up_aop = t.take((K ? (size_t)(L / alpha) : 0) * D * aop_words(mfma_ks(alpha)) * sizeof(u64));
    l.dn_aop = t.take(L * aop_words(mfma_ks(K)) * sizeof(u64));
    l.end = t.o;
    return l;
}

static LevelLayout level_layout(size_t base, u32 ell, u32 K, u32 alpha) {
    const size_t D = ell + K, K1 = K ? K : 1;
    Taker t{base};
    LevelLayout l;
    l.sc_up = t.take(ell * sizeof(InvScale));
    l.up_hatinv = t.take(ell * 2 * sizeof(u64));
    l.up_chat = t.take(ell * D * sizeof(u64));
    l.dn_chat = t.take(K1 * ell * sizeof(u64));
    l.pinv = t.take(ell * sizeof(PinvConst));
    l.pmod = t.take(ell * sizeof(u64));
    l.up_aop = t.take((K && ell % alpha ? D : 0) * aop_words(mfma_ks(alpha)) * sizeof(u64));  // a shorter last digit
    l.end = t.o;
    return l;
}

// rescale from ell limbs to ell - 1: one source prime (q_{ell-1}), targets q_0..q_{ell-2}
static RescaleLayout rescale_layout(size_t base, u32 ell) {
    const size_t T = ell - 1;
    Taker t{base};
    RescaleLayout l;
    l.sc_dn = t.take(sizeof(InvScale));
    l.pinv = t.take(T * sizeof(PinvConst));
    l.end = t.o;
    return l;
}

// ModDown merged with the rescale after it, from level ell: sources q_{ell-1}, p_0..p_{K-1}; targets q_0..q_{ell-2}
struct MergedLayout {
    size_t sc_dn, pinv, dn_aop, end;
};
static MergedLayout merged_layout(size_t base, u32 ell, u32 K) {
    const size_t T = ell - 1, S = K + 1;
    Taker t{base};
    MergedLayout l;
    l.sc_dn = t.take(S * sizeof(InvScale));
    l.pinv = t.take(T * sizeof(PinvConst));
    l.dn_aop = t.take(T * aop_words(mfma_ks((u32)S)) * sizeof(u64));
    l.end = t.o;
    return l;
}

static size_t table_total(u32 logN, u32 L, u32 K, u32 dnum) {
    const u32 alpha = (L + dnum - 1) / dnum;
    size_t o = shared_layout(logN, L, K, alpha).end;
    for (u32 ell = 1; ell <= L; ell++) o = level_layout(o, ell, K, alpha).end;
    for (u32 ell = 2; ell <= L; ell++) o = rescale_layout(o, ell).end;
    if (K)
        for (u32 ell = 2; ell <= L; ell++) o = merged_layout(o, ell, K).end;
    return o;
}

// per-kernel timing: when enabled, every launch is bracketed by two HIP events recorded on the
// launch stream; ckks_profile_read waits for them and sums elapsed time per kernel instantiation
// (named as the profiler names it, e.g. "fwd_strided_kernel<FpAr, 8, 1>").
struct ProfRec {
    int kind;
    hipEvent_t a, b;
};
struct ProfKindStat {
    std::string name;
    double ms = 0;
    u64 launches = 0, bytes = 0;
};
struct ProfState {
    bool on = false;
    std::vector<ProfRec> pending;
    std::vector<hipEvent_t> pool;
    std::vector<ProfKindStat> kinds;
    int kind_of(const std::string& name) {
        for (size_t i = 0; i < kinds.size(); i++)
            if (kinds[i].name == name) return (int)i;
        kinds.emplace_back();
        kinds.back().name = name;
        return (int)kinds.size() - 1;
    }
};

// Overlap of the two arithmetic classes: between fork() and join() the launches on IntAr limbs
// (integer-VALU bound) go to a side stream and run concurrently with the launches on FpAr limbs
// (memory bound) of the caller's stream.  Ordering is by events only; both streams have default priority.
struct SideStream {
    bool enabled = false;  // off by default; ckks_set_overlap switches it
    bool active = false;
    bool fp_pending = false;  // an FpAr conversion is running on the side stream (see decompose_extend)
    hipStream_t stream = nullptr;
    std::vector<hipEvent_t> events;
    size_t next = 0;
};

struct Shared {
    std::string err;
    ProfState prof;
    SideStream side;
};

// Constant operands of the matrix-core conversions of one direction (device pointers; ConvArgs states the layout)
struct ConvTab {
    const u64* aop = nullptr;
    const u64* aop_part = nullptr;
    u32 n_full = 0;
    u32 ks = 0;  // products per coefficient group; 0 = few sources, converted directly
    u32 sources = 0;
    // a lane half loads one word fewer than the products take
    bool fewer() const { return ks && ks <= 2 && (sources + 1) / 2 < 2 * ks; }
};

// One level of the context: everything a launch needs.  `primes` is the level's basis in limb order.
struct View {
    u32 logN = 0, L = 0, K = 0, dnum = 0, alpha = 0, D = 0;
    std::vector<u64> primes;
    Tables tb;
    bool mixed_classes = false;  // both FpAr and IntAr primes present
    ConvTab up, dn;              // conversions of ModUp and ModDown
    Shared* sh = nullptr;
};

// Scratch memory of ckks_rescale_static, the entry point for callers that cannot allocate or bring a
// workspace: one array per GPU, held from the moment the code object is loaded on that GPU until the process
// ends.  In host code the name `scratch` is only a handle for hipGetSymbolAddress: the address a kernel may
// use is looked up once per device (at context creation, with that device current) and kept in the context.
static __device__ __align__(256) unsigned char scratch[CKKS_STATIC_SCRATCH_BYTES];

struct ckks_ctx {
    int device = -1;               // the device that was current at creation: tables and scratch live there
    void* scratch_ptr = nullptr;   // device address of `scratch` on that device
    u32 logN, L, K, dnum, alpha, D;
    std::vector<u64> primes, psi;
    std::vector<View> level;    // [ell], 1 <= ell <= L: key switching at ell active q-limbs; level[L] is the full one
    std::vector<View> rescale;  // [ell], 2 <= ell <= L: the step from ell limbs to ell - 1 (K = 1, "special" prime q_{ell-1})
    std::vector<View> merged;   // [ell], 2 <= ell <= L, K > 0: ModDown from level ell that also divides by q_{ell-1}
    mutable Shared sh;
    const View* full() const { return &level[L]; }
};

static hipEvent_t side_event(SideStream& sd) {
    if (sd.events.size() < 16) {
        hipEvent_t e = nullptr;
        if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) return nullptr;
        sd.events.push_back(e);
        return e;
    }
    return sd.events[sd.next++ % sd.events.size()];
}

static bool side_stream_ready(SideStream& sd) {
    if (!sd.stream && hipStreamCreateWithFlags(&sd.stream, hipStreamNonBlocking) != hipSuccess) {
        sd.stream = nullptr;
        sd.enabled = false;
        (void)hipGetLastError();
        return false;
    }
    return true;
}

// From here on IntAr launches go to the side stream, ordered after everything enqueued on s so far.
static void fork_side(const View* c, hipStream_t s) {
    SideStream& sd = c->sh->side;
    if (!sd.enabled || !c->mixed_classes || sd.active) return;
    if (!side_stream_ready(sd)) return;
    hipEvent_t e = side_event(sd);
    if (!e || hipEventRecord(e, s) != hipSuccess || hipStreamWaitEvent(sd.stream, e, 0) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    sd.active = true;
}

// s waits for everything the side stream was given; IntAr launches return to s.
static void join_side(const View* c, hipStream_t s) {
    SideStream& sd = c->sh->side;
    if (!sd.active) return;
    sd.active = false;
    hipEvent_t e = side_event(sd);
    if (!e || hipEventRecord(e, sd.stream) != hipSuccess || hipStreamWaitEvent(s, e, 0) != hipSuccess) {
        // cannot order by event: fall back to a full wait so that correctness never depends on it
        (void)hipGetLastError();
        (void)hipStreamSynchronize(sd.stream);
    }
}

static hipEvent_t prof_event(ProfState& p) {
    if (!p.pool.empty()) {
        hipEvent_t e = p.pool.back();
        p.pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

struct ProfScope {
    ProfState* p = nullptr;
    hipStream_t s;
    ProfRec rec;
    // alg_limbs: limbs (N words each) the launch must read plus write once
    ProfScope(const View* c, const std::string& name, u64 alg_limbs, hipStream_t stream) : s(stream) {
        if (!c->sh->prof.on) return;
        p = &c->sh->prof;
        rec.kind = p->kind_of(name);
        p->kinds[rec.kind].launches++;
        p->kinds[rec.kind].bytes += (alg_limbs * sizeof(u64)) << c->logN;
        rec.a = prof_event(*p);
        rec.b = prof_event(*p);
        if (!rec.a || !rec.b) {
            p = nullptr;
            return;
        }
        (void)hipEventRecord(rec.a, s);
    }
    ~ProfScope() {
        if (!p) return;
        (void)hipEventRecord(rec.b, s);
        p->pending.push_back(rec);
    }
};

static void prof_drain(ProfState& p) {
    for (ProfRec& r : p.pending) {
        float ms = 0.f;
        if (hipEventSynchronize(r.b) == hipSuccess && hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess) p.kinds[r.kind].ms += ms;
        p.pool.push_back(r.a);
        p.pool.push_back(r.b);
    }
    p.pending.clear();
}

static int fail(const ckks_ctx* c, int code, const char* msg) {
    if (c) c->sh.err = msg;
    return code;
}
static int fail(const View* c, int code, const char* msg) {
    if (c) c->sh->err = msg;
    return code;
}

static int check_shape(u32 logN, u32 L, u32 K, u32 dnum) {
    if (logN < CKKS_MIN_LOGN || logN > CKKS_MAX_LOGN) return CKKS_EUNSUPPORTED;
    if (L == 0 || dnum == 0) return CKKS_EINVAL;
    if (L + K > CKKS_MAX_PRIMES) return CKKS_EUNSUPPORTED;
    if (dnum > L) return CKKS_EINVAL;
    const u32 alpha = (L + dnum - 1) / dnum;  // limbs per digit; the last digit is shorter if dnum does not divide L
    if ((L + alpha - 1) / alpha != dnum) return CKKS_EUNSUPPORTED;  // dnum is not the digit count this size gives
    if (K > CKKS_MAX_DIGIT) return CKKS_EUNSUPPORTED;
    if (K > 0 && alpha > CKKS_MAX_DIGIT) return CKKS_EUNSUPPORTED;
    return CKKS_OK;
}

extern "C" int ckks_table_bytes(uint32_t logN, uint32_t L, uint32_t K, uint32_t dnum, size_t* bytes) {
    if (!bytes) return CKKS_EINVAL;
    int rc = check_shape(logN, L, K, dnum);
    if (rc) return rc;
    *bytes = table_total(logN, L, K, dnum);
    return CKKS_OK;
}

static InvScale make_scale(u64 factor, u64 ninv, u64 wlast, u64 m, bool fp) {
    InvScale s;
    s.sx = h_mulmod(ninv, factor, m);
    s.sx_p = h_shoup(s.sx, m);
    s.sy = h_mulmod(h_mulmod(wlast, ninv, m), factor, m);
    s.sy_p = h_shoup(s.sy, m);
    s.sxd = fp ? (double)s.sx : 0.0;
    s.syd = fp ? (double)s.sy : 0.0;
    return s;
}

// (prod of src[k], k != skip) mod m
static u64 prod_except(const std::vector<u64>& src, size_t skip, u64 m) {
    u64 r = 1 % m;
    for (size_t k = 0; k < src.size(); k++)
        if (k != skip) r = h_mulmod(r, src[k] % m, m);
    return r;
}

// Constant operands of the matrix-core conversion onto one target prime m (conv_mfma_body states the layout): source
// i < ns has the constant hat[i] mod m.  aop: aop_words(ks) zeroed words.
static void build_aop(u64* aop, const std::vector<u64>& hat, u64 m) {
    for (u32 i = 0; i < hat.size(); i++) {
        u64 c = hat[i] % m;
        // source i travels in product i / 4, lane half i % 2, word (i / 2) % 2; digit row dg: byte bb = digit dg of
        // hat * 256^bb
        u64* rows = aop + (size_t)(i / 4) * 32 + i % 2 * 16 + (i / 2) % 2;
        for (u32 bb = 0; bb < 8; bb++) {
            const int64_t centred = c > m / 2 ? (int64_t)c - (int64_t)m : (int64_t)c;
            const u64 z = (u64)centred + CKKS_DIGIT_BIAS;
            for (u32 dg = 0; dg < 8; dg++) rows[2 * dg] |= (u64)(u8_of(z, dg) ^ 0x80u) << (8 * bb);
            c = h_mulmod(c, 256 % m, m);
        }
    }
}
// prod of src[k], k != i, mod m, for every i
static std::vector<u64> hats(const std::vector<u64>& src, u64 m) {
    std::vector<u64> h(src.size());
    for (size_t i = 0; i < src.size(); i++) h[i] = prod_except(src, i, m);
    return h;
}

extern "C" int ckks_ctx_create(ckks_ctx** out, uint32_t logN, uint32_t L, uint32_t K, uint32_t dnum,
                               const uint64_t* h_primes, const uint64_t* h_psi, void* d_tables, size_t table_bytes,
                               void* stream) {
    if (!out) return CKKS_EINVAL;
    *out = nullptr;
    if (!h_primes || !d_tables) return CKKS_EINVAL;
    int rc = check_shape(logN, L, K, dnum);
    if (rc) return rc;
    if (((uintptr_t)d_tables) & 255) return CKKS_EINVAL;
    const size_t total = table_total(logN, L, K, dnum);
    if (table_bytes < total) return CKKS_ENOMEM;
    const u32 D = L + K, alpha = (L + dnum - 1) / dnum;
    const SharedLayout lay = shared_layout(logN, L, K, alpha);
    const size_t N = (size_t)1 << logN;
    for (u32 i = 0; i < D; i++) {
        const u64 m = h_primes[i];
        if (m >> CKKS_MAX_PRIME_BITS) return CKKS_EUNSUPPORTED;
        if (m < 2 * N || (m - 1) % (2 * N) != 0) return CKKS_EINVAL;
        if (!h_is_prime(m)) return CKKS_EINVAL;
        for (u32 k = 0; k < i; k++)
            if (h_primes[k] == m) return CKKS_EINVAL;
        if (h_psi && h_powmod(h_psi[i], N, m) != m - 1) return CKKS_EINVAL;
    }

    ckks_ctx* c = new ckks_ctx();
    c->logN = logN, c->L = L, c->K = K, c->dnum = dnum, c->alpha = alpha, c->D = D;
    c->primes.assign(h_primes, h_primes + D);
    c->psi.resize(D);
    const std::vector<u64> specials(c->primes.begin() + L, c->primes.end());

    std::vector<unsigned char> host(total, 0);
    unsigned char* hb = host.data();
    unsigned char* dbase = (unsigned char*)d_tables;
    // ---- block shared by every level
    u64* tw = (u64*)(hb + lay.tw_int);
    double* twf = (double*)(hb + lay.tw_fp);
    PrimeConst* pc = (PrimeConst*)(hb + lay.pc);
    InvScale* sc_plain = (InvScale*)(hb + lay.sc_plain);
    InvScale* sc_dn = (InvScale*)(hb + lay.sc_dn);
    u64* dn_hatinv = (u64*)(hb + lay.dn_hatinv);
    std::vector<u64> pw(N), ninv(D), wlast(D);
    for (u32 i = 0; i < D; i++) {
        const u64 m = c->primes[i];
        const bool fp = m < CKKS_FP_PRIME_LIMIT;
        const u64 psi = h_psi ? h_psi[i] : h_min_root(m, logN);
        c->psi[i] = psi;
        const u64 psi_inv = h_invmod(psi, m);
        u64* fw = tw + (size_t)i * 4 * N;
        double* ff = twf + (size_t)i * 2 * N;
        for (int dir = 0; dir < 2; dir++) {
            const u64 base = dir ? psi_inv : psi;
            pw[0] = 1;
            for (size_t e = 1; e < N; e++) pw[e] = h_mulmod(pw[e - 1], base, m);
            u64* w = fw + (size_t)dir * 2 * N;
            for (size_t k = 0; k < N; k++) {
                w[k] = pw[h_bitrev((u32)k, logN)];
                w[N + k] = h_shoup(w[k], m);
                if (fp) ff[(size_t)dir * N + k] = (double)w[k];
            }
        }
        PrimeConst& p = pc[i];
        p.q = m;
        p.qneg = h_neg_inv64(m);
        p.r1 = (u64)(((u128)1 << 64) % m);
        p.r1_p = h_shoup(p.r1, m);
        p.r2 = h_mulmod(p.r1, p.r1, m);
        p.qd = (double)m;  // exact for FpAr primes
        p.qinv = 1.0 / (double)m;
        p.fp = fp ? 1 : 0;
        p.narrow = fp && m <= CKKS_FP_NARROW_MAX ? 1 : 0;
        ninv[i] = h_invmod(N % m, m);
        wlast[i] = fw[2 * N + 1];
        sc_plain[i] = make_scale(1, ninv[i], wlast[i], m, fp);
    }
    for (u32 k = 0; k < K; k++) {  // sources of ModDown: the special limbs, the same at every level
        const u64 pk = specials[k];
        const u64 hinv = h_invmod(prod_except(specials, k, pk), pk);
        dn_hatinv[2 * k] = hinv;
        dn_hatinv[2 * k + 1] = h_shoup(hinv, pk);
        sc_dn[k] = make_scale(hinv, ninv[L + k], wlast[L + k], pk, pc[L + k].fp != 0);
    }
    auto shared_tables = [&](Tables& tb) {
        tb.tw_int = (const u64*)(dbase + lay.tw_int);
        tb.tw_fp = (const double*)(dbase + lay.tw_fp);
        tb.pc = (const PrimeConst*)(dbase + lay.pc);
        tb.sc_plain = (const InvScale*)(dbase + lay.sc_plain);
        tb.sc_dn = (const InvScale*)(dbase + lay.sc_dn);
        tb.dn_hatinv = (const u64*)(dbase + lay.dn_hatinv);
        tb.logN = logN;
    };
    auto classes_mixed = [](const std::vector<u64>& pr) {
        bool any_fp = false, any_int = false;
        for (u64 m : pr) (m < CKKS_FP_PRIME_LIMIT ? any_fp : any_int) = true;
        return any_fp && any_int;
    };

    // constant operands of the matrix-core conversions that every level shares: full digits, and ModDown by P
    const u32 up_ks = K ? mfma_ks(alpha) : 0, dn_ks = mfma_ks(K);
    for (u32 j = 0; up_ks && j < L / alpha; j++) {
        const std::vector<u64> digit(c->primes.begin() + j * alpha, c->primes.begin() + (j + 1) * alpha);
        for (u32 t = 0; t < D; t++)
            if (t / alpha != j || t >= L)
                build_aop((u64*)(hb + lay.up_aop) + ((size_t)j * D + t) * aop_words(up_ks), hats(digit, c->primes[t]), c->primes[t]);
    }
    for (u32 t = 0; dn_ks && t < L; t++)
        build_aop((u64*)(hb + lay.dn_aop) + t * aop_words(dn_ks), hats(specials, c->primes[t]), c->primes[t]);

    // ---- one block per level: limb index i of the level is prime ph(i) of the chain
    size_t off = lay.end;
    c->level.resize(L + 1);
    for (u32 ell = 1; ell <= L; ell++) {
        const LevelLayout ll = level_layout(off, ell, K, alpha);
        off = ll.end;
        const u32 Dl = ell + K, beta = (ell + alpha - 1) / alpha;
        auto ph = [&](u32 i) { return i < ell ? i : L + (i - ell); };
        InvScale* sc_up = (InvScale*)(hb + ll.sc_up);
        u64* up_hatinv = (u64*)(hb + ll.up_hatinv);
        u64* up_chat = (u64*)(hb + ll.up_chat);
        u64* dn_chat = (u64*)(hb + ll.dn_chat);
        PinvConst* pinv = (PinvConst*)(hb + ll.pinv);
        u64* pmod = (u64*)(hb + ll.pmod);
        for (u32 j = 0; j < beta; j++) {  // ModUp constants of digit j = limbs [lo, hi)
            const u32 lo = j * alpha, hi = (j + 1) * alpha < ell ? (j + 1) * alpha : ell;
            const std::vector<u64> digit(c->primes.begin() + lo, c->primes.begin() + hi);
            for (u32 i = lo; i < hi; i++) {
                const u64 qi = c->primes[i];
                const u64 hinv = h_invmod(prod_except(digit, i - lo, qi), qi);
                up_hatinv[2 * i] = hinv;
                up_hatinv[2 * i + 1] = h_shoup(hinv, qi);
                sc_up[i] = make_scale(hinv, ninv[i], wlast[i], qi, pc[i].fp != 0);
                for (u32 t = 0; t < Dl; t++) {
                    if (t >= lo && t < hi) continue;
                    const u64 mt = c->primes[ph(t)];
                    const u64 hatb = prod_except(digit, i - lo, mt);
                    up_chat[(size_t)i * Dl + t] = h_mont(hatb, mt);
                }
            }
        }
        for (u32 i = 0; i < ell; i++) {  // ModDown constants of target q_i
            const u64 qi = c->primes[i];
            for (u32 k = 0; k < K; k++) {
                const u64 hatb = prod_except(specials, k, qi);
                dn_chat[(size_t)k * ell + i] = h_mont(hatb, qi);
            }
            pmod[i] = prod_except(specials, specials.size(), qi);
            const u64 pi = h_invmod(pmod[i], qi);
            pinv[i] = PinvConst{pi, h_shoup(pi, qi), (double)pi};
        }
        View& v = c->level[ell];
        v.logN = logN, v.L = ell, v.K = K, v.dnum = beta, v.alpha = alpha, v.D = Dl, v.sh = &c->sh;
        v.primes.resize(Dl);
        for (u32 i = 0; i < Dl; i++) v.primes[i] = c->primes[ph(i)];
        v.mixed_classes = classes_mixed(v.primes);
        Tables& tb = v.tb;
        shared_tables(tb);
        tb.sc_up = (const InvScale*)(dbase + ll.sc_up);
        tb.up_hatinv = (const u64*)(dbase + ll.up_hatinv);
        tb.up_chat = (const u64*)(dbase + ll.up_chat);
        tb.dn_chat = (const u64*)(dbase + ll.dn_chat);
        tb.pinv = (const PinvConst*)(dbase + ll.pinv);
        tb.pmod = (const u64*)(dbase + ll.pmod);
        tb.L = ell, tb.K = K, tb.dnum = beta, tb.alpha = alpha, tb.D = Dl, tb.Lfull = L, tb.Kfull = K, tb.Lq = ell;
        v.up = ConvTab{(const u64*)(dbase + lay.up_aop), (const u64*)(dbase + ll.up_aop), ell / alpha, up_ks, alpha};
        v.dn = ConvTab{(const u64*)(dbase + lay.dn_aop), nullptr, 1, dn_ks, K};
        if (up_ks && ell % alpha) {  // the last digit of this level is shorter than the chain's
            const std::vector<u64> digit(c->primes.begin() + ell / alpha * alpha, c->primes.begin() + ell);
            for (u32 t = 0; t < Dl; t++)
                if (t < ell / alpha * alpha || t >= ell)
                    build_aop((u64*)(hb + ll.up_aop) + t * aop_words(up_ks), hats(digit, v.primes[t]), v.primes[t]);
        }
    }
    // ---- one block per rescale step: a ModDown whose only "special" prime is q_{ell-1}
    c->rescale.resize(L + 1);
    for (u32 ell = 2; ell <= L; ell++) {
        const RescaleLayout rl = rescale_layout(off, ell);
        off = rl.end;
        const u32 T = ell - 1;
        const u64 ql = c->primes[T];
        InvScale* rsc = (InvScale*)(hb + rl.sc_dn);
        PinvConst* pinv = (PinvConst*)(hb + rl.pinv);
        rsc[0] = make_scale(1, ninv[T], wlast[T], ql, pc[T].fp != 0);
        for (u32 i = 0; i < T; i++) {
            const u64 qi = c->primes[i];
            const u64 pi = h_invmod(ql % qi, qi);
            pinv[i] = PinvConst{pi, h_shoup(pi, qi), (double)pi};
        }
        View& v = c->rescale[ell];
        v.logN = logN, v.L = T, v.K = 1, v.dnum = 1, v.alpha = T, v.D = ell, v.sh = &c->sh;
        v.primes.assign(c->primes.begin(), c->primes.begin() + ell);
        v.mixed_classes = classes_mixed(v.primes);
        Tables& tb = v.tb;
        memset(&tb, 0, sizeof(tb));
        shared_tables(tb);
        tb.sc_dn = (const InvScale*)(dbase + rl.sc_dn);
        tb.dn_hatinv = nullptr;
        tb.pinv = (const PinvConst*)(dbase + rl.pinv);
        tb.L = T, tb.K = 1, tb.dnum = 1, tb.alpha = T, tb.D = ell, tb.Lfull = ell, tb.Kfull = 0, tb.Lq = ell;  // phys() is the identity
    }
    // ---- one block per merged ModDown + rescale: sources q_{ell-1}, p_0..p_{K-1} (limbs ell-1 .. of level ell)
    c->merged.resize(L + 1);
    for (u32 ell = 2; K > 0 && ell <= L; ell++) {
        const MergedLayout ml = merged_layout(off, ell, K);
        off = ml.end;
        const u32 T = ell - 1, S = K + 1;
        std::vector<u64> src(1, c->primes[T]);
        src.insert(src.end(), specials.begin(), specials.end());
        auto sph = [&](u32 k) { return k == 0 ? T : L + (k - 1); };  // chain index of source k
        InvScale* msc = (InvScale*)(hb + ml.sc_dn);
        PinvConst* pinv = (PinvConst*)(hb + ml.pinv);
        for (u32 k = 0; k < S; k++) {
            const u64 sk = src[k];
            const u64 hinv = h_invmod(prod_except(src, k, sk), sk);
            msc[k] = make_scale(hinv, ninv[sph(k)], wlast[sph(k)], sk, pc[sph(k)].fp != 0);
        }
        for (u32 i = 0; i < T; i++) {
            const u64 qi = c->primes[i];
            const u64 pi = h_invmod(prod_except(src, src.size(), qi), qi);
            pinv[i] = PinvConst{pi, h_shoup(pi, qi), (double)pi};
        }
        View& v = c->merged[ell];
        v.logN = logN, v.L = T, v.K = S, v.dnum = 1, v.alpha = T, v.D = ell + K, v.sh = &c->sh;
        v.primes = c->level[ell].primes;  // same limb order as the level: q_0..q_{ell-1}, p_0..p_{K-1}
        v.mixed_classes = c->level[ell].mixed_classes;
        Tables& tb = v.tb;
        memset(&tb, 0, sizeof(tb));
        shared_tables(tb);
        tb.sc_dn = (const InvScale*)(dbase + ml.sc_dn);
        tb.dn_hatinv = nullptr;
        tb.pinv = (const PinvConst*)(dbase + ml.pinv);
        tb.L = T, tb.K = S, tb.dnum = 1, tb.alpha = T, tb.D = ell + K, tb.Lfull = L, tb.Kfull = K, tb.Lq = ell;
        v.dn = ConvTab{(const u64*)(dbase + ml.dn_aop), nullptr, 1, mfma_ks(S), S};
        for (u32 t = 0; t < T; t++)
            build_aop((u64*)(hb + ml.dn_aop) + t * aop_words(v.dn.ks), hats(src, c->primes[t]), c->primes[t]);
    }

    hipStream_t s = (hipStream_t)stream;
    hipError_t e = hipMemcpyAsync(d_tables, host.data(), total, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    // this device's copy of the static scratch array (every GPU has its own, at its own address)
    if (e == hipSuccess) e = hipGetDevice(&c->device);
    if (e == hipSuccess) e = hipGetSymbolAddress(&c->scratch_ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !c->scratch_ptr) {
        (void)hipGetLastError();
        delete c;
        return CKKS_EHIP;
    }
    *out = c;
    return CKKS_OK;
}

extern "C" void ckks_ctx_destroy(ckks_ctx* ctx) {
    if (!ctx) return;
    prof_drain(ctx->sh.prof);
    for (hipEvent_t e : ctx->sh.prof.pool) (void)hipEventDestroy(e);
    if (ctx->sh.side.stream) {
        (void)hipStreamSynchronize(ctx->sh.side.stream);
        (void)hipStreamDestroy(ctx->sh.side.stream);
    }
    for (hipEvent_t e : ctx->sh.side.events) (void)hipEventDestroy(e);
    delete ctx;
}

extern "C" int ckks_profile_enable(ckks_ctx* ctx, int on) {
    if (!ctx) return CKKS_EINVAL;
    prof_drain(ctx->sh.prof);
    ctx->sh.prof.on = on != 0;
    ctx->sh.prof.kinds.clear();
    return CKKS_OK;
}

extern "C" int ckks_profile_read(ckks_ctx* ctx, uint32_t index, const char** name, uint64_t* launches,
                                 double* total_ms, uint64_t* alg_bytes) {
    if (!ctx) return CKKS_EINVAL;
    prof_drain(ctx->sh.prof);
    if (index >= ctx->sh.prof.kinds.size()) return CKKS_EINVAL;
    const ProfKindStat& k = ctx->sh.prof.kinds[index];
    if (name) *name = k.name.c_str();
    if (launches) *launches = k.launches;
    if (total_ms) *total_ms = k.ms;
    if (alg_bytes) *alg_bytes = k.bytes;
    return CKKS_OK;
}

extern "C" int ckks_set_overlap(ckks_ctx* ctx, int on) {
    if (!ctx) return CKKS_EINVAL;
    if (ctx->sh.side.active) return fail(ctx, CKKS_EINVAL, "cannot change overlap inside an operation");
    ctx->sh.side.enabled = on != 0;
    return CKKS_OK;
}

extern "C" const char* ckks_last_error(const ckks_ctx* ctx) { return ctx ? ctx->sh.err.c_str() : "null context"; }

extern "C" uint64_t ckks_ctx_psi(const ckks_ctx* ctx, uint32_t i) { return (ctx && i < ctx->D) ? ctx->psi[i] : 0; }

// ----------------------------------------------------------------------------- launches
static inline bool misaligned(const void* p, size_t a) { return ((uintptr_t)p & (a - 1)) != 0; }

static int hip_check(const View* c, const char* what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        c->sh->err = std::string(what) + ": " + hipGetErrorString(e);
        return CKKS_EHIP;
    }
    return CKKS_OK;
}

// grid of an XCD-aware launch: groups padded to a multiple of 8, times the instances per group
static inline u32 xcd_grid(u32 groups, u32 inst) { return ((groups + 7) / 8) * 8 * inst; }
static inline u32 cdiv(u32 a, u32 b) { return (a + b - 1) / b; }
static inline u32 tiles_of(const View* c) { return (1u << (c->logN - 8)) / 16; }

// Maximal runs of consecutive primes [lo, hi) that share an arithmetic (FpAr / IntAr).
struct ClassRun {
    u32 first, count;
    bool fp;
};
static std::vector<ClassRun> class_runs(const View* c, u32 lo, u32 hi) {
    std::vector<ClassRun> r;
    for (u32 i = lo; i < hi; i++) {
        const bool fp = c->primes[i] < CKKS_FP_PRIME_LIMIT;
        if (!r.empty() && r.back().fp == fp) r.back().count++;
        else r.push_back(ClassRun{i, 1, fp});
    }
    return r;
}

static bool any_fp_prime(const View* c, u32 lo, u32 hi) {
    for (u32 i = lo; i < hi; i++)
        if (c->primes[i] < CKKS_FP_PRIME_LIMIT) return true;
    return false;
}

// Words that one launch leaves for the next, `limbs` of them: written and read with ordinary accesses they may stay in the 256 MB
// Infinity Cache, which nontemporal ones leave empty; below 64 MiB there is no difference (46 MiB 53.6 / 53.6 us), more than it holds only
// evicts it (322 MiB and more written so: 2 to 10 % slower).  Times without / with, N = 2^16, one call after the other, us.  Rescale, 24 limbs: 3
// ciphertexts (69 MiB) 77.8 / 76.4, 4 (92) 94.3 / 88.3, 8 (184) 170 / 151, 12 (276, written so, read nontemporal) 253 / 233.  First
// forward pass of 24 limbs (the transform): 6 instances (72 MiB) 54.9 / 53.8, 16 (192) 136 / 128, 20 (240) 178 / 173; of 24 + 6 limbs: 6 (90)
// 76 / 78, 12 (180) 137 / 135.  On operands that were written just before, whose lines fill the cache, less: rescales behind the
// multiplication that they follow 0 to 2 % of both (8 ciphertexts 895 / 884), behind a copy -9 (4) to +6 % (3).  Not the ModDown conversions on
// the matrix cores, whose launches share the cache with the digits (HMult, batch 8: 699 / 704), nor conversions whose readers read nontemporal.
static bool stores_cached(const View* c, u64 limbs) { return (limbs * 8 << c->logN) >= (64ull << 20) && (limbs * 8 << c->logN) <= (320ull << 20); }
static bool loads_cached(const View* c, u64 limbs) { return stores_cached(c, limbs) && (limbs * 8 << c->logN) <= (224ull << 20); }

// A launcher type L provides
//   template <class AR, int A> static void go(grid, stream, args, tables, run)   the launch
//   static std::string name(const char* ar, int A)                               the profiler's kernel name
template <class L, class ArgT>
static void dispatch_kernel(const View* c, bool fp, dim3 grid, hipStream_t s, const ArgT& a, LimbRun run) {
#define CKKS_CASE_A(AV)                                               \
    case AV:                                                          \
        if (fp) L::template go<FpAr, AV>(grid, s, a, c->tb, run);     \
        else L::template go<IntAr, AV>(grid, s, a, c->tb, run);       \
        break;
    switch (c->logN - 8) {
        CKKS_CASE_A(4)
        CKKS_CASE_A(5)
        CKKS_CASE_A(6)
        CKKS_CASE_A(7)
        CKKS_CASE_A(8)
    }
#undef CKKS_CASE_A
}

template <class L, class ArgT>
static void dispatch_any(const View* c, dim3 grid, hipStream_t s, const ArgT& a, LimbRun run) {
    switch (c->logN - 8) {
        case 4: L::template go<AnyAr, 4>(grid, s, a, c->tb, run); break;
        case 5: L::template go<AnyAr, 5>(grid, s, a, c->tb, run); break;
        case 6: L::template go<AnyAr, 6>(grid, s, a, c->tb, run); break;
        case 7: L::template go<AnyAr, 7>(grid, s, a, c->tb, run); break;
        case 8: L::template go<AnyAr, 8>(grid, s, a, c->tb, run); break;
    }
}

static std::string kname(const char* base, const char* ar, int A, const char* tail) {
    return std::string(base) + "<" + ar + ", " + std::to_string(A) + tail + ">";
}

// One launch per arithmetic run of the primes [lo, hi).  limb_base converts a prime index into the kernel's limb index;
// groups = run limbs x groups_n, instances = inst_n.  alg(first, count) gives the algorithmic limbs (read + written once)
// of the launch covering primes [first, first+count).
// A range that mixes the arithmetics is one launch of the AnyAr form where the launcher has one (L::any: the plain passes)
// and the integer limbs do not run on the side stream.  Against a launch per arithmetic, forward / inverse: 30 FP64 and
// integer limbs x 48 at N = 2^14 135.9 against 144.4 us / 133.2 against 148.6; x 16 at N = 2^16 204.4 against 210.1 / 213.3
// against 223.8; small grids gain the launch; the closest is N = 2^13, inverse x 48, 74.5 against 73.6.
template <class L, class ArgT, class AlgFn>
static void launch_runs(const View* c, u32 lo, u32 hi, u32 limb_base, u32 groups_n, u32 inst_n, const ArgT& a, hipStream_t s,
                        AlgFn alg) {
    const std::vector<ClassRun> runs = class_runs(c, lo, hi);
    if constexpr (L::any) {
        if (runs.size() > 1 && !c->sh->side.active) {
            const LimbRun run = {lo - limb_base, hi - lo};
            const dim3 grid(xcd_grid((hi - lo) * groups_n, inst_n));
            ProfScope ps(c, c->sh->prof.on ? L::name("AnyAr", (int)c->logN - 8) : std::string(), c->sh->prof.on ? alg(lo, hi - lo) : 0, s);
            dispatch_any<L>(c, grid, s, a, run);
            return;
        }
    }
    for (const ClassRun& cr : runs) {
        const LimbRun run = {cr.first - limb_base, cr.count};
        hipStream_t rs = (!cr.fp && c->sh->side.active) ? c->sh->side.stream : s;
        ProfScope ps(c, c->sh->prof.on ? L::name(cr.fp ? "FpAr" : "IntAr", (int)c->logN - 8) : std::string(),
                     c->sh->prof.on ? alg(cr.first, cr.count) : 0, rs);
        dispatch_kernel<L>(c, cr.fp, dim3(xcd_grid(cr.count * groups_n, inst_n)), rs, a, run);
    }
}

template <int LOAD>
struct InvContigL {
    static constexpr bool any = LOAD == INV_PLAIN;
    template <class AR, int A>
    static void go(dim3 g, hipStream_t s, const InvContigArgs& a, const Tables& tb, LimbRun run) {
        hipLaunchKernelGGL((inv_contig_kernel<AR, A, LOAD>), g, dim3(inv_one_kernel(A) ? 16 << A : 256), 0, s, a, tb, run);
    }
    static std::string name(const char* ar, int A) {
        return kname("inv_contig_kernel", ar, A, LOAD == 0 ? ", 0" : LOAD == 1 ? ", 1" : ", 2");
    }
};
struct InvStridedL {
    static constexpr bool any = true;
    template <class AR, int A>
    static void go(dim3 g, hipStream_t s, const InvStridedArgs& a, const Tables& tb, LimbRun run) {
        hipLaunchKernelGGL((inv_strided_kernel<AR, A>), g, dim3(256), 0, s, a, tb, run);
    }
    static std::string name(const char* ar, int A) { return kname("inv_strided_kernel", ar, A, ""); }
};
struct InvStridedSumL {
    static constexpr bool any = false;
    template <class AR, int A>
    static void go(dim3 g, hipStream_t s, const InvStridedSumArgs& a, const Tables& tb, LimbRun run) {
        hipLaunchKernelGGL((inv_strided_sum_kernel<AR, A>), g, dim3(1024), 0, s, a, tb, run);
    }
    static std::string name(const char* ar, int A) { return kname("inv_strided_sum_kernel", ar, A, ""); }
};
struct FwdStridedL {
    static constexpr bool any = true;
    template <class AR, int A>
    static void go(dim3 g, hipStream_t s, const FwdStridedArgs& a, const Tables& tb, LimbRun run) {
        if constexpr (!inv_one_kernel(A) || (A == 5 && __is_same(AR, IntAr)))  // what launch_forward sends here
            hipLaunchKernelGGL((fwd_strided_kernel<AR, A>), g, dim3(256), 0, s, a, tb, run);
    }
    static std::string name(const char* ar, int A) { return kname("fwd_strided_kernel", ar, A, ""); }
};
struct FwdStridedCachedL {
    static constexpr bool any = true;
    template <class AR, int A>
    static void go(dim3 g, hipStream_t s, const FwdStridedArgs& a, const Tables& tb, LimbRun run) {
        if constexpr (!inv_one_kernel(A)) hipLaunchKernelGGL((fwd_strided_cached_kernel<AR, A>), g, dim3(256), 0, s, a, tb, run);
        else FwdStridedL::go<AR, A>(g, s, a, tb, run);  // two passes for a few limbs only: not reached
    }
    static std::string name(const char* ar, int A) { return kname("fwd_strided_cached_kernel", ar, A, ""); }
};
// ModDown from a single source with ordinary stores (enough targets for four FpAr ones per workgroup)
struct ConvOneCachedL {
    static constexpr bool packed = false;
    template <class AR>
    static constexpr int per_block() { return AR::is_fp ? 4 : 1; }
    template <class AR, int A>
    static void go(dim3 g, hipStream_t s, const ConvArgs& a, const Tables& tb, LimbRun run) {
        hipLaunchKernelGGL((conv_one_cached_kernel<AR, A, per_block<AR>()>), g, dim3(256), 0, s, a, tb, run);
    }
    static std::string name(const char* ar, int A) { return kname("conv_one_cached_kernel", ar, A, ar[0] == 'F' ? ", 4" : ", 1"); }
};
// Conversions: KS products per coefficient group on the matrix cores, or (KS = 0) a single source and TB targets per
// workgroup (one for IntAr).  KS > 0 and TB = 1: ModDown with two FpAr targets per workgroup instead of four
template <int DIR, int KS, int TB = 0, int... NW>
struct ConvL {
    static constexpr bool packed = KS > 0;  // blocks are numbered over the targets alone, without a digit's own limbs
    template <class AR>
    static constexpr int single() { return AR::is_fp ? TB : 1; }
    template <class AR>
    static constexpr int ntt() { return DIR == CONV_DN && TB ? 1 : conv_mfma_ntt<AR>(); }
    template <class AR>
    static constexpr int per_block() { return KS ? 2 * ntt<AR>() : single<AR>(); }
    template <class AR, int A>
    static void go(dim3 g, hipStream_t s, const ConvArgs& a, const Tables& tb, LimbRun run) {
        constexpr int NTT = ntt<AR>();
        if constexpr (KS == 0) hipLaunchKernelGGL((conv_fwd_strided_kernel<AR, A, DIR, single<AR>(), true>), g, dim3(256), 0, s, a, tb, run);
        else if constexpr (AR::is_fp && DIR == CONV_DN)
            hipLaunchKernelGGL((conv_mfma_kernel<A, KS, DIR, NTT, NW...>), g, dim3(512), 0, s, a, tb, run);
        else hipLaunchKernelGGL((conv_fwd_strided_kernel<AR, A, DIR, KS + NTT, false, NW...>), g, dim3(512), 0, s, a, tb, run);
    }
    static std::string name(const char* ar, int A) {
        const bool fp = ar[0] == 'F';
        const int t = fp ? ntt<FpAr>() : ntt<IntAr>();
        const std::string dir = std::to_string(DIR), words = sizeof...(NW) ? ", " + std::to_string((0 + ... + NW)) : std::string();
        if (KS && fp && DIR == CONV_DN) return "conv_mfma_kernel<" + std::to_string(A) + ", " + std::to_string(KS) + ", " + dir + ", " + std::to_string(t) + words + ">";
        return kname("conv_fwd_strided_kernel", ar, A, (", " + dir + ", " + std::to_string(KS ? KS + t : fp ? TB : 1) + (KS ? ", false" : ", true") + words).c_str());
    }
    struct Halves {  // IntAr targets in workgroups of 256 lanes
        static constexpr int words = sizeof...(NW) ? (0 + ... + NW) : 2 * KS;
        template <class AR, int A>
        static void go(dim3 g, hipStream_t s, const ConvArgs& a, const Tables& tb, LimbRun run) {
            if constexpr (!AR::is_fp && KS) hipLaunchKernelGGL((conv_int_kernel<A, KS, DIR, words>), g, dim3(256), 0, s, a, tb, run);
        }
        static std::string name(int A) {
            return "conv_int_kernel<" + std::to_string(A) + ", " + std::to_string(KS) + ", " + std::to_string(DIR) + ", " + std::to_string(words) + ">";
        }
    };
};
struct FwdContigL {
    static constexpr bool any = true;
    template <class AR, int A>
    static void go(dim3 g, hipStream_t s, const FwdContigArgs& a, const Tables& tb, LimbRun run) {
        hipLaunchKernelGGL((fwd_contig_kernel<AR, A>), g, dim3(256), 0, s, a, tb, run);
    }
    static std::string name(const char* ar, int A) { return kname("fwd_contig_kernel", ar, A, ""); }
};
template <int OWN, bool HOISTED, bool FUSED>
struct KsInnerL {
    template <class AR, int A>
    static void go(dim3 g, hipStream_t s, const InnerArgs& a, const Tables& tb, LimbRun run) {
        hipLaunchKernelGGL((ks_inner_kernel<AR, A, OWN, HOISTED, FUSED>), g, dim3(256), 0, s, a, tb, run);
    }
    static std::string name(const char* ar, int A) {
        return kname("ks_inner_kernel", ar, A,
                     (std::string(", ") + std::to_string(OWN) + (HOISTED ? ", true" : ", false") + (FUSED ? ", true" : ", false"))
                         .c_str());
    }
};
template <int MODE>
struct KsFinalL {
    static constexpr bool any = false;
    template <class AR, int A>
    static void go(dim3 g, hipStream_t s, const FinalArgs& a, const Tables& tb, LimbRun run) {
        hipLaunchKernelGGL((ks_final_kernel<AR, A, MODE>), g, dim3(256), 0, s, a, tb, run);
    }
    static std::string name(const char* ar, int A) {
        return kname("ks_final_kernel", ar, A, (std::string(", ") + std::to_string(MODE)).c_str());
    }
};
struct KsFinalCachedL {
    static constexpr bool any = false;
    template <class AR, int A>
    static void go(dim3 g, hipStream_t s, const FinalArgs& a, const Tables& tb, LimbRun run) {
        hipLaunchKernelGGL((ks_final_cached_kernel<AR, A>), g, dim3(256), 0, s, a, tb, run);
    }
    static std::string name(const char* ar, int A) { return kname("ks_final_cached_kernel", ar, A, ""); }
};

template <int LOAD>
static void launch_inv_contig(const View* c, const InvContigArgs& a, hipStream_t s) {
    const u32 pb = a.sel.prime_base;
    const u64 per = (u64)a.sel.n_inst * (LOAD == INV_TENSOR ? 3 : 2);
    launch_runs<InvContigL<LOAD>>(c, pb, pb + a.sel.n_l, pb, inv_one_kernel((int)c->logN - 8) ? 1 : tiles_of(c), a.sel.n_inst, a, s,
                                  [per](u32, u32 n) { return per * n; });
}

static void launch_inv_strided(const View* c, const InvStridedArgs& a, hipStream_t s) {
    const u32 pb = a.sel.prime_base;
    const u64 per = (u64)a.sel.n_inst * 2;
    launch_runs<InvStridedL>(c, pb, pb + a.sel.n_l, pb, tiles_of(c), a.sel.n_inst, a, s,
                             [per](u32, u32 n) { return per * n; });
}

// At N = 2^13 a few integer limbs are faster in two passes over twice the workgroups than in one kernel each: the workgroup
// of a limb then is all of the time, and its integer butterflies, two wavefronts a SIMD, take longer than a launch.  Forward /
// inverse, 1 limb: 12.2 against 14.0 us / 14.5 against 15.1; 24 limbs 13.2 against 14.5 / 15.5 against 15.6; 64 limbs 14.5 against
// 14.9 / 16.9 against 16.0; 80 limbs 15.0 against 15.1; 96 limbs 15.8 against 15.2.  FP64 limbs: one kernel at every size
// (1 limb 10.8 against 7.7 / 10.6 against 8.6), a range that mixes both likewise.
static bool spread_limbs(const View* c, const LimbSel& sel, u32 most) {
    return c->logN == 13 && sel.n_l * sel.n_inst <= most && !any_fp_prime(c, sel.prime_base, sel.prime_base + sel.n_l);
}

// The inverse transform of a.sel's limbs into a.dst
template <int LOAD>
static void launch_inverse(const View* c, InvContigArgs a, u32 scale, u32 out_fmt, hipStream_t s) {
    a.scale = scale, a.out_fmt = out_fmt;
    if (LOAD == INV_PLAIN && spread_limbs(c, a.sel, 24)) {
        hipStream_t rs = c->sh->side.active ? c->sh->side.stream : s;
        ProfScope ps(c, c->sh->prof.on ? kname("inv_contig_rows_kernel", "IntAr", 5, ", 0") : std::string(), (u64)a.sel.n_l * a.sel.n_inst * 2, rs);
        hipLaunchKernelGGL((inv_contig_rows_kernel<IntAr, 5, INV_PLAIN>), dim3(xcd_grid(a.sel.n_l * tiles_of(c), a.sel.n_inst)), dim3(256), 0, rs,
                           a, c->tb, LimbRun{0, a.sel.n_l});
    } else {
        launch_inv_contig<LOAD>(c, a, s);
        if (inv_one_kernel((int)c->logN - 8)) return;
    }
    const InvStridedArgs a2 = {a.dst, a.dsel, scale, out_fmt};
    launch_inv_strided(c, a2, s);
}

static void launch_fwd_strided(const View* c, const FwdStridedArgs& a, hipStream_t s, bool cached) {
    const u32 pb = a.sel.prime_base;
    const u64 per = (u64)a.sel.n_inst * 2;
    const auto alg = [per](u32, u32 n) { return per * n; };
    if (cached) launch_runs<FwdStridedCachedL>(c, pb, pb + a.sel.n_l, pb, tiles_of(c), a.sel.n_inst, a, s, alg);
    else launch_runs<FwdStridedL>(c, pb, pb + a.sel.n_l, pb, tiles_of(c), a.sel.n_inst, a, s, alg);
}

// largest number of targets of the run over the digits, and their sum: a digit's own limbs are none of its targets
static u32 conv_up_targets(const View* c, const ClassRun& cr, u32& total) {
    u32 most = 0;
    total = 0;
    for (u32 j = 0; j < c->dnum; j++) {
        const u32 own_hi = (j + 1) * c->alpha < c->L ? (j + 1) * c->alpha : c->L;
        const u32 lo = j * c->alpha > cr.first ? j * c->alpha : cr.first, hi = own_hi < cr.first + cr.count ? own_hi : cr.first + cr.count;
        const u32 n = cr.count - (hi > lo ? hi - lo : 0);
        total += n;
        if (n > most) most = n;
    }
    return most;
}

// Conversions onto IntAr targets of a launch of that many workgroups and more: 256 lanes a workgroup with two positions each instead of
// 512 with one.  The short workgroups are the faster ones while the launch is a few rounds (whole rotations, 256 / 512 lanes: below
// 600 workgroups 1.02 to 1.08), the long ones, three to a compute unit instead of two, on many (integer chains of 12 + 4 to 96 + 8 limbs,
// N = 2^12 .. 2^16, 512 / 256 lanes: 1200 to 3000 workgroups 0.99 to 1.02, from there on 1.00 to 1.04, two sources at N = 2^12 0.97 to 0.99;
// special limbs alone 0.99 to 1.02).  The conversion of 42 + 12 limbs, 10 sources, batch 4, N = 2^16: 339 -> 300 us
#define CKKS_CONV_INT_FROM 3072u
// one launch per arithmetic run of the targets
// only: -1 = every run, 0 = IntAr runs only, 1 = FpAr runs only
template <class L, int DIR>
static void launch_conv_runs(const View* c, ConvArgs a, hipStream_t s, int only) {
    for (const ClassRun& cr : class_runs(c, 0, DIR == CONV_UP ? c->D : c->L)) {
        if (only >= 0 && (int)cr.fp != only) continue;
        const u32 blk = cr.fp ? L::template per_block<FpAr>() : L::template per_block<IntAr>();
        u32 most = cr.count, written = cr.count;
        if (DIR == CONV_UP) most = conv_up_targets(c, cr, written);
        if (!most) continue;
        a.blocks = ((L::packed ? most : cr.count) + blk - 1) / blk;
        const dim3 grid(xcd_grid(a.groups_outer * (DIR == CONV_UP ? c->dnum : 1) * tiles_of(c), a.blocks));
        hipStream_t rs = (!cr.fp && c->sh->side.active) ? c->sh->side.stream : s;
        // every target written, plus the source coefficients, read once
        const u64 alg = (u64)a.groups_outer * (written + (DIR == CONV_UP ? c->L : c->K));
        if constexpr (L::packed)
            if (!cr.fp && grid.x >= CKKS_CONV_INT_FROM) {
                ProfScope ps(c, c->sh->prof.on ? L::Halves::name((int)c->logN - 8) : std::string(), alg, rs);
                dispatch_kernel<typename L::Halves>(c, false, grid, rs, a, LimbRun{cr.first, cr.count});
                continue;
            }
        ProfScope ps(c, c->sh->prof.on ? L::name(cr.fp ? "FpAr" : "IntAr", (int)c->logN - 8) : std::string(), alg, rs);
        dispatch_kernel<L>(c, cr.fp, grid, rs, a, LimbRun{cr.first, cr.count});
    }
}

// ModUp onto both arithmetics in one launch, where the chain is FpAr limbs followed by IntAr limbs (N >= 2^14; below, and with more
// than eight sources, no such kernel is built).  Two launches / one, whole calls on one stream, us: one rotation at N = 2^16, 24 + 6
// limbs 146.5 / 134, level 13 113 / 108; 2 of them 224 / 211, at level 13 8 (2304 workgroups) 414 / 405; N = 2^15, level 17, 3 145 / 135, 8
// 262 / 251; N = 2^14, 24 + 6, 12 296 / 284; from 4096 workgroups on no difference (8 of 24 + 6: 683 / 681; 8 of 35 + 7: 1086 / 1084), each
// has its own launch.  Where the targets would otherwise run beside each other on the second stream, up to `most`
// workgroups: with BESIDE 1024 (N = 2^16, 24 + 6, 2 rotations (1024) 218 / 212, 4 (2048) 361 / 374; level 13, 2 157 / 145), with
// FORK 512 (dh, 35 + 7 limbs (880), one rotation 258 / 263).  Returns false where it does not apply.
static bool conv_up_both(const View* c, const ConvArgs& base, hipStream_t s, u32 most) {
    const u32 ks = c->up.ks;
    if (c->logN < 14 || (ks != 1 && ks != 2)) return false;
    const std::vector<ClassRun> runs = class_runs(c, 0, c->D);
    if (runs.size() != 2 || !runs[0].fp) return false;
    ConvBothArgs a;
    a.fp = base;
    a.fp.aop = c->up.aop, a.fp.aop_part = c->up.aop_part, a.fp.n_full = c->up.n_full;
    a.in = a.fp;
    u32 w0, w1;
    const u32 groups = base.groups_outer * c->dnum * tiles_of(c), targets_fp = conv_up_targets(c, runs[0], w0);
    a.in.blocks = (conv_up_targets(c, runs[1], w1) + 1) / 2;
    if (!targets_fp || !a.in.blocks) return false;
    a.run_fp = LimbRun{runs[0].first, runs[0].count}, a.run_in = LimbRun{runs[1].first, runs[1].count};
    a.grid_in = xcd_grid(groups, a.in.blocks);
    a.fp.blocks = (targets_fp + 3) / 4;
    const u32 grid = a.grid_in + xcd_grid(groups, a.fp.blocks);
    if (grid > most) return false;
    const bool fewer = c->up.fewer();
    ProfScope ps(c, c->sh->prof.on ? "conv_up_both_kernel<" + std::to_string((int)c->logN - 8) + ", " + std::to_string(ks) + (fewer ? ks == 1 ? ", 1>" : ", 3>" : ">") : std::string(),
                 (u64)base.groups_outer * (w0 + w1 + c->L), s);
#define CKKS_BOTH_AS(...) hipLaunchKernelGGL((conv_up_both_kernel<__VA_ARGS__>), dim3(grid), dim3(512), 0, s, a, c->tb)
#define CKKS_BOTH(AV)                                \
    case AV:                                         \
        if (ks == 1 && fewer) CKKS_BOTH_AS(AV, 1, 1);   \
        else if (ks == 1) CKKS_BOTH_AS(AV, 1);       \
        else if (fewer) CKKS_BOTH_AS(AV, 2, 3);      \
        else CKKS_BOTH_AS(AV, 2);                    \
        break;
    switch (c->logN - 8) {
        CKKS_BOTH(6)
        CKKS_BOTH(7)
        CKKS_BOTH(8)
    }
#undef CKKS_BOTH
#undef CKKS_BOTH_AS
    return true;
}

// workgroups of a ModUp onto every class of targets, four FpAr or two IntAr targets each
static u32 conv_up_workgroups(const View* c, u32 batch) {
    u32 blocks = 0, total;
    for (const ClassRun& r : class_runs(c, 0, c->D)) blocks += cdiv(conv_up_targets(c, r, total), r.fp ? 4 : 2);
    return batch * c->dnum * tiles_of(c) * blocks;
}

// word format in which the last inverse stage leaves the sources of a conversion
static inline u32 conv_src_fmt(const ConvTab& t, int dir) { return t.ks ? SRC_DIGITS : dir == CONV_UP ? SRC_F64 : SRC_CANON; }

// cls: -1 = every target, 0 = IntAr targets only, 1 = FpAr targets only
template <int DIR>
static void launch_conv(const View* c, ConvArgs a, hipStream_t s, int cls = -1) {
    const ConvTab& t = DIR == CONV_UP ? c->up : c->dn;
    a.aop = t.aop, a.aop_part = t.aop_part, a.n_full = t.n_full;
    const u32 groups = a.groups_outer * (DIR == CONV_UP ? c->dnum : 1) * tiles_of(c), fours = groups * (((DIR == CONV_UP ? c->D : c->L) + 3) / 4);
    // ModDown onto FpAr limbs: two targets per workgroup instead of four while that leaves one workgroup per compute unit (calls
    // of one ciphertext at N = 2^16, 24 + 6 limbs: level 13 (256 workgroups of two) 107.7 -> 104.1 us, level 24 (384) 136.8 -> 137.3)
    const bool narrow = DIR == CONV_DN && fours <= 128;
#define CKKS_CONV(KS, ...)                                                                         \
    if (DIR == CONV_DN && narrow) launch_conv_runs<ConvL<DIR, KS, DIR == CONV_DN, ##__VA_ARGS__>, DIR>(c, a, s, cls); \
    else launch_conv_runs<ConvL<DIR, KS, 0, ##__VA_ARGS__>, DIR>(c, a, s, cls)
    switch (t.ks) {
        case 0:
            // Four FP64 targets share a load of the source unless that leaves fewer than two workgroups per compute unit.  Integer
            // targets are converted singly: two or four per workgroup need 146 registers, three waves per SIMD, and end in
            // half-empty rounds (rescale of 7 ciphertexts at N = 2^15, 19 integer limbs: 106 us singly, 116 with four).
            if (fours >= 512) launch_conv_runs<ConvL<DIR, 0, 4>, DIR>(c, a, s, cls);
            else launch_conv_runs<ConvL<DIR, 0, 1>, DIR>(c, a, s, cls);
            break;
        case 1:
            if (t.fewer()) { CKKS_CONV(1, 1); }
            else { CKKS_CONV(1); }
            break;
        case 2:
            if (t.fewer()) { CKKS_CONV(2, 3); }
            else { CKKS_CONV(2); }
            break;
        case 4: launch_conv_runs<ConvL<DIR, 4>, DIR>(c, a, s, cls); break;
        case 5:
            if constexpr (DIR == CONV_DN) launch_conv_runs<ConvL<DIR, 5>, DIR>(c, a, s, cls);
            break;
    }
#undef CKKS_CONV
}

static void launch_fwd_contig(const View* c, const FwdContigArgs& a, hipStream_t s) {
    const u32 pb = a.sel.prime_base;
    const u64 per = (u64)a.sel.n_inst * 2;
    launch_runs<FwdContigL>(c, pb, pb + a.sel.n_l, pb, tiles_of(c), a.sel.n_inst, a, s,
                            [per](u32, u32 n) { return per * n; });
}

// forward transform in place: one kernel where a workgroup holds a limb, else two passes
static void launch_forward(const View* c, u64* d_x, const LimbSel& sel, hipStream_t s) {
    const FwdContigArgs a2 = {d_x, sel, 0, 0};
    if (!inv_one_kernel((int)c->logN - 8) || spread_limbs(c, sel, 80)) {
        const FwdStridedArgs a1 = {d_x, d_x, sel};
        launch_fwd_strided(c, a1, s, stores_cached(c, (u64)sel.n_l * sel.n_inst));
        launch_fwd_contig(c, a2, s);
        return;
    }
    ProfScope ps(c, c->sh->prof.on ? "fwd_whole_kernel<" + std::to_string((int)c->logN - 8) + ">" : std::string(), (u64)sel.n_l * sel.n_inst * 2, s);
    const dim3 grid(xcd_grid(sel.n_l, sel.n_inst)), block(1u << (c->logN - 4));
    const LimbRun run = {0, sel.n_l};
    switch (c->logN - 8) {
        case 4: hipLaunchKernelGGL(fwd_whole_kernel<4>, grid, block, 0, s, a2, c->tb, run); break;
        case 5: hipLaunchKernelGGL(fwd_whole_kernel<5>, grid, block, 0, s, a2, c->tb, run); break;
    }
}

// Wavefronts that share the digits of a row in the inner product (InnerArgs::ways) for a launch of `wgs` workgroups of 16
// rows.  A workgroup's time is about one unit per digit it works through and one per component it ends, two workgroups
// fit a compute unit: compare rounds times units.  One HMult at N = 2^16, dnum = 4: special limbs, 96 workgroups, 48 -> 28 us (four);
// at N = 2^12, dnum = 3: special limb 14 -> 9 us, q-limbs 16 -> 10 us (four); HMult at N = 2^15, level 17, batch 3, special limbs, 144
// workgroups: the call 141 -> 133 us (two); N = 2^16, 12 + 2 limbs, dnum = 6, q-limbs, 192 workgroups: 123 -> 113 (two).  On more
// than one round of workgroups two are no gain whatever the rounds say: 768 workgroups, N = 2^16, dnum = 6, 235 -> 242 us.
static u32 inner_ways(u32 wgs, u32 dnum, u32& least) {
    u32 best = 1;
    least = (wgs + 511) / 512 * (2 * dnum + 4);
    for (u32 ways = 2; ways <= 4 && dnum > 1; ways *= 2) {
        const u32 t = (ways * wgs + 511) / 512 * (2 * ((dnum + ways - 1) / ways) + 3);
        if (t < least && (ways == 4 || wgs <= 512)) best = ways, least = t;
    }
    return best;
}
static u32 inner_ways(u32 wgs, u32 dnum) {
    u32 time;
    return inner_ways(wgs, dnum, time);
}

// limbs [lo, hi) of the extended basis.  FUSED: the launch also ends the ModDown on its limbs (all below
// a.split, after the conversion of the special part) and writes the result instead of c'.
template <int OWN, bool HOISTED, bool FUSED = false>
static void launch_ks_inner(const View* c, InnerArgs a, hipStream_t s, u32 lo, u32 hi) {
    const u64 n_inst = a.n_inst;
    typedef KsInnerL<OWN, HOISTED, FUSED> L;
    std::vector<ClassRun> runs = class_runs(c, lo, hi);
    // hoisted rotations: the FP64 limbs stream keys and digits, the integer limbs are bound by instructions; in one launch
    // they share the chip (17 rotations at N = 2^16, L = 24, in launches of 9
    // and 8: 242 + 95 and 196 + 78 us -> 325 and 271 us).  Merged rescale: limb L - 1 beside the special limbs (HMult, N = 2^15,
    // level 17, batch 3: 148 -> 136 us; N = 2^16, 24 + 6 limbs, batch 3: 330 -> 319).
    constexpr bool JOINT = HOISTED || (OWN == OWN_TENSOR && !FUSED);
    const bool any = JOINT && runs.size() > 1 && !c->sh->side.active;
    if (any) runs.assign(1, ClassRun{lo, hi - lo, true});
    for (const ClassRun& cr : runs) {
        const u32 terms = (OWN == OWN_ROT_SUM ? a.n_sum : 1) * c->dnum;
        a.ways = HOISTED ? 1 : inner_ways(cr.count * tiles_of(c) * a.n_inst, terms);
        hipStream_t rs = (!cr.fp && c->sh->side.active) ? c->sh->side.stream : s;
        u64 limbs = 0;
        for (u32 i = cr.first; i < cr.first + cr.count; i++) {
            const bool q = i < c->L;
            const u64 sums = OWN == OWN_ROT_SUM ? a.n_sum : 1;
            limbs += n_inst * (sums * ((u64)c->dnum - (q ? 1 : 0)        // extended digits outside their own limbs
                                       + (q ? (OWN == OWN_TENSOR ? 4 : 1) : 0)       // the switched polynomial (HMult: both inputs) on its own limb
                                       + (OWN == OWN_ROT || OWN == OWN_ROT_SUM ? FUSED : 0))  // sigma_g(b)
                               + 2                                     // c' (or the result) written
                               + (FUSED ? 2 : 0))                      // converted special part
                     + (HOISTED ? n_inst : sums) * 2 * (u64)c->dnum;   // key limbs
        }
        const dim3 grid(xcd_grid(cr.count * tiles_of(c) * a.ways, a.n_inst));
        ProfScope ps(c, c->sh->prof.on ? L::name(any ? "AnyAr" : cr.fp ? "FpAr" : "IntAr", (int)c->logN - 8) : std::string(), limbs, rs);
        if constexpr (JOINT)
            if (any) {
                dispatch_any<L>(c, grid, rs, a, LimbRun{cr.first, cr.count});
                continue;
            }
        dispatch_kernel<L>(c, cr.fp, grid, rs, a, LimbRun{cr.first, cr.count});
    }
}
#define CKKS_BSGS_EPT 4
struct BsgsMacL {
    template <class AR, int A>
    static void go(dim3 g, hipStream_t s, const BsgsMacArgs& a, const Tables& tb, LimbRun run) {
        hipLaunchKernelGGL((bsgs_mac_kernel<AR, CKKS_BSGS_EPT>), g, dim3(256), 0, s, a, tb, run);
    }
    static std::string name(const char* ar, int) {
        return std::string("bsgs_mac_kernel<") + ar + ", " + std::to_string(CKKS_BSGS_EPT) + ">";
    }
};

static void launch_bsgs_mac(const View* c, const BsgsMacArgs& a, hipStream_t s) {
    const u32 chunks = (1u << c->logN) / (256 * CKKS_BSGS_EPT);
    for (const ClassRun& cr : class_runs(c, 0, c->D)) {
        const LimbRun run = {cr.first, cr.count};
        hipStream_t rs = (!cr.fp && c->sh->side.active) ? c->sh->side.stream : s;
        // per limb and giant step: n1 rotations (2 components) and n1 plaintexts read, 2 components written
        ProfScope ps(c, c->sh->prof.on ? BsgsMacL::name(cr.fp ? "FpAr" : "IntAr", 0) : std::string(),
                     (u64)cr.count * a.n2 * (3 * (u64)a.n1 + 2), rs);
        dispatch_kernel<BsgsMacL>(c, cr.fp, dim3(xcd_grid(cr.count * chunks, a.n2)), rs, a, run);
    }
}

// All limbs of the extended basis in one launch.  Chains of integer primes alone take the narrow form: with few digits the
// unreduced sums save an integer limb no products, and three waves per SIMD leave it waiting where FP64 limbs beside it would
// fill in.  9 rotations at N = 2^16, L + K = 12 + 4, dnum = 3: the call 248 us before the wide form, 268 with it, 257 with
// the narrow one; at N = 2^15, 27 + 3, dnum = 9, 5 rotations: 346, 365, 346.  On mixed chains the wide form is the faster one
// (18 rotations, 24 + 6, dnum = 4: 669 against 683 us).
static void launch_dh_accum_run(const View* c, DhInnerArgs a, u32 first, u32 count, bool all_int, hipStream_t s) {
    const u64 n_rot = a.n_rot, acc = a.accumulate ? 2 : 0, dnum = c->dnum, sums = a.sums ? a.sums : 1;
    a.first = first, a.count = count;
    // With few rotations the accumulation is a chain of a few waits on the keys, which more wavefronts in flight shorten
    // (N = 2^16, 26 + 6 limbs, dnum 5: 3 rotations 317 us wide, 310 narrow, 6 rotations 441 / 425, 8 rotations 507 / 497); from
    // about ten on the wide rows of a mixed chain are even or up to 3 % faster.  Several sums: narrow rows, for the registers (four
    // sums of 8 rotations, 24 + 6 limbs, in rows of 256 words at two waves per SIMD: the call 956 us with four rows a workgroup and
    // 1005 with one shared, against 955).
    const bool narrow = all_int || n_rot <= 8 || sums > 1;
    const u32 rows = count * ((1u << c->logN) / (64 * (narrow ? 2 : 4)));
    // Four rows per workgroup, or one whose rotations the four wavefronts share.  Narrow, one sum: fewer rounds of the 1280 resident
    // workgroups times rotations per wavefront.  Several sums: sums_waves has the rule and both sides.  Wide: with fewer than eight
    // rotations the wavefronts would end up with unequal shares, which only a grid below two workgroups per compute unit makes up for.
    const u32 resident = 1280;
    if (sums > 1) a.waves = sums_waves(rows, a.n_rot);
    else if (narrow) a.waves = (rows + resident - 1) / resident * ((a.n_rot + 3) / 4) < (rows / 4 + resident - 1) / resident * a.n_rot ? 4 : 1;
    else a.waves = n_rot >= 8 || (rows / 4 < 512 && n_rot > 1) ? 4 : 1;
    u64 limbs = 0;  // per limb and rotation: the digits, the plaintexts, both key components (and b on q-limbs); C_t written
    for (u32 i = first; i < first + count; i++) limbs += n_rot * (3 * dnum + (a.pt ? sums : 0) + (i < c->L ? 1 : 0)) + (a.each ? 2 * n_rot : 2 * sums) + acc;
    const std::string form = std::string(all_int ? "IntAr, " : "AnyAr, ") + (narrow ? "2" : "4") + (sums > 1 ? ", " + std::to_string(sums) : std::string());
    ProfScope ps(c, c->sh->prof.on ? "dh_accum_kernel<" + form + ">" : std::string(), limbs, s);
    const dim3 grid((rows * a.waves / 4 + 7) / 8 * 8);
#define CKKS_DH(...)                                                                                                 \
    if (all_int) hipLaunchKernelGGL((dh_accum_kernel<IntAr, __VA_ARGS__>), grid, dim3(256), 0, s, a, c->tb);         \
    else hipLaunchKernelGGL((dh_accum_kernel<AnyAr, __VA_ARGS__>), grid, dim3(256), 0, s, a, c->tb)
    switch (sums) {
        case 2: CKKS_DH(2, 2); break;
        case 3: CKKS_DH(2, 3); break;
        case 4: CKKS_DH(2, 4); break;
        default:
            if (narrow) { CKKS_DH(2); }
            else hipLaunchKernelGGL((dh_accum_kernel<AnyAr, 4>), grid, dim3(256), 0, s, a, c->tb);
    }
#undef CKKS_DH
}
// limbs [0, hi) in one launch, or one per arithmetic while the integer limbs have the side stream
static void launch_dh_accum(const View* c, const DhInnerArgs& a, hipStream_t s, u32 hi) {
    if (!c->sh->side.active) return launch_dh_accum_run(c, a, 0, hi, !any_fp_prime(c, 0, hi), s);
    for (const ClassRun& r : class_runs(c, 0, hi)) launch_dh_accum_run(c, a, r.first, r.count, !r.fp, r.fp ? s : c->sh->side.stream);
}

template <int MODE, bool CACHED = false>
static void launch_ks_final(const View* c, const FinalArgs& a, hipStream_t s) {
    u64 per;  // algorithmic limbs per q-limb
    if (MODE == FIN_HOISTED) per = (u64)a.n_rot * (2 + 2 + 1 + 1) + (2 + (a.accumulate ? 2 : 0));
    else if (MODE == FIN_SUMMED) per = (u64)a.n_rot * (2 + 1) + (2 + 2 + (a.accumulate ? 2 : 0));
    else per = (u64)a.n_inst * 3;
    launch_runs<typename std::conditional<CACHED, KsFinalCachedL, KsFinalL<MODE>>::type>(c, 0, c->L, 0, tiles_of(c), a.n_inst, a, s, [per](u32, u32 n) { return per * n; });
}

template <int AL>
static void launch_modup_a(const View* c, const u64* in, u64* out, u32 batch, hipStream_t s) {
    const dim3 grid((1u << c->logN) / 256, c->dnum, batch), block(256);
    ProfScope ps(c, std::string("modup_kernel"), (u64)batch * (2 * (u64)c->L + (u64)c->dnum * (c->D - c->alpha)), s);
    hipLaunchKernelGGL(modup_kernel<AL>, grid, block, 0, s, in, out, c->tb);
}
static void launch_modup(const View* c, const u64* in, u64* out, u32 batch, hipStream_t s) {
    switch (c->alpha) {
        case 1: launch_modup_a<1>(c, in, out, batch, s); break;
        case 2: launch_modup_a<2>(c, in, out, batch, s); break;
        case 3: launch_modup_a<3>(c, in, out, batch, s); break;
        case 4: launch_modup_a<4>(c, in, out, batch, s); break;
        case 5: launch_modup_a<5>(c, in, out, batch, s); break;
        case 6: launch_modup_a<6>(c, in, out, batch, s); break;
        case 7: launch_modup_a<7>(c, in, out, batch, s); break;
        case 8: launch_modup_a<8>(c, in, out, batch, s); break;
        case 9: launch_modup_a<9>(c, in, out, batch, s); break;
        case 10: launch_modup_a<10>(c, in, out, batch, s); break;
        case 11: launch_modup_a<11>(c, in, out, batch, s); break;
        case 12: launch_modup_a<12>(c, in, out, batch, s); break;
        case 13: launch_modup_a<13>(c, in, out, batch, s); break;
        case 14: launch_modup_a<14>(c, in, out, batch, s); break;
        case 15: launch_modup_a<15>(c, in, out, batch, s); break;
        case 16: launch_modup_a<16>(c, in, out, batch, s); break;
    }
}

template <int KK>
static void launch_moddown_k(const View* c, const u64* in, u64* out, u32 groups, hipStream_t s) {
    const dim3 grid((1u << c->logN) / 256, groups), block(256);
    ProfScope ps(c, std::string("moddown_kernel"), (u64)groups * (c->K + 2 * (u64)c->L), s);
    hipLaunchKernelGGL(moddown_kernel<KK>, grid, block, 0, s, in, out, c->tb);
}
static void launch_moddown(const View* c, const u64* in, u64* out, u32 groups, hipStream_t s) {
    switch (c->K) {
        case 1: launch_moddown_k<1>(c, in, out, groups, s); break;
        case 2: launch_moddown_k<2>(c, in, out, groups, s); break;
        case 3: launch_moddown_k<3>(c, in, out, groups, s); break;
        case 4: launch_moddown_k<4>(c, in, out, groups, s); break;
        case 5: launch_moddown_k<5>(c, in, out, groups, s); break;
        case 6: launch_moddown_k<6>(c, in, out, groups, s); break;
        case 7: launch_moddown_k<7>(c, in, out, groups, s); break;
        case 8: launch_moddown_k<8>(c, in, out, groups, s); break;
        case 9: launch_moddown_k<9>(c, in, out, groups, s); break;
        case 10: launch_moddown_k<10>(c, in, out, groups, s); break;
        case 11: launch_moddown_k<11>(c, in, out, groups, s); break;
        case 12: launch_moddown_k<12>(c, in, out, groups, s); break;
        case 13: launch_moddown_k<13>(c, in, out, groups, s); break;
        case 14: launch_moddown_k<14>(c, in, out, groups, s); break;
        case 15: launch_moddown_k<15>(c, in, out, groups, s); break;
        case 16: launch_moddown_k<16>(c, in, out, groups, s); break;
    }
}

// ---------------------------------------------------------------------- workspace carving
// x  [xg][L][N]        coefficients of the switched polynomial (raw after pass 1, then canonical * pre-factor)
// dt [dg][dnum][D][N]  extended digits (first forward pass done; own-digit limbs unused)
// cq [cg][2][L][N]     c' on the q-limbs, canonical evaluation form
// cp [cg][2][K][N]     c' on the special limbs: raw after the first inverse pass, then coefficients * pre-factor
// cv [cg][2][L][N]     Conv_{P->Q} of the special part, first forward pass done
struct Workspace {
    u64 *x, *dt, *cq, *cp, *cv;
};

// with_cq = false: the plain key-switch pipeline, whose c' on the q-limbs never leaves the registers of the kernel
// that accumulates it: no cq (a fifth of the workspace at (24,6,4))
static size_t ks_workspace_words(const View* c, u32 xg, u32 dg, u32 cg, bool with_cq = true) {
    const size_t N = (size_t)1 << c->logN;
    return ((size_t)xg * c->L + (size_t)dg * c->dnum * c->D + (size_t)cg * 2 * ((with_cq ? 2 : 1) * (size_t)c->L + c->K)) * N;
}

static Workspace carve(const View* c, void* ws, u32 xg, u32 dg, u32 cg, bool with_cq = true) {
    const size_t N = (size_t)1 << c->logN;
    Workspace w;
    w.x = (u64*)ws;
    w.dt = w.x + (size_t)xg * c->L * N;
    w.cq = w.dt + (size_t)dg * c->dnum * c->D * N;
    w.cp = w.cq + (with_cq ? (size_t)cg * 2 * c->L * N : 0);
    w.cv = w.cp + (size_t)cg * 2 * c->K * N;
    if (!with_cq) w.cq = nullptr;
    return w;
}

static int view_workspace_bytes(const View* v, int op, uint32_t batch_or_nrot, size_t* bytes) {
    if (batch_or_nrot == 0) return fail(v, CKKS_EINVAL, "batch must be positive");
    switch (op) {
        case CKKS_OP_NTT:
        case CKKS_OP_MODUP:
        case CKKS_OP_MODDOWN:
        case CKKS_OP_AUTOMORPH: *bytes = 0; return CKKS_OK;
        case CKKS_OP_KEYSWITCH:
        case CKKS_OP_HMULT_RELIN:
        case CKKS_OP_HROT:
            if (v->K == 0) return fail(v, CKKS_EUNSUPPORTED, "context has no special primes");
            *bytes = ks_workspace_words(v, batch_or_nrot, batch_or_nrot, batch_or_nrot, false) * sizeof(u64);
            return CKKS_OK;
        case CKKS_OP_HROT_HOISTED_MAC: {
            if (v->K == 0) return fail(v, CKKS_EUNSUPPORTED, "context has no special primes");
            const u32 chunk = batch_or_nrot < CKKS_ROT_CHUNK ? batch_or_nrot : CKKS_ROT_CHUNK;
            *bytes = ks_workspace_words(v, 1, 1, chunk) * sizeof(u64);
            return CKKS_OK;
        }
        case CKKS_OP_HROT_DH_MAC:
            if (v->K == 0) return fail(v, CKKS_EUNSUPPORTED, "context has no special primes");
            *bytes = ks_workspace_words(v, 1, 1, 1) * sizeof(u64);
            return CKKS_OK;
        case CKKS_OP_RESCALE:  // last-limb coefficients [b][2][N] + converted part [b][2][ell-1][N]
            if (v->L < 2) return fail(v, CKKS_EINVAL, "rescale needs at least two limbs");
            *bytes = ((size_t)batch_or_nrot * 2 * v->L * sizeof(u64)) << v->logN;
            return CKKS_OK;
    }
    return fail(v, CKKS_EINVAL, "unknown op selector");
}

static const View* view_at(const ckks_ctx* ctx, uint32_t level) {
    if (level == 0 || level > ctx->L) {
        ctx->sh.err = "level must be between 1 and L";
        return nullptr;
    }
    return &ctx->level[level];
}

extern "C" int ckks_workspace_bytes_at(const ckks_ctx* ctx, int op, uint32_t level, uint32_t batch_or_nrot,
                                       size_t* bytes) {
    if (!ctx || !bytes) return CKKS_EINVAL;
    const View* v = view_at(ctx, level);
    if (!v) return CKKS_EINVAL;
    return view_workspace_bytes(v, op, batch_or_nrot, bytes);
}

extern "C" int ckks_workspace_bytes(const ckks_ctx* ctx, int op, uint32_t batch_or_nrot, size_t* bytes) {
    if (!ctx) return CKKS_EINVAL;
    return ckks_workspace_bytes_at(ctx, op, ctx->L, batch_or_nrot, bytes);
}

// --------------------------------------------------------------------------- entry points
static int check_limb_range(const View* c, u32 prime_first, u32 n_limbs, u32 batch) {
    if (n_limbs == 0 || batch == 0) return fail(c, CKKS_EINVAL, "n_limbs and batch must be positive");
    if ((u64)prime_first + n_limbs > c->D) return fail(c, CKKS_EINVAL, "limb range exceeds the prime chain");
    if ((u64)n_limbs * batch > (1u << 20)) return fail(c, CKKS_EINVAL, "batch too large");
    return CKKS_OK;
}

static int ntt_entry(ckks_ctx* ctx, uint64_t* d_x, uint32_t prime_first, uint32_t n_limbs, uint32_t batch,
                     void* stream, bool inverse) {
    if (!ctx) return CKKS_EINVAL;
    const View* c = ctx->full();
    if (!d_x || misaligned(d_x, 16)) return fail(c, CKKS_EINVAL, "d_x is null or not 16-byte aligned");
    int rc = check_limb_range(c, prime_first, n_limbs, batch);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    const LimbSel sel = {n_limbs, batch, n_limbs, 0, prime_first};
    if (!inverse) {
        launch_forward(c, d_x, sel, s);
    } else {
        InvContigArgs a1 = {d_x, nullptr, d_x, sel, sel, {1}, 0};
        launch_inverse<INV_PLAIN>(c, a1, SC_PLAIN, SRC_CANON, s);
    }
    return hip_check(c, inverse ? "ckks_intt" : "ckks_ntt");
}

extern "C" int ckks_ntt(ckks_ctx* ctx, uint64_t* d_x, uint32_t prime_first, uint32_t n_limbs, uint32_t batch,
                        void* stream) {
    return ntt_entry(ctx, d_x, prime_first, n_limbs, batch, stream, false);
}

extern "C" int ckks_intt(ckks_ctx* ctx, uint64_t* d_x, uint32_t prime_first, uint32_t n_limbs, uint32_t batch,
                         void* stream) {
    return ntt_entry(ctx, d_x, prime_first, n_limbs, batch, stream, true);
}

static int check_ks_ctx(const View* c, u32 batch) {
    if (c->K == 0) return fail(c, CKKS_EUNSUPPORTED, "context has no special primes");
    if (batch == 0 || batch > 4096) return fail(c, CKKS_EINVAL, "batch out of range");
    return CKKS_OK;
}

extern "C" int ckks_modup(ckks_ctx* ctx, const uint64_t* d_in, uint64_t* d_out, uint32_t batch, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    const View* c = ctx->full();
    if (!d_in || !d_out || misaligned(d_in, 16) || misaligned(d_out, 16))
        return fail(c, CKKS_EINVAL, "null or misaligned buffer");
    int rc = check_ks_ctx(c, batch);
    if (rc) return rc;
    launch_modup(c, d_in, d_out, batch, (hipStream_t)stream);
    return hip_check(c, "ckks_modup");
}

extern "C" int ckks_moddown(ckks_ctx* ctx, const uint64_t* d_in, uint64_t* d_out, uint32_t batch, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    const View* c = ctx->full();
    if (!d_in || !d_out || misaligned(d_in, 16) || misaligned(d_out, 16))
        return fail(c, CKKS_EINVAL, "null or misaligned buffer");
    int rc = check_ks_ctx(c, batch);
    if (rc) return rc;
    launch_moddown(c, d_in, d_out, batch, (hipStream_t)stream);
    return hip_check(c, "ckks_moddown");
}

static int check_galois(const View* c, u32 g) {
    if ((g & 1) == 0 || g >= (2u << c->logN)) return fail(c, CKKS_EINVAL, "Galois element must be odd and below 2N");
    return CKKS_OK;
}

extern "C" int ckks_automorph(ckks_ctx* ctx, const uint64_t* d_in, uint64_t* d_out, uint32_t prime_first,
                              uint32_t n_limbs, uint32_t galois, int eval_domain, uint32_t batch, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    const View* c = ctx->full();
    if (!d_in || !d_out || misaligned(d_in, 16) || misaligned(d_out, 16))
        return fail(c, CKKS_EINVAL, "null or misaligned buffer");
    if (d_in == d_out) return fail(c, CKKS_EINVAL, "automorphism cannot run in place");
    int rc = check_limb_range(c, prime_first, n_limbs, batch);
    if (rc) return rc;
    rc = check_galois(c, galois);
    if (rc) return rc;
    if (batch > 65535) return fail(c, CKKS_EINVAL, "batch too large");
    const dim3 grid((1u << c->logN) / 256, n_limbs, batch), block(256);
    hipStream_t s = (hipStream_t)stream;
    ProfScope ps(c, std::string(eval_domain ? "automorph_eval_kernel" : "automorph_coeff_kernel"), (u64)batch * n_limbs * 2, s);
    if (eval_domain) {
        hipLaunchKernelGGL(automorph_eval_kernel, grid, block, 0, s, d_in, d_out, c->logN, n_limbs, galois);
    } else {
        // inverse of g modulo 2N (a power of two): Newton iteration on 32-bit words, then mask
        u32 inv = galois;
        for (int i = 0; i < 5; i++) inv *= 2 - galois * inv;
        inv &= (2u << c->logN) - 1;
        hipLaunchKernelGGL(automorph_coeff_kernel, grid, block, 0, s, d_in, d_out, c->tb.pc, c->logN, n_limbs,
                           prime_first, inv);
    }
    return hip_check(c, "ckks_automorph");
}

extern "C" int ckks_pointwise(ckks_ctx* ctx, int op, const uint64_t* d_a, const uint64_t* d_b, uint64_t* d_out,
                              uint32_t prime_first, uint32_t n_limbs, uint32_t batch, uint32_t b_period, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    const View* c = ctx->full();
    if (!d_a || !d_b || !d_out || misaligned(d_a, 16) || misaligned(d_b, 16) || misaligned(d_out, 16))
        return fail(c, CKKS_EINVAL, "null or misaligned buffer");
    if (op < CKKS_PW_ADD || op > CKKS_PW_MAC) return fail(c, CKKS_EINVAL, "unknown limb-wise operation");
    int rc = check_limb_range(c, prime_first, n_limbs, batch);
    if (rc) return rc;
    if (batch > 65535) return fail(c, CKKS_EINVAL, "batch too large");
    if (b_period == 0 || b_period > batch) return fail(c, CKKS_EINVAL, "b_period must be in 1..batch");
    const dim3 grid((1u << c->logN) / 512, n_limbs, batch), block(256);
    hipStream_t s = (hipStream_t)stream;
    static const char* const names[4] = {"pointwise_kernel<add>", "pointwise_kernel<sub>", "pointwise_kernel<mul>",
                                         "pointwise_kernel<mac>"};
    ProfScope ps(c, std::string(names[op]), (u64)batch * n_limbs * (op == CKKS_PW_MAC ? 3 : 2) + (u64)b_period * n_limbs, s);
    switch (op) {
        case CKKS_PW_ADD:
            hipLaunchKernelGGL(pointwise_kernel<PW_ADD>, grid, block, 0, s, d_a, d_b, d_out, c->tb.pc, c->logN, n_limbs,
                               prime_first, b_period);
            break;
        case CKKS_PW_SUB:
            hipLaunchKernelGGL(pointwise_kernel<PW_SUB>, grid, block, 0, s, d_a, d_b, d_out, c->tb.pc, c->logN, n_limbs,
                               prime_first, b_period);
            break;
        case CKKS_PW_MUL:
            hipLaunchKernelGGL(pointwise_kernel<PW_MUL>, grid, block, 0, s, d_a, d_b, d_out, c->tb.pc, c->logN, n_limbs,
                               prime_first, b_period);
            break;
        default:
            hipLaunchKernelGGL(pointwise_kernel<PW_MAC>, grid, block, 0, s, d_a, d_b, d_out, c->tb.pc, c->logN, n_limbs,
                               prime_first, b_period);
            break;
    }
    return hip_check(c, "ckks_pointwise");
}

// [p, p + bytes) ranges that share at least one byte
static inline bool ranges_overlap(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a && b && a0 < b0 + b_bytes && b0 < a0 + a_bytes;
}
// The kernels of a call read the inputs (permuted gathers, tensor terms, later chunks of rotations) after the
// first words of the output have been written, so an output that shares memory with an input, or an output or
// input that shares memory with the workspace, gives wrong words without any error: rejected here.
static int check_no_alias(const View* c, const void* out, size_t out_bytes, const void* in1, size_t in1_bytes,
                          const void* in2, size_t in2_bytes, const void* ws, size_t ws_bytes) {
    if (ranges_overlap(out, out_bytes, in1, in1_bytes) || ranges_overlap(out, out_bytes, in2, in2_bytes))
        return fail(c, CKKS_EINVAL, "output overlaps an input");
    if (ranges_overlap(out, out_bytes, ws, ws_bytes) || ranges_overlap(in1, in1_bytes, ws, ws_bytes) ||
        ranges_overlap(in2, in2_bytes, ws, ws_bytes))
        return fail(c, CKKS_EINVAL, "workspace overlaps an operand");
    return CKKS_OK;
}
static inline size_t limb_bytes(const View* c, size_t limbs) { return (limbs * sizeof(u64)) << c->logN; }

static int check_ks_args(const View* c, const void* a, const void* b, const void* out, u32 batch, int op,
                         const void* ws, size_t ws_bytes) {
    if (!a || !b || !out || misaligned(a, 16) || misaligned(b, 16) || misaligned(out, 16))
        return fail(c, CKKS_EINVAL, "null or misaligned buffer");
    int rc = check_ks_ctx(c, batch);
    if (rc) return rc;
    if (!ws || misaligned(ws, 256)) return fail(c, CKKS_EINVAL, "workspace is null or not 256-byte aligned");
    size_t need = 0;
    rc = view_workspace_bytes(c, op, batch, &need);
    if (rc) return rc;
    if (ws_bytes < need) return fail(c, CKKS_ENOMEM, "workspace too small");
    return CKKS_OK;
}

// Conversions from a single limb on small grids: the inverse pass that leaves the source's words is repeated by the workgroup of every
// target, a launch and a round trip less.  Counted in workgroups of a tile and a target.  Calls before / with it, us:
// ModUp (digits of one limb; both arithmetics' targets share the launch too), HMult with K = 1 as a whole: N = 2^12, 3 + 1 limbs (12
// workgroups) 52.8 / 43.2, 35-bit primes 36.8 / 32.1, 12 + 1, 2 ciphertexts (312) 78.7 / 70.6; N = 2^13, 3 + 1 (24) 61.6 / 52.2, 12 + 1, 2
// (624) 92.2 / 87.6 (1000 and more: worse); N = 2^14, 3 + 1 (48) 63.0 / 52.2, 5 + 1, 4 (480) 75.4 / 68.8; N = 2^16, 3 + 1 (192) 71.5 / 59.8;
// all of 55 bits 3 to 7 % of the call.  N = 2^14 .. 2^16, 2 to 15 limbs, HMult and HRot, before / with it as a quotient: 320 to 480 workgroups 1.08 to
// 1.13 (50-bit limbs, 60-bit special limb), 1.03 to 1.06 (36 bits), 1.00 to 1.03 (all of 55 bits and more); 528 to 600 1.03 to 1.08, 1.00 to 1.03 and 0.98
// to 1.00; 720 and 768 1.05 to 1.09, 1.00 to 1.04, 0.98 to 1.00; 960 1.02 to 1.07, 0.99 to 1.02, 0.96 to 0.99.  One line for all of them, two workgroups
// to a compute unit, where the first of them begin to lose.
static bool up_with_inverse(const View* c, u32 batch) {
    return !c->up.ks && !c->sh->side.active && batch * c->dnum * c->D * tiles_of(c) <= (c->logN <= 13 ? 640u : 512u);
}
// ModDown by one prime.  After an inner product, which has run the first inverse pass: HMult with digits of two limbs, N = 2^12, 6 + 1 limbs (12)
// 59.0 / 57.2, N = 2^16, 6 + 1 (192) 79.6 / 75.7, 8 + 1, 3 ciphertexts (768) 124.3 / 124.9 (an integer special prime).  Rescale: N = 2^14, 24 -> 23
// limbs (192) 22.7 / 19.4, N = 2^16, 7 limbs (192) 24.3 / 20.7, 25 (768) 36.4 / 35.1, 17, 2 ciphertexts (1024) 42.0 / 41.6, 3 (1536) 55 / 57.
// Those are targets of one arithmetic.  Targets of both take a launch for every run of one, and each repeats the pass: two runs from an FpAr source,
// rescales of 4 to 20 targets, N = 2^14 .. 2^16, up to 512 workgroups 1.05 to 1.09 of the time with it, 576 to 768 0.99 to 1.04; from an
// integer source 0.97 to 1.02 and 0.91 to 0.97 (behind an inner product at N = 2^12 and 2^13 1.00 to 1.02); three runs 0.98 to 1.03 and 0.90 to
// 0.97; four 0.97 to 1.00 and 0.88 to 0.93; primes in turn 0.79 to 1.0 (N = 2^14, 12 limbs, 49 and 55 bits, 4 ciphertexts 225 / 247 us).
// whole: both passes in one workgroup, whose launch serves every target: N = 2^12, 17 limbs, 2 (64) 18.6 / 15.5, 23, 9 (396) 26.7 / 26.0 (528: 30.6 / 31.1);
// N = 2^13, 23, 3 (264) 26.0 / 23.3 (400: 28.0 / 31.7), few integer limbs 31.3 / 32.8 (spread_limbs: two passes are the faster ones there).
static bool dn_with_inverse(const View* c, u32 sources, bool whole) {
    if (c->K != 1 || c->sh->side.active) return false;
    const u32 tiles = sources * tiles_of(c);
    const bool integer = c->primes[c->L] >= CKKS_FP_PRIME_LIMIT;
    u32 most = c->logN == 12 ? 448 : 288;
    if (!whole) {
        const size_t runs = class_runs(c, 0, c->L).size();
        most = runs == 1 ? (integer ? 512 : 768) : runs == 2 && (!integer || c->logN <= 13) ? 512 : 0;
    }
    return tiles * c->L <= most && tiles * cdiv(c->L, 4) < 512;  // fewer than 512: launch_conv takes single targets
}
template <int LOAD, int DIR>
static void launch_inv_whole_conv_one(const View* c, InvContigArgs a, u64* dst, hipStream_t s) {
    const u32 sources = a.sel.n_inst * a.sel.n_l, targets = DIR == CONV_UP ? c->D : c->L;
    a.scale = DIR == CONV_UP ? SC_UP : SC_DN, a.out_fmt = SRC_CANON;
    ProfScope ps(c, c->sh->prof.on ? "inv_whole_conv_one_kernel<" + std::to_string((int)c->logN - 8) + ", " + std::to_string(LOAD) + ", " + std::to_string(DIR) + ">" : std::string(),
                 (u64)sources * (targets + (LOAD == INV_TENSOR ? 2 : 1)), s);
    const dim3 grid(xcd_grid(sources, targets));
    if (c->logN == 12) hipLaunchKernelGGL((inv_whole_conv_one_kernel<4, LOAD, DIR>), grid, dim3(256), 0, s, a, dst, c->tb);
    else hipLaunchKernelGGL((inv_whole_conv_one_kernel<5, LOAD, DIR>), grid, dim3(512), 0, s, a, dst, c->tb);
}

// ModUp side shared by every key switch: w.x holds the coefficients of the polynomial(s) times the conversion pre-factor
// (launch_decompose_inverse); conversion fused into the first forward pass of every extended limb.
template <int LOAD>
static void launch_decompose_inverse(const View* c, const InvContigArgs& a, hipStream_t s) {
    launch_inverse<LOAD>(c, a, SC_UP, conv_src_fmt(c->up, CONV_UP), s);
}
// What follows the ModUp: PLAIN on one stream; BESIDE the FpAr targets may run on the side stream (keyswitch_pipeline); FORK the
// integer limbs take the side stream from here on.
enum ExtendMode { EXTEND_PLAIN, EXTEND_BESIDE, EXTEND_FORK };
static void decompose_extend(const View* c, const Workspace& w, u32 groups, hipStream_t s, ExtendMode mode) {
    const ConvArgs a3 = {w.x, w.dt, groups, 0, nullptr, nullptr, 0, 0};
    SideStream& sd = c->sh->side;
    const bool second = mode != EXTEND_PLAIN && sd.enabled && c->mixed_classes;
    if (conv_up_both(c, a3, s, !second ? 4095 : mode == EXTEND_BESIDE ? 1024 : 512)) {  // before a fork: what follows on either stream comes after it
        if (mode == EXTEND_FORK) fork_side(c, s);
        return;
    }
    // below 512 workgroups the events cost more than the second stream gives (N = 2^13, 24 + 6 limbs, overlap on, HMult of 4 (256) 110 us
    // forked, 99 on one stream; 8 (512) 128 / 131; N = 2^12, 3 + 1 limbs, one 72 / 53), unless a workgroup takes long: more than eight
    // sources (N = 2^13, 92 + 5 limbs, 9 digits, one rotation (432) 0.87 of the time on one stream; N = 2^12, 57 + 5, 5 digits, 4 (300) 0.88)
    const bool worth = c->up.ks >= 4 || conv_up_workgroups(c, groups) >= 512;
    if (mode == EXTEND_BESIDE && second && !sd.active && worth && side_stream_ready(sd)) {
        // the IntAr targets first, on s; the FpAr targets on the side stream from the moment those are done, beside
        // whatever s runs next (the caller joins before it reads the FpAr limbs of dt)
        launch_conv<CONV_UP>(c, a3, s, 0);
        hipEvent_t e = side_event(sd);
        if (e && hipEventRecord(e, s) == hipSuccess && hipStreamWaitEvent(sd.stream, e, 0) == hipSuccess) {
            launch_conv<CONV_UP>(c, a3, sd.stream, 1);
            sd.fp_pending = true;
            return;
        }
        (void)hipGetLastError();
        launch_conv<CONV_UP>(c, a3, s, 1);
        return;
    }
    if (mode == EXTEND_FORK) fork_side(c, s);
    launch_conv<CONV_UP>(c, a3, s);
}

// Both: a's limbs into their extended digits
template <int LOAD>
static void decompose(const View* c, const InvContigArgs& a, const Workspace& w, hipStream_t s, ExtendMode mode) {
    const u32 groups = a.sel.n_inst;
    if (!up_with_inverse(c, groups) || (LOAD == INV_PLAIN && spread_limbs(c, a.sel, 24))) {
        launch_decompose_inverse<LOAD>(c, a, s);
        decompose_extend(c, w, groups, s, mode);
        return;
    }
    if (inv_one_kernel((int)c->logN - 8)) {
        launch_inv_whole_conv_one<LOAD, CONV_UP>(c, a, w.dt, s);
    } else {
        launch_inv_contig<LOAD>(c, a, s);
        ProfScope ps(c, c->sh->prof.on ? "inv_conv_one_kernel<" + std::to_string((int)c->logN - 8) + ">" : std::string(), (u64)groups * c->L * (c->D + 1), s);
        const dim3 grid(xcd_grid(groups * c->dnum * tiles_of(c), c->D));
        const ConvArgs a3 = {w.x, w.dt, groups, 0, nullptr, nullptr, 0, 0};
        switch (c->logN) {
            case 14: hipLaunchKernelGGL(inv_conv_one_kernel<6>, grid, dim3(256), 0, s, a3, c->tb); break;
            case 15: hipLaunchKernelGGL(inv_conv_one_kernel<7>, grid, dim3(256), 0, s, a3, c->tb); break;
            case 16: hipLaunchKernelGGL(inv_conv_one_kernel<8>, grid, dim3(256), 0, s, a3, c->tb); break;
        }
    }
    if (mode == EXTEND_FORK) fork_side(c, s);
}

// s waits for the FpAr conversion that decompose_extend put on the side stream
static void join_fp_beside(const View* c, hipStream_t s) {
    SideStream& sd = c->sh->side;
    if (!sd.fp_pending) return;
    sd.fp_pending = false;
    hipEvent_t e = side_event(sd);
    if (!e || hipEventRecord(e, sd.stream) != hipSuccess || hipStreamWaitEvent(s, e, 0) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipStreamSynchronize(sd.stream);
    }
}

// ModDown side: w.cp holds c' on the special limbs after the first inverse pass (done = false) or as coefficients times the
// conversion pre-factor.  cached: the converted part, from a single source, is stored with ordinary accesses (stores_cached).
static void moddown_convert(const View* c, const Workspace& w, u32 cg, hipStream_t s, bool done = false, bool cached = false) {
    const bool inverse = !done && dn_with_inverse(c, cg * 2, false);
    if (!done && !inverse) {
        const InvStridedArgs a6 = {w.cp, LimbSel{c->K, cg * 2, c->K, 0, c->L}, SC_DN, conv_src_fmt(c->dn, CONV_DN)};
        launch_inv_strided(c, a6, s);
    }
    join_side(c, s);  // the conversion reads every special limb
    const ConvArgs a7 = {w.cp, w.cv, cg * 2, 0, nullptr, nullptr, 0, inverse};
    if (cached) launch_conv_runs<ConvOneCachedL, CONV_DN>(c, a7, s, -1);
    else launch_conv<CONV_DN>(c, a7, s);
}

// the same from the special limbs in evaluation form, a's source: their inverse transform into w.cp and the conversion
static void moddown_from_eval(const View* c, const InvContigArgs& a, const Workspace& w, u32 cg, hipStream_t s, bool cached = false) {
    const bool whole = inv_one_kernel((int)c->logN - 8);
    if (!dn_with_inverse(c, cg * 2, whole) || spread_limbs(c, a.sel, 24)) {
        launch_inverse<INV_PLAIN>(c, a, SC_DN, conv_src_fmt(c->dn, CONV_DN), s);
        moddown_convert(c, w, cg, s, true, cached);
    } else if (whole) {
        launch_inv_whole_conv_one<INV_PLAIN, CONV_DN>(c, a, w.cv, s);
    } else {
        launch_inv_contig<INV_PLAIN>(c, a, s);
        moddown_convert(c, w, cg, s);
    }
}

// second forward pass of every extended digit of one decomposition
static void launch_extended_fwd_contig(const View* c, const Workspace& w, hipStream_t s) {
    const FwdContigArgs a = {w.dt, LimbSel{c->D, c->dnum, c->D, 0, 0}, c->alpha, c->L};
    launch_fwd_contig(c, a, s);
}

// most rotations whose special parts may be added as integers: the eight digits of a conversion's source word hold the sum
static u32 summed_rotations_max(const View* c) {
    u64 most = 0;
    for (u32 i = c->L; i < c->D; i++) most = c->primes[i] > most ? c->primes[i] : most;
    const u64 fit = CKKS_DIGIT_MAX / most;
    return fit < CKKS_ROT_CHUNK ? (u32)fit : CKKS_ROT_CHUNK;
}

// Giant rotations with one ModDown (summed_rotations) instead of as a batch: conversions, inverse pass, q-limb product and sum of 8 x 4 at
// N = 2^16, 24 + 6 limbs 300 -> 241 us.  But a workgroup of the q-limb product then runs over the digits of all of them, and what does not
// fit one sum (3 rotations near 2^61, 7 just above 2^60, 15 at 2^59) starts over.  Batch / sum, whole transforms of 2 to 21 giant steps, by
// the workgroups of the smallest q-limb launch, N = 2^12 .. 2^16: up to 64 0.60 to 1.01 (runs of one limb, the arithmetics alternating, 0.42 to 0.92), 72 and
// 80 0.97 to 1.05, 96 and more 0.98 to 1.20, one giant step 0.94 to 1.0; where the sums are more than the launches of a batch: 96 0.89 to 0.99, 144 and
// 160 0.92 to 1.0, 192 0.97 to 1.05, 256 and more 1.0 to 1.12, but three a sum 0.78 to 1.02 up to 560.  And never where the q-limb
// product by itself, in the units of inner_ways, would take more than 5/4 of the batch's (3 steps, 70 + 14 integer limbs in 24 digits,
// N = 2^13, 140 workgroups: 75 against 52 units, the transform with 2 baby steps 1127 against 993 us; 20 + 4 limbs in 5 digits, N = 2^15, 19 / 14, the call 0.98)
static bool giants_summed(const View* c, u32 n) {
    if (n < 2 || !c->dn.ks) return false;  // one special prime is reduced directly: there are no digits to add
    const u32 at_once = summed_rotations_max(c), sums = cdiv(n, at_once);
    u32 least = ~0u, one = 0, batch = 0, t;
    for (const ClassRun& r : class_runs(c, 0, c->L)) {
        const u32 wgs = r.count * tiles_of(c);
        if (wgs < least) least = wgs;
        inner_ways(wgs, cdiv(n, sums) * c->dnum, t), one += t;
        inner_ways(wgs * n, c->dnum, t), batch += t;
    }
    if (4 * sums * one > 5 * batch) return false;
    return sums == cdiv(n, CKKS_ROT_CHUNK) ? least >= 96 : least >= 192 && at_once >= 6;
}

// out = the sum of n (at most CKKS_ROT_CHUNK) rotated ciphertexts, each with its own element and key
static void summed_rotations(const View* c, const u64* in, u32 n, const u32* galois, const u64* const* keys, u64* out, void* ws, hipStream_t s) {
    const Workspace w = carve(c, ws, n, n, n, false);
    const LimbSel sel = {c->L, n, c->L, 0, 0};
    InvContigArgs a1;
    memset(&a1, 0, sizeof(a1));
    a1.src = in, a1.dst = w.x, a1.sel = sel, a1.dsel = sel, a1.per_inst = 1;
    InnerArgs ia;
    memset(&ia, 0, sizeof(ia));
    ia.dt = w.dt, ia.own = in, ia.cp = w.cp, ia.n_inst = n, ia.split = c->L, ia.per_inst = 1;
    for (u32 g = 0; g < n; g++) a1.galois[g] = ia.galois[g] = galois[g], ia.key[g] = keys[g];
    decompose<INV_ROT>(c, a1, w, s, EXTEND_BESIDE);
    if (any_fp_prime(c, c->L, c->D)) join_fp_beside(c, s);  // as in keyswitch_pipeline
    launch_ks_inner<OWN_COPY, false, false>(c, ia, s, c->L, c->D);
    const InvStridedSumArgs a2 = {w.cp, LimbSel{c->K, 2, c->K, 0, c->L}, SC_DN, n};
    launch_runs<InvStridedSumL>(c, c->L, c->D, c->L, tiles_of(c), 2, a2, s, [n](u32, u32 limbs) { return (u64)2 * limbs * (n + 1); });
    moddown_convert(c, w, 1, s, true);
    ia.cv = w.cv, ia.out = out, ia.fin_pinv = c->tb.pinv, ia.n_inst = 1, ia.n_sum = n;
    join_fp_beside(c, s);
    launch_ks_inner<OWN_ROT_SUM, false, true>(c, ia, s, 0, c->L);
}

// cm: the view whose ModDown ends the pipeline: c itself, or the merged view of c's level (the ModDown then
// also divides by the last q-limb: limb c->L - 1 joins the special limbs and the output has c->L - 1 limbs)
// multi_galois / multi_keys (rotations only, batch <= CKKS_ROT_CHUNK): one Galois element and key per instance.
template <int LOAD, int OWN>
static void keyswitch_pipeline(const View* c, const View* cm, const u64* in1, const u64* in2, const u64* key, u64* out,
                               u32 batch, u32 galois, void* ws, hipStream_t s, const u32* multi_galois = nullptr,
                               const u64* const* multi_keys = nullptr) {
    Workspace w = carve(c, ws, batch, batch, batch, false);
    if (cm != c)  // cv shrinks by one limb per component, cp grows by one: still inside the level's workspace
        w.cv = w.cp + ((size_t)batch * 2 * cm->K << c->logN);
    const LimbSel sel = {c->L, batch, c->L, 0, 0};
    InvContigArgs a1;
    memset(&a1, 0, sizeof(a1));
    a1.src = in1, a1.src2 = in2, a1.dst = w.x, a1.sel = sel, a1.dsel = sel, a1.galois[0] = galois;
    InnerArgs ia;
    memset(&ia, 0, sizeof(ia));
    ia.key[0] = key, ia.galois[0] = galois;
    if (multi_galois) {
        a1.per_inst = ia.per_inst = 1;
        for (u32 b = 0; b < batch; b++)
            a1.galois[b] = ia.galois[b] = multi_galois[b], ia.key[b] = multi_keys[b];
    }
    decompose<LOAD>(c, a1, w, s, EXTEND_BESIDE);
    ia.dt = w.dt, ia.own = in1, ia.own2 = in2;
    ia.cp = w.cp, ia.n_inst = batch, ia.split = cm->L;
    // the limbs that feed the ModDown conversion first; the q-limbs then finish in one kernel, c' in registers.
    // Those of them that are FpAr primes (special primes below the FP64 limit; limb cm->L of the merged rescale) take
    // their digits from the FpAr conversion, which may still be running on the side stream.
    if (any_fp_prime(c, cm->L, c->D)) join_fp_beside(c, s);
    if (cm != c) {
        launch_ks_inner<OWN, false, false>(c, ia, s, cm->L, c->D);
    } else {
        // special limbs belong to no digit, so every variant computes the same on them: the leanest one runs
        launch_ks_inner<OWN_COPY, false, false>(c, ia, s, c->L, c->D);
    }
    moddown_convert(cm, w, batch, s);
    ia.cv = w.cv, ia.out = out, ia.fin_pinv = cm->tb.pinv;
    join_fp_beside(c, s);
    launch_ks_inner<OWN, false, true>(c, ia, s, 0, cm->L);
}

extern "C" int ckks_keyswitch_at(ckks_ctx* ctx, uint32_t level, const uint64_t* d_d, const uint64_t* d_key,
                                 uint64_t* d_out, uint32_t batch, void* d_ws, size_t ws_bytes, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    const View* c = view_at(ctx, level);
    if (!c) return CKKS_EINVAL;
    int rc = check_ks_args(c, d_d, d_key, d_out, batch, CKKS_OP_KEYSWITCH, d_ws, ws_bytes);
    if (rc) return rc;
    rc = check_no_alias(c, d_out, limb_bytes(c, (size_t)batch * 2 * c->L), d_d, limb_bytes(c, (size_t)batch * c->L), nullptr, 0,
                        d_ws, ws_bytes);
    if (rc) return rc;
    keyswitch_pipeline<INV_PLAIN, OWN_COPY>(c, c, d_d, nullptr, d_key, d_out, batch, 1, d_ws, (hipStream_t)stream);
    return hip_check(c, "ckks_keyswitch");
}

extern "C" int ckks_hmult_relin_at(ckks_ctx* ctx, uint32_t level, const uint64_t* d_ct1, const uint64_t* d_ct2,
                                   const uint64_t* d_evk, uint64_t* d_out, uint32_t batch, void* d_ws, size_t ws_bytes,
                                   void* stream) {
    if (!ctx) return CKKS_EINVAL;
    const View* c = view_at(ctx, level);
    if (!c) return CKKS_EINVAL;
    if (!d_ct2 || misaligned(d_ct2, 16)) return fail(c, CKKS_EINVAL, "null or misaligned buffer");
    int rc = check_ks_args(c, d_ct1, d_evk, d_out, batch, CKKS_OP_HMULT_RELIN, d_ws, ws_bytes);
    if (rc) return rc;
    const size_t ctb = limb_bytes(c, (size_t)batch * 2 * c->L);
    rc = check_no_alias(c, d_out, ctb, d_ct1, ctb, d_ct2, ctb, d_ws, ws_bytes);
    if (rc) return rc;
    keyswitch_pipeline<INV_TENSOR, OWN_TENSOR>(c, c, d_ct1, d_ct2, d_evk, d_out, batch, 1, d_ws,
                                                          (hipStream_t)stream);
    return hip_check(c, "ckks_hmult_relin");
}

extern "C" int ckks_hmult_relin_rescale_at(ckks_ctx* ctx, uint32_t level, const uint64_t* d_ct1, const uint64_t* d_ct2,
                                           const uint64_t* d_evk, uint64_t* d_out, uint32_t batch, void* d_ws,
                                           size_t ws_bytes, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    const View* c = view_at(ctx, level);
    if (!c) return CKKS_EINVAL;
    if (level < 2) return fail(c, CKKS_EINVAL, "rescale needs at least two limbs");
    if (!d_ct2 || misaligned(d_ct2, 16)) return fail(c, CKKS_EINVAL, "null or misaligned buffer");
    int rc = check_ks_args(c, d_ct1, d_evk, d_out, batch, CKKS_OP_HMULT_RELIN, d_ws, ws_bytes);
    if (rc) return rc;
    const size_t ctb = limb_bytes(c, (size_t)batch * 2 * c->L);
    rc = check_no_alias(c, d_out, limb_bytes(c, (size_t)batch * 2 * (c->L - 1)), d_ct1, ctb, d_ct2, ctb, d_ws, ws_bytes);
    if (rc) return rc;
    keyswitch_pipeline<INV_TENSOR, OWN_TENSOR>(c, &ctx->merged[level], d_ct1, d_ct2, d_evk, d_out, batch, 1,
                                                             d_ws, (hipStream_t)stream);
    return hip_check(c, "ckks_hmult_relin_rescale");
}

extern "C" int ckks_hrot_at(ckks_ctx* ctx, uint32_t level, const uint64_t* d_ct, uint32_t galois, const uint64_t* d_rk,
                            uint64_t* d_out, uint32_t batch, void* d_ws, size_t ws_bytes, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    const View* c = view_at(ctx, level);
    if (!c) return CKKS_EINVAL;
    int rc = check_ks_args(c, d_ct, d_rk, d_out, batch, CKKS_OP_HROT, d_ws, ws_bytes);
    if (rc) return rc;
    rc = check_galois(c, galois);
    if (rc) return rc;
    const size_t ctb = limb_bytes(c, (size_t)batch * 2 * c->L);
    rc = check_no_alias(c, d_out, ctb, d_ct, ctb, nullptr, 0, d_ws, ws_bytes);
    if (rc) return rc;
    keyswitch_pipeline<INV_ROT, OWN_ROT>(c, c, d_ct, nullptr, d_rk, d_out, batch, galois, d_ws,
                                                   (hipStream_t)stream);
    return hip_check(c, "ckks_hrot");
}

extern "C" int ckks_keyswitch(ckks_ctx* ctx, const uint64_t* d_d, const uint64_t* d_key, uint64_t* d_out,
                              uint32_t batch, void* d_ws, size_t ws_bytes, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    return ckks_keyswitch_at(ctx, ctx->L, d_d, d_key, d_out, batch, d_ws, ws_bytes, stream);
}

extern "C" int ckks_hmult_relin(ckks_ctx* ctx, const uint64_t* d_ct1, const uint64_t* d_ct2, const uint64_t* d_evk,
                                uint64_t* d_out, uint32_t batch, void* d_ws, size_t ws_bytes, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    return ckks_hmult_relin_at(ctx, ctx->L, d_ct1, d_ct2, d_evk, d_out, batch, d_ws, ws_bytes, stream);
}

extern "C" int ckks_hrot(ckks_ctx* ctx, const uint64_t* d_ct, uint32_t galois, const uint64_t* d_rk, uint64_t* d_out,
                         uint32_t batch, void* d_ws, size_t ws_bytes, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    return ckks_hrot_at(ctx, ctx->L, d_ct, galois, d_rk, d_out, batch, d_ws, ws_bytes, stream);
}

// Rescale = a ModDown whose only special prime is the last active limb: inverse transform of that
// limb, reduction modulo every remaining prime fused into their first forward pass, second forward
// pass fused with (c_i - .) * q_last^-1.
static int rescale_impl(ckks_ctx* ctx, uint32_t level, const uint64_t* d_ct, uint64_t* d_out, uint32_t batch,
                        void* d_ws, size_t ws_bytes, void* stream, bool static_scratch) {
    if (!ctx) return CKKS_EINVAL;
    if (level < 2 || level > ctx->L) return fail(ctx, CKKS_EINVAL, "rescale needs a level between 2 and L");
    const View* c = &ctx->rescale[level];  // c->L = level - 1 targets, c->K = 1
    if (!d_ct || !d_out || misaligned(d_ct, 16) || misaligned(d_out, 16))
        return fail(c, CKKS_EINVAL, "null or misaligned buffer");
    if (batch == 0 || batch > 4096) return fail(c, CKKS_EINVAL, "batch out of range");
    if (!d_ws || misaligned(d_ws, 256)) return fail(c, CKKS_EINVAL, "workspace is null or not 256-byte aligned");
    const size_t N = (size_t)1 << c->logN;
    if (ws_bytes < (size_t)batch * 2 * level * N * sizeof(u64))
        return fail(c, CKKS_ENOMEM, static_scratch ? "batch * 2 * level * N words exceed CKKS_STATIC_SCRATCH_BYTES"
                                                   : "workspace too small");
    int rc = check_no_alias(c, d_out, limb_bytes(c, (size_t)batch * 2 * (level - 1)), d_ct, limb_bytes(c, (size_t)batch * 2 * level),
                            nullptr, 0, d_ws, ws_bytes);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    Workspace w;
    w.x = w.dt = w.cq = nullptr;
    w.cp = (u64*)d_ws;                    // [b][2][1][N]
    w.cv = w.cp + (size_t)batch * 2 * N;  // [b][2][level-1][N]
    const LimbSel src = {1, batch * 2, level, level - 1, level - 1};  // limb level-1 of every component
    const LimbSel dst = {1, batch * 2, 1, 0, level - 1};
    InvContigArgs a1 = {d_ct, nullptr, w.cp, src, dst, {1}, 0};
    moddown_from_eval(c, a1, w, batch, s, stores_cached(c, (u64)batch * 2 * c->L));
    FinalArgs fa;
    memset(&fa, 0, sizeof(fa));
    fa.cq = d_ct, fa.cq_L = level, fa.cv = w.cv, fa.out = d_out, fa.n_inst = 2 * batch;
    if (loads_cached(c, (u64)batch * 2 * c->L)) launch_ks_final<FIN_KS, true>(c, fa, s);
    else launch_ks_final<FIN_KS>(c, fa, s);
    return hip_check(c, "ckks_rescale");
}

extern "C" int ckks_rescale(ckks_ctx* ctx, uint32_t level, const uint64_t* d_ct, uint64_t* d_out, uint32_t batch,
                            void* d_ws, size_t ws_bytes, void* stream) {
    return rescale_impl(ctx, level, d_ct, d_out, batch, d_ws, ws_bytes, stream, false);
}

// The same launches with the workspace in this GPU's static scratch array: no allocation of any kind, no
// workspace argument.  Every word of the scratch that the kernels read has been written earlier in the same
// call (last-limb coefficients, then the converted part), so nothing has to be cleared between calls.
extern "C" int ckks_rescale_static(ckks_ctx* ctx, uint32_t level, const uint64_t* d_ct, uint64_t* d_out, uint32_t batch,
                                   void* stream) {
    if (!ctx) return CKKS_EINVAL;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != ctx->device)
        return fail(ctx, CKKS_EINVAL, "the current device is not the one the context was created on");
    return rescale_impl(ctx, level, d_ct, d_out, batch, ctx->scratch_ptr, CKKS_STATIC_SCRATCH_BYTES, stream, true);
}

// Hoisted rotate-MAC: the plaintext products of c' summed before the ModDowns' converted parts join them (FIN_SUMMED), which takes the
// round trip of every rotation's c' away, needs half the ModDown launches, and costs one launch and the joint launch of both
// arithmetics.  Times of the other form / this one, 17 to 40 rotations unless said:
//   chains of integer primes (9 + 1 to 20 + 5 limbs, 1 to 9 digits, N = 2^12 .. 2^16) 1.02 to 1.25, half of them integer 1.2 to 1.36
//   N = 2^16, FP64 limbs: 1.02 to 1.17 for up to 10 digits (20 + 1 limbs, 20 digits 1.06; 30 + 1, 30 1.04); 12, 14, 16 rotations of 9 limbs and
//   more 1.02 to 1.11, of fewer 0.98 to 1.01; N = 2^15, 12, 24 + 6 434 / 440 us
//   smaller rings: the accumulation and the special limbs' launch follow one another where the other form has one launch, each as long as
//   dnum digits take on a few workgroups.  Up to four digits 1.00 to 1.15 (3 + 1 limbs at N = 2^12, four workgroups a rotation:
//   0.97 to 1.01); more: 0.75 to 1.0 below 16 dnum workgroups a rotation (20 + 1, 20 digits, N = 2^12 0.84; 9 + 1, 9, N = 2^14 0.92;
//   20 + 2, 10, N = 2^14 0.95), 0.97 to 1.11 above (10 + 2, 5, N = 2^15 1.01; 24 + 4, 6, N = 2^14 1.02; 20 + 2, 10, N = 2^15 1.04)
static bool hoisted_summed(const View* c, u32 n_rot) {
    if (n_rot <= CKKS_ROT_CHUNK && !(c->logN == 16 && n_rot >= 12 && c->L >= 9)) return false;
    u32 integer = 0;
    for (u32 i = 0; i < c->L; i++) integer += c->primes[i] >= CKKS_FP_PRIME_LIMIT;
    return 2 * integer >= c->L || c->dnum <= 4 || c->D * tiles_of(c) >= 16 * c->dnum;
}

extern "C" int ckks_hrot_hoisted_mac_at(ckks_ctx* ctx, uint32_t level, const uint64_t* d_ct, uint32_t n_rot,
                                        const uint32_t* h_galois, const uint64_t* const* h_rk_ptrs, const uint64_t* d_pt,
                                        uint64_t* d_out, void* d_ws, size_t ws_bytes, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    const View* c = view_at(ctx, level);
    if (!c) return CKKS_EINVAL;
    if (!h_galois || !h_rk_ptrs) return fail(c, CKKS_EINVAL, "null host array");
    if (n_rot == 0 || n_rot > 65535) return fail(c, CKKS_EINVAL, "n_rot out of range");
    if (!d_ct || !d_pt || !d_out || misaligned(d_ct, 16) || misaligned(d_pt, 16) || misaligned(d_out, 16))
        return fail(c, CKKS_EINVAL, "null or misaligned buffer");
    if (!d_ws || misaligned(d_ws, 256)) return fail(c, CKKS_EINVAL, "workspace is null or not 256-byte aligned");
    size_t need = 0;
    int rc = view_workspace_bytes(c, CKKS_OP_HROT_HOISTED_MAC, n_rot, &need);
    if (rc) return rc;
    if (ws_bytes < need) return fail(c, CKKS_ENOMEM, "workspace too small");
    for (u32 r = 0; r < n_rot; r++) {
        if (!h_rk_ptrs[r] || misaligned(h_rk_ptrs[r], 16)) return fail(c, CKKS_EINVAL, "null or misaligned key");
        rc = check_galois(c, h_galois[r]);
        if (rc) return rc;
    }
    rc = check_no_alias(c, d_out, limb_bytes(c, 2 * (size_t)c->L), d_ct, limb_bytes(c, 2 * (size_t)c->L), d_pt,
                        limb_bytes(c, (size_t)n_rot * c->L), d_ws, ws_bytes);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    const size_t N = (size_t)1 << c->logN;
    const SideStream& sd = c->sh->side;
    // decompose a = ct[1] once and finish the transform of every extended limb
    auto decompose_input = [&](const Workspace& w, ExtendMode mode) {
        const LimbSel src = {c->L, 1, c->L, c->L, 0};  // limbs L .. 2L-1 of ct, primes 0 .. L-1
        const LimbSel dst = {c->L, 1, c->L, 0, 0};
        InvContigArgs a1 = {d_ct, nullptr, w.x, src, dst, {1}, 0};
        decompose<INV_PLAIN>(c, a1, w, s, mode);
        launch_extended_fwd_contig(c, w, s);
    };
    if (hoisted_summed(c, n_rot)) {
        // Equal chunks of as many rotations as the workspace has room for: x and dt, then the sum on the q-limbs ([2][L]) and, per
        // rotation, the special limbs ([2][K]) and the converted part ([2][L]).  That of m = min(n_rot, CKKS_ROT_CHUNK) rotations of the other
        // form, L + dnum D + 2 m (2 L + K) limbs, holds (m (2 L + K) - L) / (L + K): m at least, 28 at 24 + 6 limbs, never 2 CKKS_ROT_CHUNK - 1.
        // One launch of the special limbs for a chunk: in two, of equal parts, each ends in a round of workgroups that is half empty
        // (N = 2^16, 24 + 6 limbs: 17 rotations 990 -> 979 us, 18 1043 -> 1020, 24 1331 -> 1303; 16 even).
        Workspace w = carve(c, d_ws, 1, 1, 1);
        u64 *const cq = w.cq, *const cp = cq + (size_t)2 * c->L * N;
        const size_t fit = (need / sizeof(u64) / N - 3 * (size_t)c->L - (size_t)c->dnum * c->D) / (2 * (size_t)c->D);
        static_assert(2 * CKKS_ROT_CHUNK - 2 <= CKKS_DH_CHUNK, "a chunk is one launch");
        const u32 chunk = cdiv(n_rot, cdiv(n_rot, (u32)fit));
        // Second stream: the integer special limbs' inner products and inverse transforms beside the sum on the q-limbs.  Not where the
        // special limbs mix the arithmetics, whose joint launches it would split (one stream / two, us: 40 + 9 limbs, 49, 59 and 60 bits in
        // turn, N = 2^14, 17 rotations 598 / 889, 32 960 / 1281; 24 + 6, N = 2^15, 17 588 / 754, 32 1013 / 1173; all of 59 bits 551 / 546,
        // 954 / 937; 560 / 580, 992 / 1005)
        const bool fork = sd.enabled && c->mixed_classes && class_runs(c, c->L, c->D).size() == 1 &&
                          (n_rot < chunk ? n_rot : chunk) * c->D * tiles_of(c) >= 5 * 512;
        decompose_input(w, fork ? EXTEND_FORK : EXTEND_PLAIN);
        for (u32 r0 = 0; r0 < n_rot; r0 += chunk) {
            const u32 nr = (n_rot - r0) < chunk ? (n_rot - r0) : chunk;
            DhInnerArgs da;
            memset(&da, 0, sizeof(da));
            for (u32 r = 0; r < nr; r++) da.key[r] = h_rk_ptrs[r0 + r], da.galois[r] = h_galois[r0 + r];
            da.dt = w.dt, da.ct = d_ct, da.pt = d_pt + (size_t)r0 * c->L * N, da.pt_limbs = c->L, da.cq = cq;
            da.n_rot = nr, da.split = c->L;
            if (fork) fork_side(c, s);  // no-op in the first chunk (still forked); later chunks wait for the previous ModDown
            launch_dh_accum(c, da, s, c->L);
            InnerArgs ia;
            memset(&ia, 0, sizeof(ia));
            for (u32 r = 0; r < nr; r++) ia.key[r] = da.key[r], ia.galois[r] = da.galois[r];
            ia.dt = w.dt, ia.own = d_ct, ia.cp = cp, ia.n_inst = nr, ia.split = c->L;
            launch_ks_inner<OWN_COPY, true>(c, ia, s, c->L, c->D);
            w.cp = cp, w.cv = cp + (size_t)nr * 2 * c->K * N;
            moddown_convert(c, w, nr, s);
            FinalArgs fa;
            memset(&fa, 0, sizeof(fa));
            fa.cq = cq, fa.cv = w.cv, fa.pt = da.pt, fa.out = d_out;
            fa.n_inst = 2, fa.n_rot = nr, fa.accumulate = r0 ? 1 : 0;
            launch_ks_final<FIN_SUMMED>(c, fa, s);
        }
        return hip_check(c, "ckks_hrot_hoisted_mac");
    }
    const u32 chunk_max = n_rot < CKKS_ROT_CHUNK ? n_rot : CKKS_ROT_CHUNK;
    const Workspace w = carve(c, d_ws, 1, 1, chunk_max);
    // rotations go through the ModDown side in chunks of at most CKKS_ROT_CHUNK, sized evenly
    const u32 n_chunks = (n_rot + CKKS_ROT_CHUNK - 1) / CKKS_ROT_CHUNK;
    const u32 chunk = (n_rot + n_chunks - 1) / n_chunks;
    // Second stream: the special-limb (IntAr) chain of a chunk beside its q-limb chain, where the inner product is at least five
    // rounds of workgroups.  Below, the launches that both classes share on one stream gain more than the events cost.
    // N = 2^16, one stream / two: L + K = 30, 7 rotations (3360 workgroups) 550 / 526 us, 3 (1440) 303 / 314, 1 182 / 198;
    // 13 + 6, chunks of 9 (2736) 730 / 710; 10 + 5, chunks of 9 (2160) 546 / 567.
    const bool fork = chunk * c->D * tiles_of(c) >= 5 * 512;
    decompose_input(w, fork ? EXTEND_FORK : EXTEND_PLAIN);
    for (u32 r0 = 0; r0 < n_rot; r0 += chunk) {
        const u32 nr = (n_rot - r0) < chunk ? (n_rot - r0) : chunk;
        InnerArgs ia;
        memset(&ia, 0, sizeof(ia));
        FinalArgs fa;
        memset(&fa, 0, sizeof(fa));
        for (u32 r = 0; r < nr; r++) {
            ia.key[r] = h_rk_ptrs[r0 + r];
            ia.galois[r] = h_galois[r0 + r];
            fa.galois[r] = h_galois[r0 + r];
        }
        ia.dt = w.dt, ia.own = d_ct, ia.cq = w.cq, ia.cp = w.cp, ia.n_inst = nr, ia.split = c->L;
        if (fork) fork_side(c, s);  // no-op in the first chunk (still forked); later chunks wait for the previous ModDown
        launch_ks_inner<OWN_COPY, true>(c, ia, s, 0, c->D);
        moddown_convert(c, w, nr, s);
        fa.cq = w.cq, fa.cq_L = c->L, fa.cv = w.cv, fa.ct1 = d_ct, fa.pt = d_pt + (size_t)r0 * c->L * N, fa.out = d_out;
        fa.n_inst = 2, fa.n_rot = nr, fa.accumulate = r0 ? 1 : 0;
        launch_ks_final<FIN_HOISTED>(c, fa, s);
    }
    return hip_check(c, "ckks_hrot_hoisted_mac");
}

extern "C" int ckks_hrot_hoisted_mac(ckks_ctx* ctx, const uint64_t* d_ct, uint32_t n_rot, const uint32_t* h_galois,
                                     const uint64_t* const* h_rk_ptrs, const uint64_t* d_pt, uint64_t* d_out,
                                     void* d_ws, size_t ws_bytes, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    return ckks_hrot_hoisted_mac_at(ctx, ctx->L, d_ct, n_rot, h_galois, h_rk_ptrs, d_pt, d_out, d_ws, ws_bytes, stream);
}

// Double-hoisted variant: the plaintext products are accumulated in the extended basis over all
// rotations (CKKS_DH_CHUNK of them per launch) and a single ModDown follows.
static int dh_mac_impl(ckks_ctx* ctx, uint32_t level, bool rescale, const uint64_t* d_ct, uint32_t n_rot,
                       const uint32_t* h_galois, const uint64_t* const* h_rk_ptrs, const uint64_t* d_pt,
                       uint64_t* d_out, void* d_ws, size_t ws_bytes, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    const View* c = view_at(ctx, level);
    if (!c) return CKKS_EINVAL;
    if (rescale && level < 2) return fail(c, CKKS_EINVAL, "rescale needs at least two limbs");
    if (!h_galois || !h_rk_ptrs) return fail(c, CKKS_EINVAL, "null host array");
    if (n_rot == 0 || n_rot > 65535) return fail(c, CKKS_EINVAL, "n_rot out of range");
    if (!d_ct || !d_pt || !d_out || misaligned(d_ct, 16) || misaligned(d_pt, 16) || misaligned(d_out, 16))
        return fail(c, CKKS_EINVAL, "null or misaligned buffer");
    if (!d_ws || misaligned(d_ws, 256)) return fail(c, CKKS_EINVAL, "workspace is null or not 256-byte aligned");
    size_t need = 0;
    int rc = view_workspace_bytes(c, CKKS_OP_HROT_DH_MAC, n_rot, &need);
    if (rc) return rc;
    if (ws_bytes < need) return fail(c, CKKS_ENOMEM, "workspace too small");
    for (u32 r = 0; r < n_rot; r++) {
        if (!h_rk_ptrs[r] || misaligned(h_rk_ptrs[r], 16)) return fail(c, CKKS_EINVAL, "null or misaligned key");
        rc = check_galois(c, h_galois[r]);
        if (rc) return rc;
    }
    rc = check_no_alias(c, d_out, limb_bytes(c, 2 * (size_t)(rescale ? c->L - 1 : c->L)), d_ct, limb_bytes(c, 2 * (size_t)c->L),
                        d_pt, limb_bytes(c, (size_t)n_rot * c->D), d_ws, ws_bytes);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    const size_t N = (size_t)1 << c->logN;
    // cm: the view whose ModDown ends the call (the merged one also divides by the last q-limb)
    const View* cm = rescale ? &ctx->merged[level] : c;
    Workspace w = carve(c, d_ws, 1, 1, 1);
    if (rescale) {
        w.cp = w.cq + (size_t)2 * cm->L * N;
        w.cv = w.cp + (size_t)2 * cm->K * N;
    }
    {  // hoisted part, as in ckks_hrot_hoisted_mac
        const LimbSel src = {c->L, 1, c->L, c->L, 0};
        const LimbSel dst = {c->L, 1, c->L, 0, 0};
        InvContigArgs a1 = {d_ct, nullptr, w.x, src, dst, {1}, 0};
        // From five rounds of extended workgroups on the integer limbs take the second stream up to the ModDown conversion (rotations:
        // one stream / two, us; N = 2^16: 40 + 10 limbs, dnum 4 (3200 workgroups) 1: 317 / 281, 6: 566 / 533, 24: 1325 / 1305; 26 + 6,
        // dnum 5 (2560) 1: 221 / 216, 6: 426 / 411).  Below, splitting the joint launches costs more (24 + 6, dnum 4 (1920) 1: 186 /
        // 196, 12: 514 / 512; level 13 (912) 1: 129 / 146, 6: 218 / 228, 12: 313 / 300).
        decompose<INV_PLAIN>(c, a1, w, s, c->dnum * c->D * tiles_of(c) >= 5 * 512 ? EXTEND_FORK : EXTEND_PLAIN);
        launch_extended_fwd_contig(c, w, s);
    }
    for (u32 r0 = 0; r0 < n_rot; r0 += CKKS_DH_CHUNK) {
        const u32 nr = (n_rot - r0) < CKKS_DH_CHUNK ? (n_rot - r0) : CKKS_DH_CHUNK;
        DhInnerArgs ia;
        memset(&ia, 0, sizeof(ia));
        for (u32 r = 0; r < nr; r++) ia.key[r] = h_rk_ptrs[r0 + r], ia.galois[r] = h_galois[r0 + r];
        ia.dt = w.dt, ia.ct = d_ct, ia.pt = d_pt + (size_t)r0 * c->D * N, ia.cq = w.cq, ia.cp = w.cp;
        ia.n_rot = nr, ia.accumulate = r0 ? 1 : 0, ia.split = cm->L, ia.pt_limbs = c->D;
        launch_dh_accum(c, ia, s, c->D);
    }
    {  // ModDown of the sum: first inverse pass of its source limbs, then the shared tail
        const LimbSel sel = {cm->K, 2, cm->K, 0, cm->L};
        InvContigArgs ic = {w.cp, nullptr, w.cp, sel, sel, {1}, 0};
        moddown_from_eval(cm, ic, w, 1, s);
    }
    FinalArgs fa;
    memset(&fa, 0, sizeof(fa));
    fa.cq = w.cq, fa.cq_L = cm->L, fa.cv = w.cv, fa.out = d_out, fa.n_inst = 2;
    launch_ks_final<FIN_KS>(cm, fa, s);
    return hip_check(c, "ckks_hrot_dh_mac");
}

extern "C" int ckks_hrot_dh_mac_at(ckks_ctx* ctx, uint32_t level, const uint64_t* d_ct, uint32_t n_rot,
                                   const uint32_t* h_galois, const uint64_t* const* h_rk_ptrs, const uint64_t* d_pt,
                                   uint64_t* d_out, void* d_ws, size_t ws_bytes, void* stream) {
    return dh_mac_impl(ctx, level, false, d_ct, n_rot, h_galois, h_rk_ptrs, d_pt, d_out, d_ws, ws_bytes, stream);
}

extern "C" int ckks_hrot_dh_mac_rescale_at(ckks_ctx* ctx, uint32_t level, const uint64_t* d_ct, uint32_t n_rot,
                                           const uint32_t* h_galois, const uint64_t* const* h_rk_ptrs,
                                           const uint64_t* d_pt, uint64_t* d_out, void* d_ws, size_t ws_bytes,
                                           void* stream) {
    return dh_mac_impl(ctx, level, true, d_ct, n_rot, h_galois, h_rk_ptrs, d_pt, d_out, d_ws, ws_bytes, stream);
}

extern "C" int ckks_hrot_dh_mac(ckks_ctx* ctx, const uint64_t* d_ct, uint32_t n_rot, const uint32_t* h_galois,
                                const uint64_t* const* h_rk_ptrs, const uint64_t* d_pt, uint64_t* d_out, void* d_ws,
                                size_t ws_bytes, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    return ckks_hrot_dh_mac_at(ctx, ctx->L, d_ct, n_rot, h_galois, h_rk_ptrs, d_pt, d_out, d_ws, ws_bytes, stream);
}

// ---------------------------------------------------------------- baby-step giant-step transform
static size_t bsgs_workspace_words(const View* c, u32 n1, u32 n2) {
    const size_t N = (size_t)1 << c->logN;
    const u32 nc = n2 < CKKS_ROT_CHUNK ? n2 : CKKS_ROT_CHUNK;
    const size_t limbs = (size_t)c->L + (size_t)c->dnum * c->D                      // x, dt of the input
                         + (size_t)n1 * 2 * c->D                                     // baby rotations, extended basis
                         + (size_t)n2 * 2 * (2 * (size_t)c->L + c->K)                // C on q / special limbs, converted part
                         + (size_t)n2 * 2 * c->L * 2;                                // inner sums, rotated inner sums
    return limbs * N + ks_workspace_words(c, nc, nc, nc, false);  // the giant rotations run the plain pipeline
}

extern "C" int ckks_lintrans_bsgs_workspace_bytes(const ckks_ctx* ctx, uint32_t level, uint32_t n1, uint32_t n2,
                                                  size_t* bytes) {
    if (!ctx || !bytes) return CKKS_EINVAL;
    const View* c = view_at(ctx, level);
    if (!c) return CKKS_EINVAL;
    if (c->K == 0) return fail(c, CKKS_EUNSUPPORTED, "context has no special primes");
    if (n1 == 0 || n1 > 64 || n2 == 0 || n2 > 64) return fail(c, CKKS_EINVAL, "n1 and n2 must be between 1 and 64");
    *bytes = bsgs_workspace_words(c, n1, n2) * sizeof(u64);
    return CKKS_OK;
}

extern "C" int ckks_lintrans_bsgs_at(ckks_ctx* ctx, uint32_t level, const uint64_t* d_ct, uint32_t n1,
                                     const uint32_t* h_baby_galois, const uint64_t* const* h_baby_rk_ptrs, uint32_t n2,
                                     const uint32_t* h_giant_galois, const uint64_t* const* h_giant_rk_ptrs,
                                     const uint64_t* d_pt, uint64_t* d_out, void* d_ws, size_t ws_bytes, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    const View* c = view_at(ctx, level);
    if (!c) return CKKS_EINVAL;
    if (!h_baby_galois || !h_baby_rk_ptrs || !h_giant_galois || !h_giant_rk_ptrs) return fail(c, CKKS_EINVAL, "null host array");
    if (!d_ct || !d_pt || !d_out || misaligned(d_ct, 16) || misaligned(d_pt, 16) || misaligned(d_out, 16))
        return fail(c, CKKS_EINVAL, "null or misaligned buffer");
    if (!d_ws || misaligned(d_ws, 256)) return fail(c, CKKS_EINVAL, "workspace is null or not 256-byte aligned");
    size_t need = 0;
    int rc = ckks_lintrans_bsgs_workspace_bytes(ctx, level, n1, n2, &need);
    if (rc) return rc;
    if (ws_bytes < need) return fail(c, CKKS_ENOMEM, "workspace too small");
    for (u32 r = 0; r < n1 + n2; r++) {
        const uint64_t* k = r < n1 ? h_baby_rk_ptrs[r] : h_giant_rk_ptrs[r - n1];
        if (!k || misaligned(k, 16)) return fail(c, CKKS_EINVAL, "null or misaligned key");
        rc = check_galois(c, r < n1 ? h_baby_galois[r] : h_giant_galois[r - n1]);
        if (rc) return rc;
    }
    rc = check_no_alias(c, d_out, limb_bytes(c, 2 * (size_t)c->L), d_ct, limb_bytes(c, 2 * (size_t)c->L), d_pt,
                        limb_bytes(c, (size_t)n1 * n2 * c->D), d_ws, ws_bytes);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    const size_t N = (size_t)1 << c->logN, LN = (size_t)c->L * N, KN = (size_t)c->K * N;
    // workspace: x | dt | Rq | Rp | Cq | Cp | Cv | inner | rot | key-switch workspace of the giant rotations
    Workspace w;
    w.x = (u64*)d_ws;
    w.dt = w.x + LN;
    u64* rq = w.dt + (size_t)c->dnum * c->D * N;
    u64* rp = rq + (size_t)n1 * 2 * LN;
    w.cq = rp + (size_t)n1 * 2 * KN;
    w.cp = w.cq + (size_t)n2 * 2 * LN;
    w.cv = w.cp + (size_t)n2 * 2 * KN;
    u64* inner = w.cv + (size_t)n2 * 2 * LN;
    u64* rot = inner + (size_t)n2 * 2 * LN;  // results to be added
    void* ks_ws = rot + (size_t)n2 * 2 * LN;
    {  // decomposition of the input, shared by every baby step
        const LimbSel src = {c->L, 1, c->L, c->L, 0};
        const LimbSel dst = {c->L, 1, c->L, 0, 0};
        InvContigArgs a1 = {d_ct, nullptr, w.x, src, dst, {1}, 0};
        decompose<INV_PLAIN>(c, a1, w, s, EXTEND_PLAIN);
        launch_extended_fwd_contig(c, w, s);
    }
    // Baby steps and combinations in one kernel where its registers hold the sums (8 x 4, N = 2^16, 24 + 6 limbs: 468 -> 354 us; on
    // integer chains of 4 + 2 and 12 + 4 limbs the call gains 2 to 4 % at N = 2^12 and 2^13, 6 to 9 % from 2^14 on; with a single baby step and
    // four giant ones, which leaves least to combine, 0 to 2.6 % at 768 to 15360 rows, N = 2^12 .. 2^16)
    if (n2 <= CKKS_DH_SUMS && n1 <= CKKS_DH_CHUNK) {
        DhInnerArgs ia;
        memset(&ia, 0, sizeof(ia));
        for (u32 b = 0; b < n1; b++) ia.key[b] = h_baby_rk_ptrs[b], ia.galois[b] = h_baby_galois[b];
        ia.dt = w.dt, ia.ct = d_ct, ia.pt = d_pt, ia.pt_limbs = c->D, ia.cq = w.cq, ia.cp = w.cp;
        ia.n_rot = n1, ia.sums = n2, ia.split = c->L;
        launch_dh_accum(c, ia, s, c->D);
    } else {
        // baby steps: R_b = P * Rot_b(ct) in the extended basis (inner product with the key, plus P * sigma_b(b))
        for (u32 b0 = 0; b0 < n1; b0 += CKKS_DH_CHUNK) {
            const u32 nb = (n1 - b0) < CKKS_DH_CHUNK ? (n1 - b0) : CKKS_DH_CHUNK;
            DhInnerArgs ia;
            memset(&ia, 0, sizeof(ia));
            for (u32 b = 0; b < nb; b++) ia.key[b] = h_baby_rk_ptrs[b0 + b], ia.galois[b] = h_baby_galois[b0 + b];
            ia.dt = w.dt, ia.ct = d_ct, ia.pt = nullptr, ia.cq = rq + (size_t)b0 * 2 * LN, ia.cp = rp + (size_t)b0 * 2 * KN;
            ia.n_rot = nb, ia.each = 1, ia.accumulate = 0, ia.split = c->L;
            launch_dh_accum(c, ia, s, c->D);
        }
        // giant-step combinations in the extended basis
        BsgsMacArgs ma = {rq, rp, d_pt, w.cq, w.cp, n1, n2};
        launch_bsgs_mac(c, ma, s);
    }
    // one ModDown per giant step (as a batch)
    {
        const LimbSel sel = {c->K, n2 * 2, c->K, 0, c->L};
        InvContigArgs ic = {w.cp, nullptr, w.cp, sel, sel, {1}, 0};
        moddown_from_eval(c, ic, w, n2, s);
    }
    FinalArgs fa;
    memset(&fa, 0, sizeof(fa));
    fa.cq = w.cq, fa.cq_L = c->L, fa.cv = w.cv, fa.out = inner, fa.n_inst = 2 * n2;
    launch_ks_final<FIN_KS>(c, fa, s);
    // Giant rotations, each inner sum with its own key, and their sum: with one ModDown for as many at a time as the digits of its
    // sources allow where that is the faster way, else as a batch
    const bool summed = giants_summed(c, n2);
    const u32 n_chunks = cdiv(n2, summed ? summed_rotations_max(c) : CKKS_ROT_CHUNK);
    const u32 chunk = summed ? cdiv(n2, n_chunks) : CKKS_ROT_CHUNK;  // a batch: full launches first (20 rotations as 10 + 10 4 % slower)
    const u32 n_sums = summed ? n_chunks : n2;
    for (u32 g0 = 0, k = 0; g0 < n2; g0 += chunk, k++) {
        const u32 ng = (n2 - g0) < chunk ? (n2 - g0) : chunk;
        const u64* in = inner + (size_t)g0 * 2 * LN;
        u64* to = n_sums == 1 ? d_out : rot + (size_t)(summed ? k : g0) * 2 * LN;
        if (summed && ng > 1) summed_rotations(c, in, ng, h_giant_galois + g0, h_giant_rk_ptrs + g0, to, ks_ws, s);
        else keyswitch_pipeline<INV_ROT, OWN_ROT>(c, c, in, nullptr, nullptr, to, ng, 1, ks_ws, s, h_giant_galois + g0, h_giant_rk_ptrs + g0);
    }
    if (n_sums > 1) {
        ProfScope ps(c, std::string("sum_instances_kernel"), (u64)(n_sums + 1) * 2 * c->L, s);
        hipLaunchKernelGGL(sum_instances_kernel, dim3((1u << c->logN) / 256, 2 * c->L), dim3(256), 0, s, rot, d_out,
                           c->tb.pc, c->logN, c->L, 2 * c->L, n_sums);
    }
    return hip_check(c, "ckks_lintrans_bsgs");
}

// Rotations of a batch of ciphertexts, each by its own Galois element with its own key (the giant steps of a
// linear transform, or the independent rotations of several activations): chunks of CKKS_ROT_CHUNK instances.
extern "C" int ckks_hrot_multi_at(ckks_ctx* ctx, uint32_t level, const uint64_t* d_ct, const uint32_t* h_galois,
                                  const uint64_t* const* h_rk_ptrs, uint64_t* d_out, uint32_t batch, void* d_ws,
                                  size_t ws_bytes, void* stream) {
    if (!ctx) return CKKS_EINVAL;
    const View* c = view_at(ctx, level);
    if (!c) return CKKS_EINVAL;
    if (!h_galois || !h_rk_ptrs) return fail(c, CKKS_EINVAL, "null host array");
    if (batch == 0) return fail(c, CKKS_EINVAL, "batch out of range");
    const u32 chunk = batch < CKKS_ROT_CHUNK ? batch : CKKS_ROT_CHUNK;
    int rc = check_ks_args(c, d_ct, h_rk_ptrs[0], d_out, chunk, CKKS_OP_HROT, d_ws, ws_bytes);
    if (rc) return rc;
    if (batch > 4096) return fail(c, CKKS_EINVAL, "batch out of range");
    for (u32 b = 0; b < batch; b++) {
        if (!h_rk_ptrs[b] || misaligned(h_rk_ptrs[b], 16)) return fail(c, CKKS_EINVAL, "null or misaligned key");
        rc = check_galois(c, h_galois[b]);
        if (rc) return rc;
    }
    const size_t ct_words = ((size_t)2 * c->L) << c->logN;
    rc = check_no_alias(c, d_out, ct_words * batch * sizeof(u64), d_ct, ct_words * batch * sizeof(u64), nullptr, 0, d_ws, ws_bytes);
    if (rc) return rc;
    for (u32 b0 = 0; b0 < batch; b0 += CKKS_ROT_CHUNK) {
        const u32 nb = (batch - b0) < CKKS_ROT_CHUNK ? (batch - b0) : CKKS_ROT_CHUNK;
        keyswitch_pipeline<INV_ROT, OWN_ROT>(c, c, d_ct + b0 * ct_words, nullptr, nullptr, d_out + b0 * ct_words, nb,
                                                       1, d_ws, (hipStream_t)stream, h_galois + b0, h_rk_ptrs + b0);
    }
    return hip_check(c, "ckks_hrot_multi");
}
