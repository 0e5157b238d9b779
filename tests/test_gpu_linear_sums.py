"""Parity where sums over rotations are formed before the ModDown's converted part joins them (needs an MI355X): rotation counts on
both sides of the rules and of every chunk, chains of either arithmetic, extreme residues, both stream modes.  Bit for bit
against the oracle, which follows the definition rotation by rotation.
"""
import numpy as np
import pytest

from paper_2310_16530_amd import synth

from test_gpu_forms_by_size import _below, _kernels
from test_gpu_parity import dev, gpu_ctx, host, orc_params

pytestmark = pytest.mark.gpu


def _inputs(ps, n, n_keys, seed, pt_primes, lead):
    rng = np.random.default_rng(seed)
    gs = [synth.galois_element((-1) ** r * (r // 2 + 1), ps.logN) for r in range(n)]
    keys = [synth.uniform_residues(rng, ps.primes, ps.N, lead=(ps.dnum, 2)) for _ in range(n_keys)]
    ct, pt = synth.uniform_residues(rng, ps.q_primes, ps.N, lead=(2,)), synth.uniform_residues(rng, pt_primes, ps.N, lead=lead)
    for x, primes in ((ct, ps.q_primes), (pt, pt_primes), *((k, ps.primes) for k in keys)):
        for i, m in enumerate(primes):
            x[..., i, : ps.N // 2] = m - 1
    return gs, keys, ct, pt


@pytest.mark.parametrize("logN,q,p,dnum,counts", [
    (12, (49,) * 3, (59,), 3, (16, 17, 24, 41)),          # three digits of one limb, one special prime
    (12, (49, 60, 50, 58), (48, 60), 2, (17, 33)),        # both arithmetics among q-limbs and special limbs
    (13, (49, 49), (59,) * 7, 1, (17, 18, 35)),           # more special than ciphertext limbs: little room per chunk
    (12, None, 2, 2, (17, 26)),                           # integer primes just below 2^61
    (16, (49,) * 9, (59,) * 3, 3, (11, 12)),              # both sides of the rule up to 16 rotations
])
def test_hoisted_sums_before_the_mod_down(orc, logN, q, p, dnum, counts):
    if q is None:
        primes = _below(1 << 61, 2 << logN, 6 + p)
        ps = synth.ExplicitParamSet("below_2_61", logN, dnum, primes[:6], primes[6:])
    else:
        ps = synth.mixed_params(logN, list(q), list(p), dnum, "sums")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    n = max(counts)
    gs, keys, ct, pt = _inputs(ps, n, 3, 1700 + logN + dnum, ps.q_primes, (n,))
    d_ct, d_pt, d_keys = dev(ct), dev(pt), [dev(k) for k in keys]
    for m in counts:
        print(logN, "rotations", m, flush=True)
        want = orc.hrot_hoisted_mac(ct, gs[:m], [keys[r % 3] for r in range(m)], pt[:m], P)
        for overlap in (False, True):
            ctx.set_overlap(overlap)
            try:
                got, names = _kernels(ctx, lambda: ctx.hrot_hoisted_mac(d_ct, gs[:m], [d_keys[r % 3] for r in range(m)], d_pt[:m].contiguous()))
            finally:
                ctx.set_overlap(False)
            assert np.array_equal(got, want), (m, overlap)
            summed = m > 16 or (logN == 16 and m >= 12 and ps.L >= 9)
            assert any(k.startswith("ks_final_kernel") and k.endswith(", 4>") for k in names) == summed, names


def _inner_time(wgs, terms):
    """Rounds of workgroups times passes per wavefront of an inner product, the best of one, two and four wavefronts a row."""
    times = [-(-wgs // 512) * (2 * terms + 4)]
    for ways in (2, 4) if terms > 1 else ():
        if ways == 4 or wgs <= 512:
            times.append(-(-ways * wgs // 512) * (2 * -(-terms // ways) + 3))
    return min(times)


def _one_mod_down(ps, level, n):
    """Whether n giant rotations share a ModDown: enough workgroups in the q-limb product's smallest launch, a run of limbs of one
    arithmetic; a product not much longer than that of a batch; and sums that hold as many rotations as a batch does or nearly so."""
    if n < 2 or ps.K < 2:
        return False
    fp = [q < 3 << 48 for q in ps.primes[:level]]
    runs = [1]
    for a, b in zip(fp, fp[1:]):
        runs[-1:] = [runs[-1] + 1] if a == b else [runs[-1], 1]
    wgs, a_sum = [r * (ps.N >> 12) for r in runs], min(16, 0x7f7f7f7f7f7f7f7f // max(ps.primes[ps.L:]))
    sums, digits = -(-n // a_sum), -(-level // -(-ps.L // ps.dnum))
    if 4 * sums * sum(_inner_time(w, -(-n // sums) * digits) for w in wgs) > 5 * sum(_inner_time(w * n, digits) for w in wgs):
        return False
    return min(wgs) >= 96 if sums == -(-n // 16) else min(wgs) >= 192 and a_sum >= 6


@pytest.mark.parametrize("logN,q,p,dnum,level,steps", [
    (12, (49,) * 6, (59, 59), 3, 6, ((1, 1), (3, 2), (2, 3), (5, 4), (2, 5), (3, 16), (33, 2))),
    (12, (49, 60, 50, 58, 49), (48, 60), 3, 4, ((2, 1), (3, 4), (2, 6))),   # both arithmetics, a partial last digit
    (13, (49,) * 3, (59,), 3, 3, ((2, 1), (2, 4))),                         # one special prime: rotations end singly
    (12, None, 2, 2, 6, ((2, 3), (2, 4), (3, 7))),                          # primes just below 2^61: three sums fit the digits
    (14, (49,) * 16, (59,) * 2, 8, 15, ((2, 2), (1, 4))),                   # more digits than one unreduced sum takes
    (16, (49,) * 8, (59,) * 4, 2, 8, ((8, 4), (3, 3))),
    (12, (49,) * 96, (59,) * 12, 12, 96, ((2, 3), (1, 5))),                 # as few workgroups as the joint ModDown takes
    (13, (49,) * 50, (59,) * 8, 7, 48, ((2, 2),)),
    (14, (49,) * 24, (49,) * 6, 4, 23, ((2, 3),)),                          # one workgroup less
    (15, (49,) * 12 + (55,) * 12, (48, 60, 59), 8, 24, ((2, 4),)),          # 96 of either arithmetic, special limbs of both
    (14, (49,) * 23 + (55,), (59, 60, 59), 8, 24, ((2, 3),)),               # a short run of integer limbs
    (16, (60,) * 12, (60,) * 2, 6, 12, ((1, 7), (1, 8))),                   # seven a sum: one sum, two sums of four
    (16, (60,) * 11, (60,) * 2, 6, 11, ((1, 8),)),                          # ... on fewer workgroups
    (13, (55,) * 70, (59,) * 3, 24, 70, ((2, 3),)),                         # many digits: the product would take longer than a batch's
    (16, None, 2, 2, 6, ((1, 3), (1, 4))),                                  # three a sum; four sums of one baby step on many integer rows
])
def test_baby_step_giant_step_sums(orc, logN, q, p, dnum, level, steps):
    if q is None:
        primes = _below(1 << 61, 2 << logN, 6 + p)
        ps = synth.ExplicitParamSet("below_2_61", logN, dnum, primes[:6], primes[6:])
    else:
        ps = synth.mixed_params(logN, list(q), list(p), dnum, "sums")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    ext = list(ps.primes[:level]) + list(ps.primes[ps.L:])
    n1, n2 = max(s[0] for s in steps), max(s[1] for s in steps)
    gs, keys, ct, pt = _inputs(ps, n1 + n2, 3, 2600 + logN + dnum, ext, (n2, n1))
    ct = np.ascontiguousarray(ct[:, :level])
    d_ct, d_keys = dev(ct), [dev(k) for k in keys]
    for a, b in steps:
        print(logN, "baby", a, "giant", b, flush=True)
        use = np.ascontiguousarray(pt[:b, :a])
        baby, giant = [keys[r % 3] for r in range(a)], [keys[(r + 1) % 3] for r in range(b)]
        want = orc.lintrans_bsgs_level(ct, gs[:a], baby, gs[n1:n1 + b], giant, use, P)
        for overlap in (False, True):
            ctx.set_overlap(overlap)
            try:
                got, names = _kernels(ctx, lambda: ctx.lintrans_bsgs_at(level, d_ct, gs[:a], [d_keys[r % 3] for r in range(a)], gs[n1:n1 + b],
                                                                        [d_keys[(r + 1) % 3] for r in range(b)], dev(use)))
            finally:
                ctx.set_overlap(False)
            assert np.array_equal(got, want), (a, b, overlap)
            assert any(k.startswith("inv_strided_sum_kernel") for k in names) == _one_mod_down(ps, level, b), names
            assert any(k.startswith("bsgs_mac_kernel") for k in names) == (a > 32 or b > 4), names


def test_baby_steps_of_many_digits_leave_room_for_eight_products(orc):
    """59 digits of one limb just below 3 * 2^48 (ten parts of an unreduced sum), every part near +q/2 on one component and -q/2 on
    the other: joined without a reduction they reach 5 q, and eight of their products with a plaintext pass 2^53."""
    L, limit = 59, 3 << 48
    primes = _below(limit, 2 << 12, L) + _below(1 << 60, 2 << 12, 1)
    ps = synth.ExplicitParamSet("many_digits", 12, L, primes[:L], primes[L:])
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(5959)
    ct = np.zeros((2, L, ps.N), dtype=np.uint64)
    ct[1] = 1  # every digit is the constant 1 on every limb
    key = synth.uniform_residues(rng, ps.primes, ps.N, lead=(L, 2))
    for i, q in enumerate(primes[:L]):
        for first in range(0, L, 6):
            last = min(first + 6, L) - 1
            for t, goal in ((0, (q - 1) // 2), (1, (q + 1) // 2)):
                rest = key[first:last, t, i].sum(axis=0, dtype=np.uint64) % np.uint64(q)
                key[last, t, i] = (np.uint64(goal) + np.uint64(q) - rest) % np.uint64(q)
    n1, n2 = 32, 2
    gs = [synth.galois_element((-1) ** r * (r // 2 + 1), ps.logN) for r in range(n1 + n2)]
    pt = synth.uniform_residues(rng, ps.primes, ps.N, lead=(n2, n1))
    d_key = dev(key)
    got = host(ctx.lintrans_bsgs_at(L, dev(ct), gs[:n1], [d_key] * n1, gs[n1:], [d_key] * n2, dev(pt)))
    assert np.array_equal(got, orc.lintrans_bsgs_level(ct, gs[:n1], [key] * n1, gs[n1:], [key] * n2, pt, P))


@pytest.mark.parametrize("logN,q,p,dnum,counts,summed", [
    (12, (49,) * 9, (59,), 9, (17, 40), False),            # many digits on few workgroups: one launch of both arithmetics
    (15, (49,) * 10, (59,) * 2, 5, (17,), True),           # as many as 16 workgroups a digit
    (12, (49, 55) * 3, (59,), 6, (40,), True),             # half the limbs integer
    (12, (49,) * 4, (59,), 4, (33, 40, 50), True)])        # two chunks: 17 and 16 rotations, 20 and 20, 25 and 25
def test_form_of_a_hoisted_sum_by_digits_and_workgroups(orc, logN, q, p, dnum, counts, summed):
    ps = synth.mixed_params(logN, list(q), list(p), dnum, "form")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    n = max(counts)
    gs, keys, ct, pt = _inputs(ps, n, 3, 1800 + logN + dnum, ps.q_primes, (n,))
    d_ct, d_pt, d_keys = dev(ct), dev(pt), [dev(k) for k in keys]
    for m in counts:
        print(logN, dnum, "rotations", m, flush=True)
        got, names = _kernels(ctx, lambda: ctx.hrot_hoisted_mac(d_ct, gs[:m], [d_keys[r % 3] for r in range(m)], d_pt[:m].contiguous()))
        assert np.array_equal(got, orc.hrot_hoisted_mac(ct, gs[:m], [keys[r % 3] for r in range(m)], pt[:m], P)), m
        assert any(k.startswith("ks_final_kernel") and k.endswith(", 4>") for k in names) == summed, names


@pytest.mark.parametrize("m,chunks", [(17, 1), (28, 1), (29, 2), (56, 2), (57, 3), (59, 3)])
def test_chunks_of_a_hoisted_sum_are_as_large_as_the_workspace(orc, m, chunks):
    """4 + 1 limbs: the workspace holds 28 rotations of this form (31 * 4 + 16 limbs over 5).  The special limbs of a chunk are one launch; 59
    rotations are chunks of 20, 20 and 19."""
    ps = synth.mixed_params(12, [49] * 4, [59], 4, "chunks")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    gs, keys, ct, pt = _inputs(ps, m, 3, 5700 + m, ps.q_primes, (m,))
    d_ct, d_pt, d_keys = dev(ct), dev(pt), [dev(k) for k in keys]
    print("rotations", m, flush=True)
    ctx.profile_enable(True)
    try:
        got = host(ctx.hrot_hoisted_mac(d_ct, gs, [d_keys[r % 3] for r in range(m)], d_pt))
        launches = {k: v[0] for k, v in ctx.profile_read().items()}
    finally:
        ctx.profile_enable(False)
    assert np.array_equal(got, orc.hrot_hoisted_mac(ct, gs, [keys[r % 3] for r in range(m)], pt, P))
    for start in ("ks_inner_kernel<IntAr, 4, 0, true", "dh_accum_kernel", "ks_final_kernel<FpAr, 4, 4>"):
        assert sum(n for k, n in launches.items() if k.startswith(start)) == chunks, launches


def test_hoisted_sums_on_integer_limbs_with_the_second_stream_at_work(orc):
    """N = 2^16, FP64 and integer q-limbs, 32 rotations in two chunks: with the second stream on the sum on the integer q-limbs is
    written there, and once more after the fork of the second chunk."""
    ps = synth.mixed_params(16, [49, 49, 49, 55, 49, 55, 49, 55], [59, 59], 2, "two_streams")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    n = 32
    gs, keys, ct, pt = _inputs(ps, n, 3, 3232, ps.q_primes, (n,))
    d_ct, d_pt, d_keys = dev(ct), dev(pt), [dev(k) for k in keys]
    call = lambda: ctx.hrot_hoisted_mac(d_ct, gs, [d_keys[r % 3] for r in range(n)], d_pt)
    want = orc.hrot_hoisted_mac(ct, gs, [keys[r % 3] for r in range(n)], pt, P)
    got, one = _kernels(ctx, call)
    assert np.array_equal(got, want) and not any(k.startswith("dh_accum_kernel<IntAr") for k in one), one
    ctx.set_overlap(True)
    try:
        got, two = _kernels(ctx, call)
        assert np.array_equal(got, want) and any(k.startswith("dh_accum_kernel<IntAr") for k in two), two
        for _ in range(3):
            assert np.array_equal(host(call()), want)
    finally:
        ctx.set_overlap(False)


def test_hoisted_sums_on_special_limbs_of_both_arithmetics_stay_on_one_stream(orc):
    """The sizes of the test above: the launches that the special limbs' arithmetics share are not split for the second stream."""
    ps = synth.mixed_params(16, [49] * 8, [49, 59], 2, "one_stream")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    n = 32
    gs, keys, ct, pt = _inputs(ps, n, 3, 3233, ps.q_primes, (n,))
    d_ct, d_pt, d_keys = dev(ct), dev(pt), [dev(k) for k in keys]
    call = lambda: ctx.hrot_hoisted_mac(d_ct, gs, [d_keys[r % 3] for r in range(n)], d_pt)
    want = orc.hrot_hoisted_mac(ct, gs, [keys[r % 3] for r in range(n)], pt, P)
    got, one = _kernels(ctx, call)
    assert np.array_equal(got, want)
    ctx.set_overlap(True)
    try:
        got, two = _kernels(ctx, call)
    finally:
        ctx.set_overlap(False)
    assert np.array_equal(got, want) and two == one, two ^ one
