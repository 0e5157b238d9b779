"""Parity where a form is chosen by the size or the primes of a call (needs an MI355X), each size on both sides of its rule, and
the form that ran by the kernels' names.  Bit for bit against the oracle, extreme residues planted.
"""
import numpy as np
import pytest

from paper_2310_16530_amd import synth

from test_gpu_parity import dev, gpu_ctx, host, orc_params

pytestmark = pytest.mark.gpu


def _kernels(ctx, call):
    ctx.profile_enable(True)
    try:
        return host(call()), set(ctx.profile_read())
    finally:
        ctx.profile_enable(False)


@pytest.mark.parametrize("n,batch", [(1, 1), (5, 5), (4, 6), (4, 20), (5, 17)])
def test_few_integer_limbs_at_n_2_13_take_two_passes(orc, n, batch):
    """N = 2^13: forward up to 80 integer limbs, inverse up to 24; ranges with an FP64 limb keep one kernel a limb."""
    ps = synth.mixed_params(13, [49, 55, 58, 60, 53], [59], 5, "spread")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(1300 + n * batch)
    first = 1
    x = synth.uniform_residues(rng, ps.primes[first:first + n], ps.N, lead=(batch,))
    for i in range(n):
        x[0, i, : ps.N // 2] = ps.primes[first + i] - 1
    print("limbs", n, "batch", batch, flush=True)
    got, names = _kernels(ctx, lambda: ctx.ntt(dev(x), first))
    assert np.array_equal(got, orc.ntt_batch(x, P, first))
    assert ("fwd_strided_kernel<IntAr, 5>" in names) == (n * batch <= 80), names
    got, names = _kernels(ctx, lambda: ctx.intt(dev(x), first))
    assert np.array_equal(got, orc.ntt_batch(x, P, first, inverse=True))
    assert ("inv_contig_rows_kernel<IntAr, 5, 0>" in names) == (n * batch <= 24), names
    y = synth.uniform_residues(rng, ps.primes[:2], ps.N, lead=(2,))
    got, names = _kernels(ctx, lambda: ctx.intt(dev(y)))
    assert np.array_equal(got, orc.ntt_batch(y, P, 0, inverse=True)) and len(names) == 1, names


def test_second_stream_leaves_the_joint_launches_of_hoisted_calls_whole(orc):
    """The decomposition of a double-hoisted or baby-step giant-step call, and a small hoisted call, launch the same kernels
    with the second stream on: split by arithmetic over two streams they took up to a tenth longer."""
    ps = synth.small_params(13, 6, 3, 2)
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(77)
    gs = [synth.galois_element(r, ps.logN) for r in (1, 2, 3)]
    rks = [synth.uniform_residues(rng, ps.primes, ps.N, lead=(ps.dnum, 2)) for _ in gs]
    d_rks = [dev(k) for k in rks]
    ct = synth.uniform_residues(rng, ps.q_primes, ps.N, lead=(2,))
    pt = synth.uniform_residues(rng, ps.primes, ps.N, lead=(3,))
    ptq = np.ascontiguousarray(pt[:, :ps.L])
    calls = ((lambda: ctx.hrot_dh_mac(dev(ct), gs, d_rks, dev(pt)), orc.hrot_dh_mac_level(ct, gs, rks, pt, P)),
             (lambda: ctx.hrot_hoisted_mac(dev(ct), gs, d_rks, dev(ptq)), orc.hrot_hoisted_mac(ct, gs, rks, ptq, P)))
    for call, want in calls:
        got, one = _kernels(ctx, call)
        assert np.array_equal(got, want)
        ctx.set_overlap(True)
        try:
            got, two = _kernels(ctx, call)
        finally:
            ctx.set_overlap(False)
        assert np.array_equal(got, want) and two == one, two ^ one


@pytest.mark.parametrize("n_rot", [16, 32])
def test_hoisted_rotations_with_the_second_stream_at_work(orc, n_rot):
    """From five rounds of inner-product workgroups on (16 rotations, L + K = 10, N = 2^16) the integer limbs run on the second
    stream; 32 rotations fork once more after the first chunk's ModDown."""
    ps = synth.small_params(16, 8, 2, 2)
    ctx = gpu_ctx(ps)
    rng = np.random.default_rng(1616)
    gs = [synth.galois_element(r + 1, ps.logN) for r in range(n_rot)]
    keys = [synth.uniform_residues(rng, ps.primes, ps.N, lead=(ps.dnum, 2)) for _ in range(3)]
    d_keys = [dev(k) for k in keys]
    ct, pt = synth.uniform_residues(rng, ps.q_primes, ps.N, lead=(2,)), synth.uniform_residues(rng, ps.q_primes, ps.N, lead=(n_rot,))
    d_ct, d_pt = dev(ct), dev(pt)
    call = lambda: ctx.hrot_hoisted_mac(d_ct, gs, [d_keys[r % 3] for r in range(n_rot)], d_pt)
    print("rotations", n_rot, flush=True)
    want = host(call())
    if n_rot == 16:
        assert np.array_equal(want, orc.hrot_hoisted_mac(ct, gs, [keys[r % 3] for r in range(n_rot)], pt, orc_params(orc, ps)))
    ctx.set_overlap(True)
    try:
        got, names = _kernels(ctx, call)
        assert np.array_equal(got, want)
        assert "ks_inner_kernel<IntAr, 8, 0, true, false>" in names, names
        for _ in range(2):
            assert np.array_equal(host(call()), want)
    finally:
        ctx.set_overlap(False)


def _below(bound, two_n, count):
    """the `count` largest primes = 1 mod two_n below bound"""
    out, c = [], (bound - 2) // two_n * two_n + 1
    while len(out) < count:
        if synth.is_prime(c):
            out.append(c)
        c -= two_n
    return tuple(out)


@pytest.mark.parametrize("logN,L,K,dnum,counts", [(12, 3, 1, 3, (1, 3, 9, 33)), (12, 9, 2, 9, (2, 17)), (13, 2, 7, 1, (4, 40)),
                                                  (16, 17, 4, 6, (9, 20)), (16, 13, 3, 3, (9, 18))])
def test_double_hoisted_sum_on_integer_chains(orc, logN, L, K, dnum, counts):
    """Chains of integer primes alone, the largest the library takes, so that every bound of the unreduced sums is met:
    rotation counts around the eight terms between two folds, one and four wavefronts per row (N = 2^16: few / many rotations),
    digit counts around the eight terms of a digit sum, more rotations than one launch takes, baby steps stored singly."""
    primes = _below(1 << 61, 2 << logN, L + K)
    ps = synth.ExplicitParamSet("below_2_61", logN, dnum, primes[:L], primes[L:])
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(6100 + logN + L)
    n = max(counts)
    gs = [synth.galois_element((-1) ** r * (r // 2 + 1), logN) for r in range(n)]
    keys = [synth.uniform_residues(rng, ps.primes, ps.N, lead=(dnum, 2)) for _ in range(3)]
    ct, pt = synth.uniform_residues(rng, ps.q_primes, ps.N, lead=(2,)), synth.uniform_residues(rng, ps.primes, ps.N, lead=(n,))
    for i, p in enumerate(ps.primes):
        for k in keys:
            k[:, :, i, : ps.N // 2] = p - 1
        pt[:, i, : ps.N // 4] = p - 1
        if i < L:
            ct[:, i, : ps.N // 8] = p - 1
    d_keys, d_ct = [dev(k) for k in keys], dev(ct)
    for m in counts:
        print(logN, L, K, dnum, "rotations", m, flush=True)
        got, names = _kernels(ctx, lambda: ctx.hrot_dh_mac(d_ct, gs[:m], [d_keys[r % 3] for r in range(m)], dev(pt[:m])))
        assert np.array_equal(got, orc.hrot_dh_mac_level(ct, gs[:m], [keys[r % 3] for r in range(m)], pt[:m], P)), m
        assert "dh_accum_kernel<IntAr, 2>" in names and not any(k.startswith("dh_accum_kernel<AnyAr") for k in names)
    if logN == 12:
        d_pt = dev(np.ascontiguousarray(pt[:2]).reshape(1, 2, L + K, ps.N))
        got = host(ctx.lintrans_bsgs_at(L, d_ct, gs[:2], d_keys[:2], gs[2:3], d_keys[2:], d_pt))
        assert np.array_equal(got, orc.lintrans_bsgs_level(ct, gs[:2], keys[:2], gs[2:3], keys[2:], pt[:2].reshape(1, 2, L + K, ps.N), P))


@pytest.mark.parametrize("logN,q,p,dnum,counts", [(12, (49, 49, 49), (59,), 3, (1, 4, 5, 8, 9)), (12, (49, 50, 60, 49, 58), (48, 60), 3, (3, 8, 9, 41)),
                                                  (16, (49,) * 17, (59,) * 4, 5, (2, 5, 8, 9)), (13, (49,) * 9, (49, 60), 9, (7,))])
def test_double_hoisted_sum_on_mixed_chains(orc, logN, q, p, dnum, counts):
    """Chains with FP64 limbs: up to eight rotations take the narrow rows, more the wide ones, 41 = a wide launch and nine more in
    a second; a unit plaintext and baby steps stored singly on narrow rows too."""
    ps = synth.mixed_params(logN, list(q), list(p), dnum, "mixed_dh")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(4900 + logN + len(q))
    n = max(counts)
    gs = [synth.galois_element((-1) ** r * (r // 2 + 1), logN) for r in range(n)]
    keys = [synth.uniform_residues(rng, ps.primes, ps.N, lead=(dnum, 2)) for _ in range(3)]
    ct, pt = synth.uniform_residues(rng, ps.q_primes, ps.N, lead=(2,)), synth.uniform_residues(rng, ps.primes, ps.N, lead=(n,))
    for x, primes in ((ct, ps.q_primes), (pt, ps.primes), *((k, ps.primes) for k in keys)):
        for i, m in enumerate(primes):
            x[..., i, : ps.N // 2] = m - 1
    d_ct, d_keys = dev(ct), [dev(k) for k in keys]
    for count in counts:
        print(logN, "rotations", count, flush=True)
        got, names = _kernels(ctx, lambda: ctx.hrot_dh_mac(d_ct, gs[:count], [d_keys[r % 3] for r in range(count)], dev(pt[:count])))
        assert np.array_equal(got, orc.hrot_dh_mac_level(ct, gs[:count], [keys[r % 3] for r in range(count)], pt[:count], P)), count
        chunks = [min(32, count - f) for f in range(0, count, 32)]
        assert {k for k in names if k.startswith("dh_")} == {"dh_accum_kernel<AnyAr, %d>" % (2 if k <= 8 else 4) for k in chunks}, names
    if logN == 12:
        d_pt = dev(np.ascontiguousarray(pt[:2]).reshape(1, 2, -1, ps.N))
        got = host(ctx.lintrans_bsgs_at(ps.L, d_ct, gs[:2], d_keys[:2], gs[2:3], d_keys[2:], d_pt))
        assert np.array_equal(got, orc.lintrans_bsgs_level(ct, gs[:2], keys[:2], gs[2:3], keys[2:], pt[:2].reshape(1, 2, -1, ps.N), P))


@pytest.mark.parametrize("logN,q,p,dnum,two", [(16, (49,) * 26, (59,) * 6, 5, True), (16, (49,) * 25, (59,) * 6, 5, False), (14, (49, 55) * 12, (48, 60, 49), 24, True),
                                               (14, (55,) * 12 + (49,) * 11, (60, 59), 23, False)])
def test_double_hoisted_calls_with_the_second_stream_at_work(orc, logN, q, p, dnum, two):
    """From dnum * (L + K) * N / 2^12 = 2560 workgroups on the integer limbs run on the second stream up to the ModDown: integer and FP64
    special limbs, alternating limbs, more rotations than one launch takes, the merged rescale, repeated calls."""
    ps = synth.mixed_params(logN, list(q), list(p), dnum, "dh_two")
    assert (dnum * (ps.L + ps.K) * (ps.N >> 12) >= 2560) == two
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(2560 + logN + len(q))
    keys = [synth.uniform_residues(rng, ps.primes, ps.N, lead=(ps.dnum, 2)) for _ in range(2)]
    d_keys = [dev(k) for k in keys]
    n = 3 if logN == 16 else 35
    gs = [synth.galois_element((-1) ** r * (r + 1), logN) for r in range(n)]
    ct, pt = synth.uniform_residues(rng, ps.q_primes, ps.N, lead=(2,)), synth.uniform_residues(rng, ps.primes, ps.N, lead=(n,))
    d_ct, d_pt = dev(ct), dev(pt)
    for count in (1, n):
        print(logN, "rotations", count, flush=True)
        args = d_ct, gs[:count], [d_keys[r % 2] for r in range(count)], d_pt[:count].contiguous()
        want = orc.hrot_dh_mac_level(ct, gs[:count], [keys[r % 2] for r in range(count)], pt[:count], P)
        merged = host(ctx.hrot_dh_mac_rescale_at(ps.L, *args))
        ctx.set_overlap(True)
        try:
            got, names = _kernels(ctx, lambda: ctx.hrot_dh_mac(*args))
            assert np.array_equal(got, want), count
            assert ("dh_accum_kernel<IntAr, 2>" in names) == two, names
            for _ in range(3):
                assert np.array_equal(host(ctx.hrot_dh_mac_rescale_at(ps.L, *args)), merged), count
                assert np.array_equal(host(ctx.hrot_dh_mac(*args)), want), count
        finally:
            ctx.set_overlap(False)


@pytest.mark.parametrize("logN", [12, 13])
@pytest.mark.parametrize("q", [(49,) * 3, (55, 56, 57), (49, 55) * 5, (49,) * 7 + (58,) * 5, (49,) * 26], ids=lambda q: str(len(q)))
def test_workgroups_of_a_limb_each_at_any_share_of_the_chip(orc, logN, q):
    """Limb counts that fill the eight dies evenly (7, 8, 14, 16, 26) and that do not (1, 3, 10, 12, 17), one to many instances:
    every workgroup finds its limb and instance either way, also with limbs of both arithmetics and an offset."""
    ps = synth.mixed_params(logN, list(q), [59], len(q), "whole")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(808 + logN + len(q))
    for n in sorted({1, 3, 7, 8, 10, 12, 14, 16, 17, 26} & set(range(len(q) + 1))):
        for batch in (1, 5, 33):
            first = (len(q) - n) // 2
            x = synth.uniform_residues(rng, ps.primes[first:first + n], ps.N, lead=(batch,))
            assert np.array_equal(host(ctx.ntt(dev(x), first)), orc.ntt_batch(x, P, first)), (n, batch)
            assert np.array_equal(host(ctx.intt(dev(x), first)), orc.ntt_batch(x, P, first, inverse=True)), (n, batch)
    print(logN, len(q), "limbs", flush=True)
    ct = synth.uniform_residues(rng, ps.q_primes, ps.N, lead=(9, 2))
    assert np.array_equal(host(ctx.rescale(len(q), dev(ct))), orc.rescale(ct, P))
