"""Parity of the fused base conversions where their forms change (needs an MI355X): the number of source limbs around
every multiple the matrix-core operands are cut at (1, 2, 4, 5, 8, 9, 16, 17), target counts that leave the last block of
targets partly filled, both arithmetics as sources and targets, and single-source launches on either side of the grid
size from which four targets share a load.  Bit for bit against the oracle, extreme residues planted.
"""
import numpy as np
import pytest

from paper_2310_16530_amd import synth

from test_gpu_parity import dev, gpu_ctx, host, orc_params

pytestmark = pytest.mark.gpu

# (logN, L, K, dnum, q bits, p bits, batch)
SHAPES = [(12, 3, 1, 3, 49, 59, 2), (13, 5, 2, 3, 49, 59, 2), (12, 7, 4, 2, 49, 59, 2), (13, 9, 5, 2, 49, 59, 1),
          (12, 9, 8, 1, 49, 59, 2), (14, 10, 9, 2, 55, 59, 1), (12, 17, 16, 2, 49, 59, 1), (12, 18, 16, 2, 55, 59, 1),
          (13, 4, 3, 2, 35, 40, 2), (14, 6, 3, 2, 49, 59, 1), (15, 9, 5, 2, 49, 59, 1), (14, 7, 2, 4, 49, 59, 3),
          (16, 5, 4, 2, 49, 59, 1), (15, 4, 1, 4, 48, 49, 14)]


def _extreme(rng, primes, N, lead):
    x = synth.uniform_residues(rng, primes, N, lead=lead)
    for i, p in enumerate(primes):
        x[..., i, : N // 4] = p - 1
        x[..., i, N // 4: N // 4 + 64] = 0
    return x


@pytest.mark.parametrize("shape", SHAPES)
def test_conversions_at_the_edges_of_their_forms(orc, shape):
    *set_, batch = shape
    ps = synth.small_params(*set_)
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(77000 + sum(shape))
    key = synth.uniform_residues(rng, ps.primes, ps.N, lead=(ps.dnum, 2))
    d_key = dev(key)
    g = synth.galois_element(5, ps.logN)
    for ell in sorted({ps.L, max(2, ps.L - 1), min(ps.L, ps.alpha + 1)}, reverse=True):
        print(shape, "level", ell, flush=True)
        q = ps.q_primes[:ell]
        ct1, ct2 = (_extreme(rng, q, ps.N, (batch, 2)) for _ in range(2))
        hr = host(ctx.hrot_at(ell, dev(ct1), g, d_key))
        hm = host(ctx.hmult_relin_rescale_at(ell, dev(ct1), dev(ct2), d_key))
        for b in range(0, batch, 5):
            assert np.array_equal(hr[b], orc.hrot_level(ct1[b], g, key, P)), (ell, b)
            assert np.array_equal(hm[b], orc.hmult_relin_rescale_level(ct1[b], ct2[b], key, P)), (ell, b)
        assert np.array_equal(host(ctx.rescale(ell, dev(ct1))), orc.rescale(ct1, P)), ell


# (logN, q floors, p floors, batch): digits of one limb and one special prime, grids on both sides of 512 workgroups of four
# targets; floors from 50 bits on are integer arithmetic
SINGLE = [(15, (49, 49, 49, 49), 59, 4), (15, (49, 49, 49, 49), 59, 14), (15, (49, 49, 49, 49), 59, 32),
          (14, (49, 50, 58, 55, 55, 58, 60), 48, 32), (13, (55, 56, 57, 58, 59, 60), 60, 8), (13, (55, 56, 57, 58, 59, 60), 60, 40)]


@pytest.mark.parametrize("logN,q,p,batch", SINGLE)
def test_single_source_conversions_share_a_load_for_fp64_targets_only(orc, logN, q, p, batch):
    """ModUp, ModDown and rescale from one limb: FP64 targets four per workgroup from 512 workgroups on, integer ones singly."""
    ps = synth.mixed_params(logN, list(q), [p], len(q), "single")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(5120 + logN + batch)
    key = synth.uniform_residues(rng, ps.primes, ps.N, lead=(ps.dnum, 2))
    d_key = dev(key)
    g = synth.galois_element(3, ps.logN)
    tiles, A = ps.N >> 12, logN - 8

    def check(call, up_targets, dn_targets):
        ctx.profile_enable(True)
        try:
            got, names = host(call()), set(ctx.profile_read())
        finally:
            ctx.profile_enable(False)
        forms = {n for n in names if n.startswith("conv_fwd_strided_kernel") and n.endswith("true>")}
        wgs = {1: batch * ps.dnum * tiles * -(-up_targets // 4), 2: 2 * batch * tiles * -(-dn_targets // 4)}
        allowed = {"conv_fwd_strided_kernel<%s, %d, %d, %d, true>" % (ar, A, d, 4 if ar == "FpAr" and wgs[d] >= 512 else 1)
                   for ar in ("FpAr", "IntAr") for d in (1, 2)}
        assert forms and forms <= allowed, (forms, wgs)
        return got, forms

    for ell in (ps.L, ps.L - 1):
        print(logN, "batch", batch, "level", ell, flush=True)
        ct1, ct2 = (_extreme(rng, ps.q_primes[:ell], ps.N, (batch, 2)) for _ in range(2))
        if ell == ps.L:
            got, forms = check(lambda: ctx.hrot_at(ell, dev(ct1), g, d_key), ell + 1, ell)
            assert len(forms) == 2 * len({b >= 50 for b in q}) + (p < 50 <= min(q)) + (max(q) < 50 <= p), forms
            for b in range(0, batch, 6):
                assert np.array_equal(got[b], orc.hrot_level(ct1[b], g, key, P)), (ell, b)
        got, _ = check(lambda: ctx.rescale(ell, dev(ct1)), ell + 1, ell - 1)
        assert np.array_equal(got[::6], orc.rescale(ct1[::6], P)), ell
        hm = host(ctx.hmult_relin_rescale_at(ell, dev(ct1), dev(ct2), d_key))
        for b in range(0, batch, 6):
            assert np.array_equal(hm[b], orc.hmult_relin_rescale_level(ct1[b], ct2[b], key, P)), (ell, b)


@pytest.mark.parametrize("logN,L,K,dnum,batch,order", [
    (14, 10, 2, 5, 1, "fp first"), (14, 12, 5, 3, 1, "fp first"), (15, 11, 6, 2, 2, "fp first"), (14, 14, 7, 2, 3, "fp first"),
    (14, 16, 8, 2, 1, "fp first"), (14, 9, 3, 3, 30, "fp first"), (15, 13, 6, 3, 5, "alternating"), (16, 6, 2, 3, 1, "fp first"),
    (16, 13, 6, 3, 1, "fp first"), (12, 12, 6, 2, 1, "fp first"), (13, 7, 5, 2, 40, "fp first"),
    (13, 39, 5, 3, 1, "fp first")])  # thirteen sources: on two streams whatever the number of workgroups
def test_source_words_and_joint_conversions(orc, logN, L, K, dnum, batch, order):
    """Two, three and five to eight sources (a lane half loads half of them, rounded up), both classes of targets in one launch where
    the FP64 limbs come first and N >= 2^14, ModDowns with two FP64 targets per workgroup and with four, target counts that
    leave the last workgroup one to three, a partial last digit; both stream modes, extreme residues."""
    q = [49] * L if order == "fp first" else [(49, 55)[i % 2] for i in range(L)]
    ps = synth.mixed_params(logN, q, [59] * K, dnum, "words")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(100 * logN + L)
    ct, key = synth.uniform_residues(rng, ps.q_primes, ps.N, lead=(2, 2)), synth.uniform_residues(rng, ps.primes, ps.N, lead=(dnum, 2))
    for i, p in enumerate(ps.primes):
        key[..., i, : ps.N // 2] = p - 1
        if i < L:
            ct[0, :, i, ps.N // 4:] = p - 1
    d_ct, d_key, g = dev(np.concatenate([ct[:1]] * (batch - 1) + [ct[1:]])), dev(key), synth.galois_element(5, logN)
    want = [orc.hrot(c, g, key, P) for c in ct]
    for overlap in (False, True):
        ctx.set_overlap(overlap)
        ctx.profile_enable(True)
        try:
            got, names = host(ctx.hrot(d_ct, g, d_key)), set(ctx.profile_read())
        finally:
            ctx.profile_enable(False)
            ctx.set_overlap(False)
        print(logN, L, K, dnum, batch, order, overlap, flush=True)
        assert np.array_equal(got[-1], want[1]) and all(np.array_equal(x, want[0]) for x in got[:-1])
        joint = any(k.startswith("conv_up_both_kernel") for k in names)
        assert joint == (order == "fp first" and logN >= 14 and not (overlap and batch == 30)), names


@pytest.mark.parametrize("batch", [23, 24, 82, 117])
def test_converted_part_through_the_cache_by_its_size(orc, batch):
    """Rescale of 12 limbs at N = 2^14, both arithmetics: the converted part is stored with ordinary accesses from 64 to 320 MiB and read
    so up to 224 MiB; 63, 66, 226 and 322 MiB."""
    ps = synth.mixed_params(14, [49, 55, 49] * 4, [59], 12, "cached")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(64 + batch)
    ct = _extreme(rng, ps.q_primes, ps.N, (3, 2))
    which = np.arange(batch) % 3
    d_ct, want = dev(ct)[dev(which)].contiguous(), dev(orc.rescale(ct, P))
    print("batch", batch, flush=True)
    ctx.profile_enable(True)
    try:
        got, names = ctx.rescale(ps.L, d_ct), set(ctx.profile_read())
    finally:
        ctx.profile_enable(False)
    assert bool((got == want[dev(which)]).all())
    assert any(n.startswith("conv_one_cached_kernel") for n in names) == (24 <= batch <= 82), names
    assert any(n.startswith("ks_final_cached_kernel") for n in names) == (batch == 24), names


@pytest.mark.parametrize("first,n,batch,ar", [(0, 8, 63, "FpAr"), (0, 8, 64, "FpAr"), (8, 4, 128, "IntAr"), (3, 9, 57, "AnyAr"), (3, 9, 56, "AnyAr")])
def test_transform_through_the_cache_by_its_size(orc, first, n, batch, ar):
    """The first forward pass stores with ordinary accesses from 64 MiB on: N = 2^14, ranges of either arithmetic and of both."""
    ps = synth.mixed_params(14, [49] * 8 + [55] * 4, [59], 12, "cached")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    x = _extreme(np.random.default_rng(64 + n), ps.primes[first:first + n], ps.N, (3,))
    which = np.arange(batch) % 3
    d_x, want = dev(x)[dev(which)].contiguous(), dev(orc.ntt_batch(x, P, first))
    print(ar, "batch", batch, flush=True)
    ctx.profile_enable(True)
    try:
        got, names = ctx.ntt(d_x, first), set(ctx.profile_read())
    finally:
        ctx.profile_enable(False)
    assert bool((got == want[dev(which)]).all())
    assert ("fwd_strided_cached_kernel<%s, 6>" % ar in names) == (n * batch >= 512), names


@pytest.mark.parametrize("logN,L,K,dnum,batch,up,dn", [
    (12, 24, 2, 12, 22, True, False), (12, 24, 2, 12, 20, False, False), (12, 48, 5, 6, 64, True, True),   # two, five and eight sources; no exchange at N = 2^12
    (13, 20, 10, 2, 77, True, True), (13, 20, 10, 2, 76, False, False),                                    # ten sources, 3080 and 3040 workgroups
    (14, 13, 3, 3, 64, True, True),                                                                        # a last workgroup of one target, a short last digit
    (15, 30, 6, 5, 13, True, True)])                                                                       # six sources, three words a lane half
def test_integer_targets_of_many_workgroups(orc, logN, L, K, dnum, batch, up, dn):
    """Conversions onto integer limbs from 3072 workgroups on: 256 lanes with two positions each."""
    ps = synth.mixed_params(logN, [55] * L, [59] * K, dnum, "halves")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(256 + logN + L)
    ct, key = _extreme(rng, ps.q_primes, ps.N, (3, 2)), _extreme(rng, ps.primes, ps.N, (dnum, 2))
    which, g = np.arange(batch) % 3, synth.galois_element(-3, logN)
    d_ct, want = dev(ct)[dev(which)].contiguous(), dev(np.stack([orc.hrot(c, g, key, P) for c in ct]))
    print(logN, L, K, "batch", batch, flush=True)
    ctx.profile_enable(True)
    try:
        got, names = ctx.hrot(d_ct, g, dev(key)), set(ctx.profile_read())
    finally:
        ctx.profile_enable(False)
    assert bool((got == want[dev(which)]).all())
    halves = {int(n.split(", ")[2]) for n in names if n.startswith("conv_int_kernel<%d, " % (logN - 8))}
    assert halves == {d for d, is_on in ((1, up), (2, dn)) if is_on}, names


def test_integer_targets_of_many_workgroups_from_seventeen_sources(orc):
    """The ModDown merged with a rescale: sixteen special primes and the last limb."""
    ps = synth.mixed_params(13, [55] * 24, [59] * 16, 2, "halves")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(1717)
    a, b, key = _extreme(rng, ps.q_primes, ps.N, (2, 2)), _extreme(rng, ps.q_primes, ps.N, (2, 2)), _extreme(rng, ps.primes, ps.N, (2, 2))
    which = np.arange(64) % 2
    want = dev(np.stack([orc.hmult_relin_rescale_level(x, y, key, P) for x, y in zip(a, b)]))
    print("seventeen sources", flush=True)
    ctx.profile_enable(True)
    try:
        got, names = ctx.hmult_relin_rescale_at(ps.L, dev(a)[dev(which)].contiguous(), dev(b)[dev(which)].contiguous(), dev(key)), set(ctx.profile_read())
    finally:
        ctx.profile_enable(False)
    assert bool((got == want[dev(which)]).all())
    assert "conv_int_kernel<5, 5, 2, 10>" in names, names
