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
SINGLE = [(15, (49, 49, 49, 49), 59, 3), (15, (49, 49, 49, 49), 59, 14), (15, (49, 49, 49, 49), 59, 32),
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
