"""Parity of the transforms where their forms change (needs an MI355X): limbs that one workgroup holds (N <= 2^13) and limbs
in two passes, ranges of one arithmetic and ranges that mix both, with and without the second stream, every load of the
inverse transform (plain, product of two ciphertexts, rotation).  Bit for bit against the oracle, extreme residues planted.
"""
import numpy as np
import pytest

from paper_2310_16530_amd import synth

from test_gpu_parity import dev, gpu_ctx, host, orc_params

pytestmark = pytest.mark.gpu

FLOORS = {"fp_then_int": ([49, 49, 49], [59, 59]), "alternating": ([49, 55, 36, 58], [59, 49])}


@pytest.mark.parametrize("logN", [12, 13, 14, 15, 16])
@pytest.mark.parametrize("chain", sorted(FLOORS))
def test_transform_forms(orc, chain, logN):
    qf, pf = FLOORS[chain]
    ps = synth.mixed_params(logN, qf, pf, 2, chain + str(logN))
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(5000 + logN)
    D, N = ps.L + ps.K, ps.N
    x = synth.uniform_residues(rng, ps.primes, N, lead=(3,))
    for i, p in enumerate(ps.primes):
        x[1, i, :] = p - 1
        x[2, i, : N // 2] = 0
    want, want_inv = orc.ntt_batch(x, P, 0), orc.ntt_batch(x, P, 0, inverse=True)
    for first, n in ((0, D), (0, 1), (1, 2), (ps.L - 1, 2), (ps.L, ps.K)):
        print(chain, logN, "limbs", first, n, flush=True)
        sub = np.ascontiguousarray(x[:, first:first + n])
        assert np.array_equal(host(ctx.ntt(dev(sub), first)), want[:, first:first + n])
        assert np.array_equal(host(ctx.intt(dev(sub), first)), want_inv[:, first:first + n])
        assert np.array_equal(host(ctx.ntt(dev(sub[:1]), first)), want[:1, first:first + n])
    ct = synth.uniform_residues(rng, ps.q_primes, N, lead=(2, 2))
    key = synth.uniform_residues(rng, ps.primes, N, lead=(ps.dnum, 2))
    gs = [synth.galois_element(r, logN) for r in (1, -3)]
    rks = [key, synth.uniform_residues(rng, ps.primes, N, lead=(ps.dnum, 2))]
    pt = synth.uniform_residues(rng, ps.primes, N, lead=(2,))
    wants = (orc.hmult_relin(ct[0], ct[1], key, P), orc.hrot(ct[0], gs[1], rks[1], P),
             orc.hrot_hoisted_mac(ct[0], gs, rks, np.ascontiguousarray(pt[:, :ps.L]), P),
             orc.hrot_dh_mac_level(ct[0], gs, rks, pt, P), orc.rescale(ct, P))
    d_rks = [dev(k) for k in rks]
    for overlap in (False, True):
        print(chain, logN, "overlap", overlap, flush=True)
        ctx.set_overlap(overlap)
        try:
            assert np.array_equal(host(ctx.hmult_relin(dev(ct[0]), dev(ct[1]), d_rks[0])), wants[0])
            assert np.array_equal(host(ctx.hrot(dev(ct[0]), gs[1], d_rks[1])), wants[1])
            assert np.array_equal(host(ctx.hrot_hoisted_mac(dev(ct[0]), gs, d_rks, dev(pt[:, :ps.L]))), wants[2])
            assert np.array_equal(host(ctx.hrot_dh_mac(dev(ct[0]), gs, d_rks, dev(pt))), wants[3])
            assert np.array_equal(host(ctx.rescale(ps.L, dev(ct))), wants[4])
        finally:
            ctx.set_overlap(False)
