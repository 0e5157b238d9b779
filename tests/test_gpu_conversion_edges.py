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
