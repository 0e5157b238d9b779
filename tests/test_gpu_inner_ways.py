"""Parity of the key inner product where its digits are shared by the wavefronts of a workgroup (needs an MI355X): digit
counts below, at and above the four wavefronts, batches on either side of the grid size at which the sharing ends, every
operation's own-digit operand, both arithmetics, the merged rescale.  Bit for bit against the oracle.
"""
import numpy as np
import pytest

from paper_2310_16530_amd import synth

from test_gpu_parity import dev, gpu_ctx, host, orc_params

pytestmark = pytest.mark.gpu

# (logN, L, K, dnum, q bits, p bits), batches
SHAPES = [((12, 2, 1, 2, 49, 59), (1, 5)), ((13, 4, 1, 4, 49, 59), (1, 13)), ((12, 9, 2, 5, 55, 59), (1, 3)),
          ((14, 9, 1, 9, 49, 59), (1, 4)), ((13, 6, 6, 1, 49, 59), (2,)), ((15, 8, 2, 4, 49, 59), (1, 2, 3))]


@pytest.mark.parametrize("shape,batches", SHAPES)
def test_inner_product_with_shared_digits(orc, shape, batches):
    ps = synth.small_params(*shape)
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(99000 + sum(shape))
    key = synth.uniform_residues(rng, ps.primes, ps.N, lead=(ps.dnum, 2))
    for i, p in enumerate(ps.primes):
        key[:, :, i, : ps.N // 2] = p - 1
    d_key, g = dev(key), synth.galois_element(-2, ps.logN)
    for batch in batches:
        print(shape, "batch", batch, flush=True)
        ct1, ct2 = (synth.uniform_residues(rng, ps.q_primes, ps.N, lead=(batch, 2)) for _ in range(2))
        for i, p in enumerate(ps.q_primes):
            ct1[..., i, : ps.N // 3] = p - 1
        d1, d2 = dev(ct1), dev(ct2)
        ks, hr = host(ctx.keyswitch(dev(ct1[:, 1]), d_key)), host(ctx.hrot(d1, g, d_key))
        hm, hmr = host(ctx.hmult_relin(d1, d2, d_key)), host(ctx.hmult_relin_rescale_at(ps.L, d1, d2, d_key))
        for b in {0, batch - 1}:
            assert np.array_equal(ks[b], orc.keyswitch(ct1[b, 1], key, P)), b
            assert np.array_equal(hr[b], orc.hrot(ct1[b], g, key, P)), b
            assert np.array_equal(hm[b], orc.hmult_relin(ct1[b], ct2[b], key, P)), b
            assert np.array_equal(hmr[b], orc.hmult_relin_rescale_level(ct1[b], ct2[b], key, P)), b
