"""Parity of the passes that skip their reductions for narrow primes (needs an MI355X): primes on both sides of the bound 17 * 2^45, alone and within one
workgroup's targets, extreme residues, digit counts on both sides of the five products between reductions.  Bit for bit against
the oracle.
"""
import numpy as np
import pytest

from paper_2310_16530_amd import synth

from test_gpu_forms_by_size import _below
from test_gpu_linear_sums import _inputs
from test_gpu_mixed_primes import _every_composed_operation_once
from test_gpu_parity import dev, gpu_ctx, host, orc_params

pytestmark = pytest.mark.gpu
BOUND = 17 << 45


def _chain(name, logN, below, above, specials, dnum):
    """`below` primes just under the bound and `above` just over it, in turn."""
    two_n = 2 << logN
    lo, hi = list(_below(BOUND + 1, two_n, below)), list(synth.primes_above(BOUND, two_n, above))
    q = [p for k in range(max(below, above)) for p in lo[k:k + 1] + hi[k:k + 1]]
    return synth.ExplicitParamSet(name, logN, dnum, tuple(q), synth.primes_above(1 << specials, two_n, 2 if logN > 12 else 3))


@pytest.mark.parametrize("logN,below,above,specials,dnum", [
    (12, 6, 0, 59, 6), (12, 6, 0, 59, 1), (12, 7, 0, 50, 7),  # six and seven products a sum; FP64 special limbs above the bound
    (13, 3, 3, 59, 2), (14, 5, 2, 59, 7), (16, 4, 2, 59, 6), (16, 4, 0, 59, 2),
])
def test_every_operation_around_the_bound(orc, logN, below, above, specials, dnum):
    ps = _chain("narrow", logN, below, above, specials, dnum)
    print(logN, [p.bit_length() for p in ps.primes], flush=True)
    for seed in (2, 3):  # the second stream off and on, other levels
        _every_composed_operation_once(orc, ps, seed, corners=True)
    x = np.stack([np.full(ps.N, p - 1, dtype=np.uint64) for p in ps.q_primes])[None]
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    got = host(ctx.ntt(dev(x)))[0]
    for i, p in enumerate(ps.q_primes):
        assert np.array_equal(got[i], orc.ntt(x[0, i], logN, p, P.psi[i])), i


@pytest.mark.parametrize("n_rot", [5, 16, 17, 22])
def test_sums_over_rotations_around_the_bound(orc, n_rot):
    ps = _chain("narrow sums", 12, 4, 1, 59, 2)
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    gs, keys, ct, pt = _inputs(ps, n_rot, 3, 4100 + n_rot, ps.q_primes, (n_rot,))
    use = [keys[r % 3] for r in range(n_rot)]
    d_keys = [dev(k) for k in keys]
    got = host(ctx.hrot_hoisted_mac(dev(ct), gs, [d_keys[r % 3] for r in range(n_rot)], dev(pt)))
    assert np.array_equal(got, orc.hrot_hoisted_mac(ct, gs, use, pt, P))
