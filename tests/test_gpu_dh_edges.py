"""Parity of the double-hoisted accumulation where its forms change (needs an MI355X): rotation counts around the number
of wavefronts that share a row and around one launch's limit, digit counts around the terms an unreduced sum holds (6 on
FP64 limbs, 8 on integer ones, b times P being one more), and grids on either side of the row-sharing rule.  Bit for bit
against the oracle, extreme residues planted.
"""
import numpy as np
import pytest

from paper_2310_16530_amd import synth

from test_gpu_parity import dev, gpu_ctx, host, orc_params

pytestmark = pytest.mark.gpu

# (logN, L, K, dnum, q bits, p bits), rotation counts
SHAPES = [((12, 3, 1, 3, 49, 59), (1, 2, 4, 5, 9)), ((12, 6, 1, 6, 49, 59), (1, 3, 8)), ((12, 9, 1, 9, 49, 59), (2, 7)),
          ((12, 9, 1, 9, 55, 59), (1, 7)), ((12, 8, 1, 8, 55, 59), (3,)), ((12, 2, 1, 2, 49, 59), (33, 65)),
          ((16, 8, 2, 4, 49, 59), (1, 7, 8))]


@pytest.mark.parametrize("shape,counts", SHAPES)
def test_double_hoisted_sum_at_the_edges_of_its_forms(orc, shape, counts):
    ps = synth.small_params(*shape)
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(88000 + sum(shape))
    n = max(counts)
    gs = [synth.galois_element((-1) ** r * (r // 2 + 1), ps.logN) for r in range(n)]
    keys = [synth.uniform_residues(rng, ps.primes, ps.N, lead=(ps.dnum, 2)) for _ in range(min(n, 9))]
    ct = synth.uniform_residues(rng, ps.q_primes, ps.N, lead=(2,))
    pt = synth.uniform_residues(rng, ps.primes, ps.N, lead=(n,))
    for i, p in enumerate(ps.primes):
        keys[0][:, :, i, : ps.N // 2] = p - 1
        pt[0, i, : ps.N // 4] = p - 1
        if i < ps.L:
            ct[:, i, : ps.N // 8] = p - 1
    rks = [keys[r % len(keys)] for r in range(n)]
    d_keys = [dev(k) for k in keys]
    for m in counts:
        print(shape, "rotations", m, flush=True)
        got = host(ctx.hrot_dh_mac(dev(ct), gs[:m], [d_keys[r % len(keys)] for r in range(m)], dev(pt[:m])))
        assert np.array_equal(got, orc.hrot_dh_mac_level(ct, gs[:m], rks[:m], pt[:m], P)), m
