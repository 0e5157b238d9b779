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


@pytest.mark.parametrize("n,batch", [(1, 1), (5, 5), (4, 6), (4, 16), (5, 13)])
def test_few_integer_limbs_at_n_2_13_take_two_passes(orc, n, batch):
    """N = 2^13: forward up to 64 integer limbs, inverse up to 24; ranges with an FP64 limb keep one kernel a limb."""
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
    assert ("fwd_strided_kernel<IntAr, 5>" in names) == (n * batch <= 64), names
    got, names = _kernels(ctx, lambda: ctx.intt(dev(x), first))
    assert np.array_equal(got, orc.ntt_batch(x, P, first, inverse=True))
    assert ("inv_contig_rows_kernel<IntAr, 5, 0>" in names) == (n * batch <= 24), names
    y = synth.uniform_residues(rng, ps.primes[:2], ps.N, lead=(2,))
    got, names = _kernels(ctx, lambda: ctx.intt(dev(y)))
    assert np.array_equal(got, orc.ntt_batch(y, P, 0, inverse=True)) and len(names) == 1, names
