"""Parity of the kernel that forms several giant-step sums at once (needs an MI355X): one digit and more than an unreduced sum holds, fewer
baby steps than wavefronts that share a row, both sides of the row count from which they do not, chains of integer primes alone.
Bit for bit against the oracle.
"""
import numpy as np
import pytest

from paper_2310_16530_amd import synth

from test_gpu_forms_by_size import _kernels
from test_gpu_linear_sums import _inputs
from test_gpu_parity import dev, gpu_ctx, orc_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("logN,q,p,dnum,steps", [
    (12, (49, 49), (59,) * 3, 1, ((1, 2), (2, 3), (3, 4))),  # one digit; wavefronts without a rotation
    (12, (49, 60, 50, 58, 49, 49, 49), (48, 60), 7, ((5, 4),)),  # seven digits, both arithmetics
    (13, (49,) * 23, (59,) * 4, 6, ((5, 2),)),  # 1728 rows: four wavefronts share each
    (13, (49,) * 24, (59,) * 4, 6, ((3, 3),)),  # 1792: one wavefront each
    (12, (49,) * 24, (59,) * 3, 6, ((2, 2), (1, 3))),  # 864 rows: two rotations shared by four wavefronts, one by none
    (12, (49,) * 24, (59,) * 4, 6, ((2, 2), (1, 3))),  # 896: neither
    (13, (55,) * 12, (59,) * 4, 3, ((2, 4), (1, 4))),  # integer primes alone
])
def test_several_sums_in_one_kernel(orc, logN, q, p, dnum, steps):
    ps = synth.mixed_params(logN, list(q), list(p), dnum, "giant sums")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    n1, n2 = max(s[0] for s in steps), max(s[1] for s in steps)
    gs, keys, ct, pt = _inputs(ps, n1 + n2, 3, 3100 + logN + dnum, ps.primes, (n2, n1))
    d_ct, d_keys = dev(ct), [dev(k) for k in keys]
    for a, b in steps:
        print(logN, "baby", a, "giant", b, flush=True)
        use = np.ascontiguousarray(pt[:b, :a])
        want = orc.lintrans_bsgs_level(ct, gs[:a], [keys[r % 3] for r in range(a)], gs[n1:n1 + b], [keys[(r + 1) % 3] for r in range(b)], use, P)
        got, names = _kernels(ctx, lambda: ctx.lintrans_bsgs_at(ps.L, d_ct, gs[:a], [d_keys[r % 3] for r in range(a)], gs[n1:n1 + b],
                                                                [d_keys[(r + 1) % 3] for r in range(b)], dev(use)))
        assert np.array_equal(got, want), (a, b)
        form = "dh_accum_kernel<%s, 2, %d>" % ("IntAr" if min(q + p) > 49 else "AnyAr", b)
        assert form in names and not any(k.startswith("bsgs_mac_kernel") for k in names), names
