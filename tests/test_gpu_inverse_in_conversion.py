"""Parity of conversions from a single limb that repeat the inverse pass of their source (needs an MI355X): both sides of the sizes up to which
they do, at every ring degree, sources and targets of either arithmetic, both stream modes.  Bit for bit against the oracle, extreme
residues planted.
"""
import numpy as np
import pytest

from paper_2310_16530_amd import synth

from test_gpu_conversion_edges import _extreme
from test_gpu_forms_by_size import _kernels
from test_gpu_parity import dev, gpu_ctx, host, orc_params

pytestmark = pytest.mark.gpu


def _up(logN, L, batch):
    return batch * L * (L + 1) << (logN - 12) <= (640 if logN <= 13 else 512)


def _dn(logN, sources, targets, int_source, whole):
    """targets: their sizes in bits, integer arithmetic from 50 on; a launch for every run of one arithmetic, but one for all where whole"""
    tiles, n = sources << (logN - 12), len(targets)
    runs = 1 + sum((a >= 50) != (b >= 50) for a, b in zip(targets, targets[1:]))
    most = (448 if logN == 12 else 288) if whole else (512 if int_source else 768) if runs == 1 else 512 if runs == 2 and (not int_source or logN <= 13) else 0
    return tiles * n <= most and tiles * -(-n // 4) < 512


# (logN, q, p, batch): digits of one limb, one special prime; floors from 50 bits on are integer arithmetic
KEY_SWITCH = [(12, (35,) * 3, 36, 1), (12, (49,) * 8, 59, 8), (12, (49,) * 8, 59, 9), (12, (49, 55, 58, 49), 49, 2), (12, (55,) * 8, 59, 32), (12, (49,) * 8, 59, 33),
              (13, (49,) * 5, 59, 10), (13, (49,) * 5, 59, 11), (13, (55, 49, 60), 60, 2), (14, (49,) * 4, 59, 5), (14, (49,) * 4, 59, 6), (14, (49,) * 4, 59, 7), (14, (55, 49, 58), 48, 3),
              (15, (49, 49), 59, 9), (15, (55, 56), 59, 10), (15, (55, 56), 59, 11), (16, (49, 49), 48, 4), (16, (58, 49), 59, 5), (16, (49,) * 2, 59, 9)]


@pytest.mark.parametrize("logN,q,p,batch", KEY_SWITCH)
def test_key_switches(orc, logN, q, p, batch):
    ps = synth.mixed_params(logN, list(q), [p], len(q), "repeated inverse")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(9100 + logN + batch)
    key = synth.uniform_residues(rng, ps.primes, ps.N, lead=(ps.dnum, 2))
    ct1, ct2 = (_extreme(rng, ps.q_primes, ps.N, (batch, 2)) for _ in range(2))
    d_key, d1, d2 = dev(key), dev(ct1), dev(ct2)
    g, L, whole = synth.galois_element(5, logN), ps.L, logN <= 13
    up, dn = _up(logN, L, batch), _dn(logN, 2 * batch, q, p >= 50, False)
    for overlap in (False, True):
        ctx.set_overlap(overlap)
        try:
            print(logN, L, "batch", batch, "overlap", overlap, flush=True)
            hm, names = _kernels(ctx, lambda: ctx.hmult_relin_at(L, d1, d2, d_key))
            hr, _ = _kernels(ctx, lambda: ctx.hrot_at(L, d1, g, d_key))
            ks, _ = _kernels(ctx, lambda: ctx.keyswitch_at(L, dev(ct1[:, 0]), d_key))
        finally:
            ctx.set_overlap(False)
        for b in range(0, batch, 8 if logN < 15 else batch - 1):
            assert np.array_equal(hm[b], orc.hmult_relin_level(ct1[b], ct2[b], key, P)), b
            assert np.array_equal(hr[b], orc.hrot_level(ct1[b], g, key, P)), b
            assert np.array_equal(ks[b], orc.keyswitch_level(ct1[b, 0], key, P)), b
        if whole:
            assert any(n.startswith("inv_whole_conv_one_kernel") for n in names) == up, names
            assert any(n.startswith("inv_strided_kernel") for n in names) == (not dn), names
        else:
            assert any(n.startswith("inv_conv_one_kernel") for n in names) == up, names
            assert any(n.startswith("inv_strided_kernel") for n in names) == (not (up and dn)), names


RESCALE = [(12, (49,) * 8, 32), (12, (49,) * 8, 33), (12, (55, 49, 58), 4), (13, (49,) * 7, 12), (13, (49,) * 7, 13), (13, (55,) * 5, 12), (13, (55,) * 5, 13),
           (14, (49, 49), 63), (14, (49, 49), 64), (14, (49, 55, 58), 9), (14, (49, 55, 49), 9), (14, (49, 55, 49), 33), (15, (55, 49, 58, 49), 2), (14, (49, 55) * 4, 3), (15, (49,) * 7, 8), (15, (49,) * 7, 9), (16, (49,) * 3, 12), (16, (49,) * 3, 13), (16, (49, 50, 55), 8)]


@pytest.mark.parametrize("logN,q,batch", RESCALE)
def test_rescales(orc, logN, q, batch):
    ps = synth.mixed_params(logN, list(q), [59], 1, "repeated inverse, rescale")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(9300 + logN + batch)
    whole = logN <= 13
    for ell in (ps.L, 2):
        ct = _extreme(rng, ps.q_primes[:ell], ps.N, (batch, 2))
        got, names = _kernels(ctx, lambda: ctx.rescale(ell, dev(ct)))
        print(logN, "level", ell, "batch", batch, sorted(names), flush=True)
        assert np.array_equal(got[::5], orc.rescale(np.ascontiguousarray(ct[::5]), P)), ell
        int_source = q[ell - 1] >= 50
        few_integer = logN == 13 and int_source and 2 * batch <= 24
        want = _dn(logN, 2 * batch, q[:ell - 1], int_source, whole) and not few_integer
        if whole:
            assert any(n.startswith("inv_whole_conv_one_kernel") for n in names) == want, names
        else:
            assert any(n.startswith("inv_strided_kernel") for n in names) == (not want), names


@pytest.mark.parametrize("logN,q,p", [(12, (49,) * 3, 59), (13, (55, 49, 58), 49), (14, (49, 49), 59)])
def test_sums_of_rotations(orc, logN, q, p):
    ps = synth.mixed_params(logN, list(q), [p], len(q), "repeated inverse, sums")
    ctx, P = gpu_ctx(ps), orc_params(orc, ps)
    rng = np.random.default_rng(9500 + logN)
    gs = [synth.galois_element(r, logN) for r in (1, 3, -2)]
    keys = [synth.uniform_residues(rng, ps.primes, ps.N, lead=(ps.dnum, 2)) for _ in gs]
    ct, pt = _extreme(rng, ps.q_primes, ps.N, (2,)), _extreme(rng, ps.primes, ps.N, (3,))
    d_ct, d_keys = dev(ct), [dev(k) for k in keys]
    q_pt = np.ascontiguousarray(pt[:, : ps.L])
    assert np.array_equal(host(ctx.hrot_hoisted_mac(d_ct, gs, d_keys, dev(q_pt))), orc.hrot_hoisted_mac(ct, gs, keys, q_pt, P))
    assert np.array_equal(host(ctx.hrot_dh_mac(d_ct, gs, d_keys, dev(pt))), orc.hrot_dh_mac_level(ct, gs, keys, pt, P))
    two = np.stack([pt[:2], pt[1:]])
    got = host(ctx.lintrans_bsgs_at(ps.L, d_ct, gs[:2], d_keys[:2], gs[1:], d_keys[1:], dev(two)))
    assert np.array_equal(got, orc.lintrans_bsgs_level(ct, gs[:2], keys[:2], gs[1:], keys[1:], two, P))
