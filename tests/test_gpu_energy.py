"""The double-precision energy re-sum (mc_energy's exact value) and the
running-energy scan against the oracle's plain double loop, at the sizes where
the re-sum's tiling can go wrong: one ion, the edges of a 64-ion group and of
a 128-ion super-row, an odd number of groups (a last super-row of one group),
one and several blocks per pair of super-rows, and the batched launch.

Tolerance: every term is within one unit in the last place of its rounded
value (2^-52 relative, as sqrt followed by a division), and a sum of m terms
in any order is within m 2^-53 of sum |term| (m <= n^2 / 2; in practice far
less): |E - E_ref| <= (2^-51 + 2 n 2^-53) sum |term| is used, n for the
longest running sum either side forms.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sys(n, seed, two_to_one=False):
    from paper_1602_05716_amd import inputs
    if n == 1:
        sy = inputs.electrolyte(1, 0, 0.0, 0.0, 1.0, 1.0, 0.05, 0.7)
        sy.xyz = np.zeros((1, 3))
        return sy
    if two_to_one:
        sy = inputs.electrolyte(n // 3, n - n // 3, 2.0, -1.0, 1.0, 0.8, 0.05, 0.9)
    else:
        sy = inputs.electrolyte(n // 2, n - n // 2, 1.0, -1.0, 1.0, 1.0, 0.05, 0.7)
    sy.q = sy.q.copy()
    sy.q[-1] -= sy.q.sum()  # neutral whatever the count
    sy.xyz = inputs.random_start(sy, seed)
    return sy


def _bound(x, q, lB):
    d = np.sqrt(((x[:, None, :] - x[None, :, :]) ** 2).sum(-1))
    np.fill_diagonal(d, np.inf)
    return (2.0 ** -51 + 2 * len(q) * 2.0 ** -53) * 0.5 * lB * float((np.abs(q[:, None] * q[None, :]) / d).sum())


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 128, 129, 192, 257, 700, 1100, 2113])
def test_resum_matches_the_plain_loop(oracle, n, precision):
    from paper_1602_05716_amd import mc
    sy = _sys(n, 900 + n, two_to_one=n % 2 == 1)
    print("[gpu-case] re-sum n=%d %s" % (n, precision), flush=True)
    with mc.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, precision=precision, max_disp=0.8, resum_every=0) as ch:
        for sweeps in (0, 1, 2):  # both position images
            ch.sweep(sweeps, 11)
            x = ch.positions()
            _, e = ch.energy(exact=True)
            assert abs(e - oracle.total_energy(x, sy.q, sy.lB)) <= _bound(x, sy.q, sy.lB)


def test_resum_of_a_batch(oracle):
    from paper_1602_05716_amd import mc
    systems = [_sys(n, 40 + n) for n in (2, 66, 130, 511, 900)]
    print("[gpu-case] re-sum of a batch", flush=True)
    with mc.Batch(systems, precision="fp32", resum_every=0) as b:
        b.sweep(1, 3)
        for k, sy in enumerate(systems):
            x = b.positions(k)
            _, e = b.energy(k, exact=True)
            assert abs(e - oracle.total_energy(x, sy.q, sy.lB)) <= _bound(x, sy.q, sy.lB)


def test_energy_series_does_not_depend_on_the_launches():
    """Per-sweep running energies: the same bits whether the sweeps run in
    one launch (and one scan) or in several, ragged group counts included."""
    from paper_1602_05716_amd import mc
    sy = _sys(4229, 5)  # 67 groups: more than one per lane of the scan
    print("[gpu-case] energy series n=%d" % sy.n, flush=True)
    series = []
    for cuts in ([19], [1, 7, 11], [8, 9, 2]):
        with mc.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, precision="fp32", max_disp=1.0, resum_every=0) as ch:
            for c in cuts:
                ch.sweep(c, 21)
            series.append(ch.energy_series(19))
            assert ch.energy() == series[-1][-1]
    assert np.array_equal(series[0], series[1]) and np.array_equal(series[0], series[2])
