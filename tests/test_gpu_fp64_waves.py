"""Double handles choose eight waves per workgroup by themselves and go to
four when a surrogate is installed.  Each move's pair sum is the same terms
in another order of double additions: dE to 1e-10, decisions and positions
exactly, against a handle on four waves throughout; a size with padding, one
group, and more groups than the band.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,band", [(64, 0), (128, 1), (512, 1), (514, 2), (2048, 2), (2050, 4)])
def test_automatic_band_of_double_chains(oracle, n, band):
    """The automatic band by size, the oracle's decisions on it, and the
    widest the two-stage kernel holds once a surrogate is installed."""
    from paper_1602_05716_amd import inputs, mc, surrogate
    sy = inputs.electrolyte(n // 2, n // 2, 1.0, -1.0, 1.0, 1.0, 0.04, 0.7)
    sy.xyz = inputs.random_start(sy, 18)
    with mc.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, precision="fp64", max_disp=0.8, resum_every=0,
                  trace_moves=2 * n) as ch:
        assert ch.stats()["band"] == band
        ch.sweep(2, 12)
        acc, de = ch.trace(2 * n)
        ch.set_surrogate(surrogate.truncated_coulomb_params(2.0), 0.5, True)
        assert ch.stats()["band"] == min(3, (n + 63) // 64 - 1)
    r = oracle.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, 1.6, seed=12).run(2, trace=2 * n)
    assert np.array_equal(acc, r["acc"])
    assert np.max(np.abs(de - r["dE"]) / np.maximum(np.abs(r["dE"]), 1.0)) < 1e-10


@pytest.mark.parametrize("n,per_ion", [(50, False), (130, True), (1000, False)])
def test_automatic_waves_and_surrogate(n, per_ion):
    from paper_1602_05716_amd import inputs, mc, surrogate
    sy = inputs.electrolyte(n // 2, n // 2, 1.0, -1.0, 1.0, 0.8 if per_ion else 1.0, 0.04, 0.7)
    sy.xyz = inputs.random_start(sy, 17)
    p = surrogate.truncated_coulomb_params(2.0)
    sweeps = 3
    got = {}
    for waves in (0, 4):
        print("[gpu-case] n=%d waves=%d" % (n, waves), flush=True)
        with mc.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, precision="fp64", max_disp=0.8, resum_every=0,
                      trace_moves=2 * sweeps * n, waves=waves, da_rcut=2.0, band=2) as ch:
            ch.sweep(sweeps, 9)
            first = ch.stats()["waves"]
            ch.set_surrogate(p, 0.5, True)
            ch.sweep(sweeps, 9)
            st = ch.stats()
            got[waves] = (first, st["waves"], st["da_kernel"], ch.positions(), ch.trace(2 * sweeps * n), ch.energy())
    assert got[0][:3] == (8, 4, 1) and got[4][:3] == (4, 4, 1)
    assert np.array_equal(got[0][3], got[4][3])
    (a0, d0), (a4, d4) = got[0][4], got[4][4]
    assert np.array_equal(a0, a4)
    ok = np.isfinite(d4)
    assert np.array_equal(ok, np.isfinite(d0)) and np.max(np.abs(d0[ok] - d4[ok]), initial=0.0) < 1e-10
    assert abs(got[0][5] - got[4][5]) < 1e-9
