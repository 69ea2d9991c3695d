"""Chains of one to eight groups, where a group's look-ahead band reaches the
groups that still read the positions it will replace: several hundred sweeps
with the widest band run through, and the double ones make the oracle's
decisions.  Tolerances: dE to 1e-10 in double (rounding of sums of a few
hundred terms of order 1), running against exact energy 1e-3 in float (500
sweeps of roundings of 1e-7 relative to terms of order 10).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sys(n, seed):
    from paper_1602_05716_amd import inputs
    sy = inputs.electrolyte(n // 2, n // 2, 1.0, -1.0, 1.0, 1.0, 0.02, 0.7)
    sy.xyz = inputs.random_start(sy, seed)
    return sy


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("n", [64, 100, 190, 256, 300, 384, 448, 512])
def test_short_chains_run_through(oracle, n, waves):
    from paper_1602_05716_amd import mc
    sy = _sys(n, 100 + n)
    print("[gpu-case] short chain n=%d waves=%d" % (n, waves), flush=True)
    with mc.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, precision="fp32", max_disp=1.0, band=4, resum_every=0,
                  waves=waves, wait_timeout_s=2.0) as ch:
        ch.sweep(500, 5)
        run, exact = ch.energy(exact=True)
        assert abs(run - exact) < 1e-3 * max(1.0, abs(exact))
        assert ch.stats()["moves"] == 500 * n
    sweeps, seed = 40, 0x51
    with mc.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, precision="fp64", max_disp=1.0, band=4, resum_every=0,
                  waves=waves, trace_moves=sweeps * n, wait_timeout_s=2.0) as ch:
        ch.sweep(sweeps, seed)
        acc, de = ch.trace(sweeps * n)
        x = ch.positions()
    ref = oracle.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, 2.0, seed=seed)
    r = ref.run(sweeps, trace=sweeps * n)
    assert np.array_equal(acc, r["acc"])
    assert np.max(np.abs(de - r["dE"]) / np.maximum(np.abs(r["dE"]), 1.0)) < 1e-10
    assert np.array_equal(x, ref.x)
