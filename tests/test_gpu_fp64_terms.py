"""The double path's pair terms and its eight-wave kernel for per-ion
diameters.

1 / r is formed from the hardware's estimate by one third-order step: the step
itself is off by far less than a rounding, its last addition rounds once (half
a unit in the last place) and the correction it adds, below 2^-24 of the
result, carries its own roundings along: at most one unit in the last place,
against a rounded square root and division (1.5).  Measured here through the
exact energy of two ions of opposite unit charge at l_B = 1, which is -1 / r,
at distances whose squares are whole numbers of 2^-2k and so exact.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_reciprocal_distance_to_one_unit_in_the_last_place():
    from paper_1602_05716_amd import mc
    rng = np.random.default_rng(7)
    worst = 0.0
    for k in range(-12, 13, 2):
        d = rng.integers(1 << 10, 1 << 20, (250, 3)).astype(np.float64)
        systems = []
        for v in d * 2.0 ** k:
            x = np.array([[0.0, 0.0, 0.0], v])
            systems.append((x, np.array([1.0, -1.0]), np.full(2, 2.0 ** (k + 8)), 2.0 ** (k + 22), 1.0))
        print("[gpu-case] 250 pairs, scale 2^%d" % k, flush=True)
        with mc.Batch(systems, precision="fp64", resum_every=0) as b:
            e = np.array([b.energy(c, exact=True)[1] for c in range(len(systems))])
        r2 = (d.astype(np.longdouble) ** 2).sum(1)
        ref = -(np.longdouble(2.0) ** -k) / np.sqrt(r2)
        ulp = np.spacing(np.abs(ref.astype(np.float64)))
        worst = max(worst, float((np.abs(e.astype(np.longdouble) - ref) / ulp).max()))
    print("[gpu-case] off by at most %.3f units in the last place" % worst, flush=True)
    assert worst <= 1.0 + 2.0 ** -10  # (the reference: 64-bit mantissas)


@pytest.mark.parametrize("n,sweeps", [(1998, 3), (6000, 2)])
def test_eight_waves_per_ion_diameters(oracle, n, sweeps):
    """Decisions and positions exactly, dE to 1e-10 (rounding of sums of a
    few thousand terms of order 1), on automatic waves and band."""
    from paper_1602_05716_amd import inputs, mc
    sy = inputs.electrolyte(n // 3, n - n // 3, 2.0, -1.0, 1.0, 0.8, 0.05, 0.7)
    sy.xyz = inputs.random_start(sy, 33)
    print("[gpu-case] double, per-ion diameters, n=%d" % n, flush=True)
    with mc.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, precision="fp64", max_disp=0.8, resum_every=0,
                  trace_moves=sweeps * n) as ch:
        ch.sweep(sweeps, 12)
        st = ch.stats()
        assert st["waves"] == 8 and st["band"] == (2 if n <= 2048 else 4)
        acc, de = ch.trace(sweeps * n)
        x = ch.positions()
    ref = oracle.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, 1.6, seed=12)
    r = ref.run(sweeps, trace=sweeps * n)
    assert np.array_equal(acc, r["acc"])
    assert np.max(np.abs(de - r["dE"]) / np.maximum(np.abs(r["dE"]), 1.0)) < 1e-10
    assert np.array_equal(x, ref.x)
