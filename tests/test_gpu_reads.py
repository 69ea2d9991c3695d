"""Reads of a chain's state at the sizes where the route changes: positions
arrive packed in pinned memory up to 16384 ions (whole fours of values, so
remainders of 3 n by 4 matter) and as they lie above; a batch reads each of
its chains by its own size.  Exact comparisons: nothing is computed.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _ions(n, rng):
    # a simple cubic lattice of neutral-by-pairs ions well inside the sphere
    m = int(np.ceil(n ** (1.0 / 3.0)))
    g = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n]
    xyz = 2.0 * (g - 0.5 * (m - 1)) + rng.uniform(-0.3, 0.3, (n, 3))
    q = np.where(np.arange(n) % 2 == 0, 1.0, -1.0)
    q[-1] -= q.sum()
    return xyz, q, np.ones(n), 2.0 * m


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_positions_of_every_route(precision):
    from paper_1602_05716_amd import mc
    rng = np.random.default_rng(5)
    as_held = np.float32 if precision == "fp32" else np.float64
    sizes = [1, 2, 3, 64, 65, 333, 16384, 16385]
    specs = [_ions(n, rng) + (0.7,) for n in sizes]
    print("[gpu-case] batch of", sizes, precision, flush=True)
    with mc.Batch(specs, max_disp=[0.4] * len(sizes), precision=precision, resum_every=0) as h:
        for _ in range(2):
            for k in reversed(range(len(sizes))):
                assert np.array_equal(h.positions(k), specs[k][0].astype(as_held).astype(np.float64)), sizes[k]
                st = h.stats(k)
                assert st["sweeps"] == 0 and st["moves"] == 0 and st["accepted"] == 0 and st["resums"] == 0
        h.sweep(1, 3)
        for k, n in enumerate(sizes):
            st = h.stats(k)
            moved = int(np.any(h.positions(k) != specs[k][0].astype(as_held), axis=1).sum())
            assert st["moves"] == n and st["accepted"] == moved, n
            assert h.energy(k) == h.energy_series(k, 1)[0]
