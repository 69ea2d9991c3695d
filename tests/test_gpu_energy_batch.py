"""A chain's energy audit, and so its running energy after a re-sum, has the
bits of the same chain alone in a handle, whatever chains share its handle:
the order of the double sum depends on the chain only."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_resum_does_not_depend_on_the_other_chains(precision):
    from paper_1602_05716_amd import inputs, mc
    systems = []
    for n in (100, 700, 2300, 4100) + (6000,) * 20:
        sy = inputs.electrolyte(n // 2, n // 2, 1.0, -1.0, 1.0, 1.0, 0.05, 0.7)
        sy.xyz = inputs.random_start(sy, 400 + n) if len(systems) < 5 else systems[4].xyz
        systems.append(sy)
    opts = dict(precision=precision, resum_every=2, waves=4, band=1)
    print("[gpu-case] re-sums of a batch and of its chains alone,", precision, flush=True)
    with mc.Batch(systems, max_disp=[0.5] * len(systems), **opts) as b:
        start = [b.energy(k, exact=True) for k in range(5)]
        b.sweep(4, 3)
        end = [b.energy(k, exact=True) for k in range(5)]
        series = [b.energy_series(k, 4) for k in range(5)]
    for k in range(5):
        sy = systems[k]
        with mc.Batch([sy], max_disp=[0.5], chain_ids=[k], **opts) as a:
            assert a.energy(0, exact=True) == start[k]
            a.sweep(4, 3)
            assert a.energy(0, exact=True) == end[k]
            assert np.array_equal(a.energy_series(0, 4), series[k])
