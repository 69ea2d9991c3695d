"""A refused mc_set_surrogate leaves the handle as it was: a float batch with
more chains than the two-stage kernel has co-resident workgroups (it runs one
workgroup per compute unit, the plain four-wave kernel two)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_refused_surrogate_changes_nothing():
    from paper_1602_05716_amd import inputs, mc, surrogate
    sy = inputs.electrolyte(160, 160, 1.0, -1.0, 1.0, 1.0, 0.02, 0.7)
    sy.xyz = inputs.random_start(sy, 5)
    many = [sy] * 276  # 256 compute units
    opts = dict(precision="fp32", waves=4, resum_every=0, da_window=3)
    got = []
    for refuse in (False, True):
        print("[gpu-case] %d chains, surrogate %s" % (len(many), "refused" if refuse else "not asked for"), flush=True)
        with mc.Batch(many, max_disp=[0.5] * len(many), **opts) as b:
            before = [b.stats(k) for k in (0, len(many) - 1)]
            assert before[0]["band"] == 4
            if refuse:
                for chain in (-1, 0):
                    with pytest.raises(mc.MCError) as ei:
                        b.set_surrogate(surrogate.truncated_coulomb_params(2.0), 0.5, True, chain=chain)
                    assert ei.value.code == -1 and "co-resident" in str(ei.value)
            assert [b.stats(k) for k in (0, len(many) - 1)] == before
            wg, _ = b.schedule()
            b.set_schedule(wg)  # uploads the chains' descriptors again
            b.timing_reset()
            b.sweep(4, 8)
            st = [b.stats(k) for k in (0, len(many) - 1)]
            got.append([(s["band"], s["da_kernel"], s["da_active"], s["accepted"]) for s in st] +
                       [b.energy_series(0, 4).tolist(), b.positions(0).tolist(), b.positions(len(many) - 1).tolist()])
    assert got[0] == got[1]
