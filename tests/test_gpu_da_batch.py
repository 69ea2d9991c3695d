"""A batch with a surrogate on one of its chains: the two-stage kernel runs
every chain of the handle, and the others must go on as plain chains (the
kernel holds a narrower band than theirs).  Double decisions against the
oracle exactly, dE to 1e-10, as for single chains.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_plain_chain_beside_a_two_stage_chain(oracle):
    from paper_1602_05716_amd import inputs, mc, surrogate
    sys_ = []
    for k, n in enumerate((512, 2304)):
        sy = inputs.electrolyte(n // 2, n // 2, 1.0, -1.0, 1.0, 1.0, 0.04, 0.7)
        sy.xyz = inputs.random_start(sy, 60 + k)
        sys_.append(sy)
    n, sweeps, seed = 2304, 3, 31
    print("[gpu-case] batch, surrogate on chain 0 only", flush=True)
    with mc.Batch(sys_, max_disp=[0.8, 0.8], precision="fp64", resum_every=0, trace_moves=sweeps * n) as h:
        h.set_surrogate(surrogate.truncated_coulomb_params(2.0), 0.5, True, chain=0)
        assert h.stats(1)["da_kernel"] == 1 and h.stats(1)["da_active"] == 0 and h.stats(1)["band"] == 3
        h.sweep(sweeps, seed)
        acc, de = h.trace(1, sweeps * n)
    sy = sys_[1]
    r = oracle.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, 1.6, seed=seed, chain=1).run(sweeps, trace=sweeps * n)
    assert np.array_equal(acc, r["acc"])
    assert np.max(np.abs(de - r["dE"]) / np.maximum(np.abs(r["dE"]), 1.0)) < 1e-10
