"""The training kernels at the batches where their tiles end: one and a few
blocks of 32 pairs, and row counts 2 * batch that leave a remainder after the
groups of 8 blocks of 32 rows a weight-gradient wave keeps in flight.

Bound: the forward and backward passes round every hidden value and every
gradient row to bfloat16 (relative 2^-9, independently), at most three such
roundings in a row: about 3 * 2^-9 = 6e-3 of a block's norm, so 1e-2.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BLOCKS = [("W1", 0, 128 * 128), ("b1", 128 * 128, 128), ("W2", 128 * 128 + 128, 128 * 128),
          ("b2", 2 * 128 * 128 + 128, 128), ("w3", 2 * 128 * 128 + 256, 128)]


@pytest.mark.parametrize("batch", [32, 96, 128, 160, 288, 1024, 1056])
def test_gradients_at_tile_remainders(oracle, batch):
    from paper_1602_05716_amd import mc
    rng = np.random.default_rng(1000 + batch)
    p = oracle.bf16(rng.normal(0.0, 0.08, oracle.da_nparam()))
    f = rng.integers(0, 256, (batch, 256)).astype(np.uint8)
    f[:, ::3] %= 5
    y = rng.normal(0.0, 1.0, batch)
    print("[gpu-case] mlp grad batch=%d" % batch, flush=True)
    loss, g = mc.mlp_grad(f, y, p)
    ref_loss, ref_g = oracle.mlp_loss_grad(p, f[:, :128].astype(float), f[:, 128:].astype(float), y)
    assert loss == pytest.approx(ref_loss, rel=2e-3)
    for name, o, n in BLOCKS:
        a, b = g[o:o + n], ref_g[o:o + n]
        err = np.linalg.norm(a - b) / np.linalg.norm(b)
        assert err <= 1e-2, (name, err)
    # a row of the batch that is left out, or taken twice, shows: the loss
    # and the gradients of a permuted batch differ by roundings only
    order = rng.permutation(batch)
    loss2, g2 = mc.mlp_grad(f[order], y[order], p)
    assert loss2 == pytest.approx(loss, rel=1e-12)
    assert np.linalg.norm(g2 - g) <= 1e-5 * np.linalg.norm(g)
