"""Pair counts at the limits of the cell-grid kernel's LDS histogram: the
largest histogram a handle accepts (48 KiB, beside the kernel's own staging),
and a chain so large that a block adds its 32-bit counters to the chain's more
than once (from 1.4 million ions on).  Integers, so equal.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_largest_histogram(oracle, precision):
    from paper_1602_05716_amd import inputs, mc
    sy = inputs.electrolyte(1200, 1200, 1.0, -1.0, 1.0, 1.0, 0.05, 0.7)
    sy.xyz = inputs.random_start(sy, 91)
    rmax, bins = 0.4 * sy.R, 3072  # 2 x 2 x 3072 x 4 bytes
    print("[gpu-case] 48 KiB histogram", precision, flush=True)
    with mc.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, precision=precision, max_disp=1.0, resum_every=0,
                  rdf_rmax=rmax, rdf_bins=bins) as ch:
        ch.sweep(1, 9)
        ch.rdf_sample()
        r, x = ch.rdf(), ch.positions()
    types, keys = sy.types()
    counts, centres = oracle.rdf_counts(x, types, len(keys), sy.R, rmax, bins)
    assert np.array_equal(r["counts"], np.asarray(counts).reshape(r["counts"].shape))
    assert np.array_equal(r["centres"], np.asarray(centres))


def test_counts_of_a_block_in_several_pieces():
    from scipy.spatial import cKDTree
    from paper_1602_05716_amd import mc
    n, space = 1600000, 2.0
    assert (n + 63) // 64 // 512 > 2 ** 32 // (64 * n)  # items of a block, and between two flushes
    rng = np.random.default_rng(92)
    m = int(np.ceil(n ** (1.0 / 3.0)))
    g = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3)[:n]
    x = (space * (g - 0.5 * (m - 1)) + rng.uniform(-0.4, 0.4, (n, 3))).astype(np.float32).astype(np.float64)
    q = np.where(rng.permutation(n) < n // 2, 1.0, -1.0)
    R, rmax = float(np.sqrt((x * x).sum(1).max())) + 1.0, 2.4
    print("[gpu-case] g(r) of %d ions" % n, flush=True)
    with mc.Chain(x, q, np.ones(n), R, 0.7, precision="fp32", max_disp=0.5, resum_every=0, rdf_rmax=rmax,
                  rdf_bins=2) as ch:
        ch.rdf_sample()
        r = ch.rdf()
        assert np.array_equal(ch.positions(), x)
    print("[gpu-case] counted, reference next", flush=True)
    inside = np.sqrt((x * x).sum(1)) <= R - rmax
    trees = [cKDTree(x[q == s]) for s in (1.0, -1.0)]  # species by decreasing charge
    for a, s in enumerate((1.0, -1.0)):
        centres = cKDTree(x[(q == s) & inside])
        assert r["centres"][a] == centres.n
        for b in range(2):
            upto = centres.count_neighbors(trees[b], [0.5 * rmax, rmax])
            assert r["counts"][a, b].tolist() == [upto[0] - (centres.n if a == b else 0), upto[1] - upto[0]]
