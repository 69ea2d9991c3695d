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


def _system(n, seed):
    from paper_1602_05716_amd import inputs
    if n % 3 == 0:
        sy = inputs.electrolyte(n // 3, n - n // 3, 2.0, -1.0, 1.0, 0.8, 0.05, 0.7)
    else:
        sy = inputs.electrolyte(n // 2, n - n // 2, 1.0, -1.0, 1.0, 1.0, 0.05, 0.7)
    sy.q = sy.q.copy()
    sy.q[-1] -= sy.q.sum()
    sy.xyz = inputs.random_start(sy, seed)
    return sy


# batches below 512 groups, on cell grids or over all pairs, and above (a full
# device), where each holds chains of both kinds
@pytest.mark.parametrize("sizes,rmax,precision", [((3999, 4000, 2000, 66, 4101), 3.3, "fp32"), ((4000, 1000), 2.0, "fp64"),
                                                  ((3998, 130, 2050), 0.8, "fp32"), ((8001,), 0.8, "fp64"),
                                                  ((130, 2500, 6400) + (6000,) * 5, 2.0, "fp32"),
                                                  ((2000, 3002, 130) + (6000,) * 5, 7.0, "fp32")])
def test_chains_of_a_batch_by_their_own_size(oracle, sizes, rmax, precision):
    """Chains go over a cell grid or over all pairs by their size, the range
    and the handle's groups, in the same sample."""
    from paper_1602_05716_amd import mc
    made = {n: _system(n, 600 + n) for n in set(sizes)}
    print("[gpu-case] g(r) of a batch", sizes, rmax, precision, flush=True)
    with mc.Batch([made[n] for n in sizes], precision=precision, max_disp=[0.5] * len(sizes), resum_every=0,
                  rdf_rmax=rmax, rdf_bins=70, rdf_every=1) as b:
        b.sweep(1, 4)
        first = [b.positions(k) for k in range(len(sizes))]
        b.sweep(1, 4)
        for k, n in enumerate(sizes[:5]):
            sy = made[n]
            types, keys = sy.types()
            r = b.rdf(k)
            two = [oracle.rdf_counts(x, types, len(keys), sy.R, rmax, 70) for x in (first[k], b.positions(k))]
            assert np.array_equal(r["counts"], sum(np.asarray(c) for c, _ in two).reshape(r["counts"].shape))
            assert np.array_equal(r["centres"], sum(np.asarray(c) for _, c in two))
