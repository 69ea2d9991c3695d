"""Pair counts on the cell grid (chains of 2000 ions and more) against the
oracle's plain double loop: integers, so equal.  Sizes around the switch from
the all-pairs kernel, ragged groups, ranges from a small fraction of the wall
radius (the grid's side then capped) to beyond it (no centres), one to three
species, both precisions and position images, and a batch whose chains are of
very different size."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sys(n, seed, kind="1:1", phi=0.05):
    from paper_1602_05716_amd import inputs
    if kind == "2:1":
        sy = inputs.electrolyte(n // 3, n - n // 3, 2.0, -1.0, 1.0, 0.8, phi, 0.9)
    else:
        sy = inputs.electrolyte(n // 2, n - n // 2, 1.0, -1.0, 1.0, 1.0, phi, 0.7)
    sy.q = sy.q.copy()
    sy.q[-1] -= sy.q.sum()
    sy.xyz = inputs.random_start(sy, seed)
    return sy


def _check(oracle, r, x, sy, rmax, margin, bins, samples=1):
    types, keys = sy.types()
    counts, centres = oracle.rdf_counts(x, types, len(keys), sy.R - margin, rmax, bins)
    assert np.array_equal(r["counts"], samples * np.asarray(counts).reshape(r["counts"].shape))
    assert np.array_equal(r["centres"], samples * np.asarray(centres))


@pytest.mark.parametrize("n,kind,frac,margin,bins,precision", [
    (1999, "1:1", 0.3, 0.0, 200, "fp32"), (2000, "1:1", 0.3, 0.0, 200, "fp32"), (2048, "2:1", 0.5, 0.0, 77, "fp64"),
    (2049, "1:1", 0.04, 0.0, 50, "fp32"), (2500, "2:1", 0.95, 0.0, 64, "fp32"), (2500, "1:1", 1.3, 0.0, 64, "fp32"),
    (3333, "2:1", 0.21, 1.5, 333, "fp64"), (5000, "1:1", 0.13, 0.0, 1000, "fp32"),
    (5003, "2:1", 0.4, 0.0, 1, "fp32")])
def test_counts_match_the_plain_loop(oracle, n, kind, frac, margin, bins, precision):
    from paper_1602_05716_amd import mc
    sy = _sys(n, 70 + n, kind)
    rmax = frac * sy.R
    print("[gpu-case] cells n=%d %s rmax=%.2f R bins=%d %s" % (n, kind, frac, bins, precision), flush=True)
    with mc.Chain(sy.xyz, sy.q, sy.sigma, sy.R, sy.lB, precision=precision, max_disp=1.0, resum_every=0,
                  rdf_rmax=rmax, rdf_bins=bins, rdf_margin=margin) as ch:
        for sweeps in (0, 1, 2):
            ch.sweep(sweeps, 9)
            ch.rdf_reset()
            ch.rdf_sample()
            _check(oracle, ch.rdf(), ch.positions(), sy, rmax, margin, bins)
        ch.rdf_sample()  # counts of a second sample add up
        _check(oracle, ch.rdf(), ch.positions(), sy, rmax, margin, bins, samples=2)


def test_batch_of_uneven_chains(oracle):
    from paper_1602_05716_amd import mc
    systems = [_sys(n, 30 + n, kind) for n, kind in ((2, "1:1"), (2111, "1:1"), (130, "2:1"), (900, "1:1"))]
    print("[gpu-case] cells, batch", flush=True)
    with mc.Batch(systems, precision="fp32", resum_every=0, rdf_rmax=3.0, rdf_bins=90) as b:
        b.sweep(1, 3)
        b.rdf_sample()
        for k, sy in enumerate(systems):
            _check(oracle, b.rdf(k), b.positions(k), sy, 3.0, 0.0, 90)
