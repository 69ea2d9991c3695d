"""Neighbour histograms between few and all partners in range: the two-stage
kernels bin a turn of near partners at once where most lanes have one, and
gather them in a ring otherwise.  Ranges at which tiles of both kinds
occur, one diameter and two, both precisions.  Band 0, so that each group's
first movers have no pending partner in range and their histograms count.
Counts exactly, dE to the bounds of the other two-stage tests.
"""
import numpy as np
import pytest

from test_gpu_da import TOL32, _check_da, _params, _sys

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,precision,two_to_one,frac,da_on", [
    (1500, "fp32", False, 0.35, False), (1500, "fp32", False, 0.8, True), (1500, "fp32", True, 0.8, False),
    (1920, "fp32", True, 1.2, True), (1101, "fp64", True, 0.6, False), (1500, "fp64", False, 1.0, True)])
def test_tiles_of_few_and_many_near_partners(oracle, n, precision, two_to_one, frac, da_on):
    if two_to_one:
        from paper_1602_05716_amd import inputs
        sy = inputs.electrolyte(n // 3, n - n // 3, 2.0, -1.0, 1.0, 0.8, 0.05, 0.7)
        sy.xyz = inputs.random_start(sy, 80 + n)
    else:
        sy = _sys(n, 0.05, 0.7, seed=80 + n)
    st, r, lg = _check_da(oracle, sy, precision, 2, 0x43, 1.5, _params(9, 0.05), da_on=da_on,
                          tol_de=TOL32 if precision == "fp32" else None, rc=frac * sy.R, band=0)
    free = ((lg["flags"] >> 2) & 1) == 0
    near = lg["feats"][free][:, :128].astype(int).sum(axis=1)
    assert free.sum() >= 2 * (n // 64) and 0 < near.min() and near.max() < n
