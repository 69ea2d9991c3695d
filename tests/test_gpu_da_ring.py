"""Neighbour histograms when every partner is in range: the two-stage
kernels note near partners in a ring of 128 entries, binned 64 at a time, and
here each partner fills it.  Band 0, so that each group's first mover has no
pending partner and its histograms count; sizes with and without slices taken
four groups at a time, and with a padded last group.  Counts exactly, dE to
the bounds of the other two-stage tests.
"""
import numpy as np
import pytest

from test_gpu_da import TOL32, _check_da, _sys

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,precision", [(130, "fp32"), (1500, "fp32"), (1500, "fp64"), (1920, "fp32")])
def test_every_partner_in_range(oracle, n, precision):
    sy = _sys(n, 0.05, 0.7, seed=70 + n)
    st, r, lg = _check_da(oracle, sy, precision, 2, 0x41, 1.5, np.zeros(oracle.da_nparam()), da_on=False,
                          tol_de=TOL32 if precision == "fp32" else None, rc=2.0 * sy.R + 1.0, band=0)
    free = ((lg["flags"] >> 2) & 1) == 0
    assert free.sum() >= 2 * ((n + 63) // 64)
    # every partner is counted once at the old position
    assert np.all(lg["feats"][free][:, :128].astype(int).sum(axis=1) == n - 1)
