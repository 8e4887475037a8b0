"""GPU: the diagnostics' reduction over partial rows, at N = 7 one row per
element: 484 (one workgroup), 529 (two and a second launch) and 131769 rows
(256 workgroups of more than 512 rows)."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1804_02221_amd.inputs import smooth_sweep


@pytest.mark.parametrize("n", [22, 23, 363])
def test_totals_against_exact_sums(n):
    """Volume, momentum and extreme heights against exactly rounded sums of
    the same terms.  A term is two products of a Jacobian of a few operations
    (8 ulp), and a sum of 8.4 million terms through 64 x 8 x 16 x 256 levels of
    adds loses at most some 60 ulp of the sum of magnitudes: 1e-14 of it."""
    from paper_1804_02221_amd import esdg
    w = smooth_sweep(n, 7, seed=3)
    s = esdg.solver_for(w, av_on=0)
    d = s.diagnostics()
    J = s.get_geometry()["J"]
    s.close()
    wt = oracle.operators(7)["w"]
    wq = J * np.outer(wt, wt).reshape(-1)
    for k, f in enumerate((w.h, w.hu, w.hv)):
        t = (wq * f).reshape(-1)
        assert abs(d[k] - math.fsum(t)) <= 1e-14 * math.fsum(np.abs(t)), k
    assert d[5] == w.h.min() and d[6] == w.h.max() and d[7] == 0
