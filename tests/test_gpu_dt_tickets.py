"""GPU: the time-step pass that reduces its own minima.  Meshes whose pass
takes 1, 8, 32, 40 and 144 workgroups: no atomics, one ticket counter, exactly
full, just two levels, two levels with unequal shares; each pass must leave
slots and counters as the next one needs them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1804_02221_amd.inputs import smooth_sweep


@pytest.mark.parametrize("n", [5, 20, 40, 48, 96])
def test_step_from_one_launch(n):
    """Step, CFL and mean-positivity bound against the oracle on the state that
    one step left.  Each is a handful of operations without cancellation on
    this flow (the bound that divides by a jump of velocity is never the
    smallest): some 50 ulp, 1e-14, held to 1e-13."""
    from paper_1804_02221_amd import esdg
    w = smooth_sweep(n, 3, seed=3, rotate_seed=1)
    s = esdg.solver_for(w)
    P = s.get_params()
    t0, _ = s.step(1)
    first, again = s.compute_dt(), s.compute_dt()
    h, hu, hv = s.get_state()
    want = oracle.dt(oracle.params(3, **P.as_dict()), w.mesh, w.b, h, hu, hv)
    t1, _ = s.step(1)
    s.close()
    assert np.array_equal(first, again)
    assert t1 - t0 == pytest.approx(first[0], rel=1e-12)
    for k in (0, 1, 3):
        assert abs(first[k] - want[k]) <= 1e-13 * want[k], k
