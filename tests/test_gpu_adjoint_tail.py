"""GPU: the last segment's stage inputs that the forward sweep leaves for the
reverse one.  One segment, several and a ragged last one: the same gradient on
a second call (which finds another segment's stage inputs in their place) and
whatever else ran in between, and the state, time and step bounds after the
sweep those of plain steps, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1804_02221_amd.inputs import bathymetry_gradient


@pytest.mark.parametrize("integrator", [0, 1])
@pytest.mark.parametrize("every", [9, 4, 2])
def test_sweeps_and_what_they_leave(every, integrator):
    from paper_1804_02221_amd import esdg
    w, x = bathymetry_gradient(n=6, N=4, n_gauges=5)
    steps, dt = 9, 2e-3
    target = np.full((steps, 5), 1.01)

    def make():
        s = esdg.solver_for(w, integrator=integrator)
        s.set_gauges(x["gelem"], x["gxi"], x["geta"])
        return s

    plain, s = make(), make()
    plain.step(steps, dt)
    loss = s.adjoint_forward(steps, dt, every, target)
    for a, b in zip(plain.get_state(), s.get_state()):
        assert np.array_equal(a, b)
    assert plain.get_time() == s.get_time()
    assert np.array_equal(plain.compute_dt(), s.compute_dt())
    first = s.adjoint_backward()
    again = s.adjoint_backward()
    s.step(2)
    s.rhs()
    later = s.adjoint_backward()
    # recorded with a timing run in between: every segment recomputed
    s.set_state(w.h, w.hu, w.hv)
    s.profile(True)
    assert s.adjoint_forward(steps, dt, every, target) == loss
    s.profile(False)
    recomputed = s.adjoint_backward()
    for a, b, c, d in zip(first, again, later, recomputed):
        assert np.array_equal(a, b) and np.array_equal(a, c) and np.array_equal(a, d)
    plain.close()
    s.close()
