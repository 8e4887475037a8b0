"""GPU: the forward sweep takes the memory of its checkpoints, the stage inputs
of a segment that of the reverse sweep: a loss alone needs none of it, whatever
the checkpoint distance.  Once a reverse sweep has taken it, a forward sweep
whose segments fit leaves its last segment's stage inputs there; gradients are
the same bits with and without them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1804_02221_amd.inputs import bathymetry_gradient

DT = 1e-4


def make(integrator=0):
    from paper_1804_02221_amd import esdg
    w, x = bathymetry_gradient(n=16, N=4, n_gauges=5)
    s = esdg.solver_for(w, integrator=integrator)
    s.set_gauges(x["gelem"], x["gxi"], x["geta"])
    return w, s


def test_loss_takes_no_stage_memory():
    import torch
    steps = 1000
    w, s = make()
    target = np.full((steps, 5), 1.01)
    s.adjoint_forward(steps, DT, 500, target)   # the cotangents, two checkpoints
    s.set_state(w.h, w.hu, w.hv)
    free = torch.cuda.mem_get_info()[0]
    s.adjoint_forward(steps, DT, steps, target)
    taken = free - torch.cuda.mem_get_info()[0]
    s.close()
    # one segment of 5001 states of 3 x 6400 doubles would be 768 MB
    assert taken < 64 << 20, taken


@pytest.mark.parametrize("integrator", [0, 1])
@pytest.mark.parametrize("every", [6, 3, 20])
def test_gradients_with_and_without_kept_stages(every, integrator):
    """every = 6 fills the memory of the first reverse sweep, 3 uses part of
    it, 20 asks for more than there is."""
    steps = 20
    target = np.full((steps, 5), 1.01)
    w, fresh = make(integrator)
    loss = fresh.adjoint_forward(steps, DT, every, target)
    want = fresh.adjoint_backward()
    fresh.close()
    w, s = make(integrator)
    s.adjoint_forward(steps, DT, 6, target)
    s.adjoint_backward()
    for _ in range(2):
        s.set_state(w.h, w.hu, w.hv)
        assert s.adjoint_forward(steps, DT, every, target) == loss
        for a, b in zip(want, s.adjoint_backward()):
            assert np.array_equal(a, b)
    s.close()
