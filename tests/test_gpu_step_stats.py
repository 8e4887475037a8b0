"""GPU: the number of elements with viscosity (step statistics) is that of
positive entries of the element viscosity: one workgroup and a part of one, a
full and a ragged number of them, more than one pass of each over the mesh;
none, some and all elements; every call leaves the counter as the next needs
it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1804_02221_amd.inputs import smooth_sweep


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [2, 16, 39, 257, 300])
def test_viscous_elements_counted(n, precision):
    from paper_1804_02221_amd import esdg
    w = smooth_sweep(n, 2, seed=5)
    rng = np.random.default_rng(n)
    K = w.mesh.K
    s = esdg.solver_for(w, precision=precision, av_on=1, eps0=0.05, sigma_min=-4.0, sigma_max=-3.0)
    for share in (0.0, 0.3, 1.0, 0.0):
        h = np.ones_like(w.h)
        rough = rng.random(K) < share
        h[rough] += 0.3 * rng.choice([-1.0, 1.0], size=h[rough].shape)
        s.set_state(h, 0.1 * h, 0.0 * h)
        want = int((s.get_eps() > 0).sum())
        assert (want > 0) == rough.any() and (share < 1.0 or want > 0.9 * K)
        for _ in range(2):
            assert s.step_stats()[1] == want
    s.close()
