"""GPU: the ensemble time-step pass beyond one chunk per counter and per
workgroup.  Chunks hold at least eight elements: an instance of 400 elements
has more chunks than there are first-level ticket counters (32), 17309 elements
make more chunks than there are workgroups (2048), so that some take two, of
different instances.  Unequal instances of one degree, with viscosity whose
bound sets the step of some and the mean-positivity bound that of others, with
and without the step check: each equals its own solve bit for bit, time included."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1804_02221_amd.inputs import dam_break, smooth_sweep


def instances(N, sizes):
    """Dam breaks at rest, whose first step the check redoes, smooth flows, and
    the same with rough heights, which the viscosity acts on everywhere."""
    ws = []
    for k, n in enumerate(sizes):
        w = (dam_break, smooth_sweep, smooth_sweep)[k % 3](n, N, seed=40 + k, rotate_seed=k)
        if k % 3 == 2:
            w.h = w.h + 0.2 * np.random.default_rng(k).uniform(-1.0, 1.0, w.h.shape)
        ws.append(w)
    return ws


@pytest.mark.parametrize("retries", [0, 3])
@pytest.mark.parametrize("N,sizes", [(3, (18, 6, 20, 3)), (2, (30, 5, 128)), (5, (17, 4, 6))])
def test_many_chunks_equal_single_solves(N, sizes, retries):
    from paper_1804_02221_amd import esdg
    ws = instances(N, sizes)
    kw = dict(av_on=1, limiter_on=1, eps0=2.0, sigma_min=-4.0, sigma_max=-3.0, integrator=1, max_dt_retries=retries)
    ens = esdg.Ensemble(0, 64)
    ids = [ens.add_workload(w, **kw) for w in ws]
    ens.step(4, raise_negmean=False)
    viscous = mean = 0
    for w, i in zip(ws, ids):
        s = esdg.solver_for(w, **kw)
        for _ in range(4):
            bounds = s.compute_dt()
            viscous += bounds[0] == bounds[2]
            mean += bounds[0] == bounds[3]
            t, _ = s.step(1, raise_negmean=False)
        assert ens.get_time(i) == t, (i, w.mesh.K)
        for a, b in zip(ens.get_state(i), s.get_state()):
            assert np.array_equal(a, b), (i, w.mesh.K)
        s.close()
    ens.close()
    assert viscous and mean
