"""GPU: an ensemble with the step check whose degree groups hold one instance
each (and one with a single instance in all): the group's step flags and retry
mask are those of one instance, and each instance equals its own solve with the
same retries bit for bit, whether its steps are redone or kept."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1804_02221_amd.inputs import dam_break, smooth_sweep

KW = dict(av_on=1, limiter_on=1, eps0=0.05, integrator=1, max_dt_retries=3)


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("lone", [False, True])
def test_lone_degree_equals_single_solve(lone, precision):
    from paper_1804_02221_amd import esdg
    ws = [dam_break(6, 3, seed=4, rotate_seed=3)]   # its first step is redone at half the size
    if not lone:
        ws += [smooth_sweep(3, 5, seed=24), dam_break(4, 7, seed=23, rotate_seed=1)]
    ens = esdg.Ensemble(0, precision)
    ids = [ens.add_workload(w, **KW) for w in ws]
    ens.step(1, raise_negmean=False)
    first = [ens.get_time(i) for i in ids]
    ens.step(3, raise_negmean=False)
    for w, i, t1 in zip(ws, ids, first):
        s = esdg.solver_for(w, precision=precision, **KW)
        bound = s.compute_dt()[0]
        assert s.step(1, raise_negmean=False)[0] == t1
        if i == ids[0] and precision == 64:
            assert t1 == pytest.approx(0.5 * bound, rel=1e-14)
        assert s.step(3, raise_negmean=False)[0] == ens.get_time(i)
        for a, b in zip(ens.get_state(i), s.get_state()):
            assert np.array_equal(a, b)
        s.close()
    ens.close()
