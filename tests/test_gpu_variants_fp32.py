"""GPU: the compiled variants of the single-precision stage kernel give the same
bits at every degree (right-hand side, two adaptive steps with viscosity and
limiter, time), on a smooth state with rough velocities and on a wet/dry one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1804_02221_amd.inputs import dam_break, smooth_sweep


@pytest.mark.parametrize("N", range(2, 9))
@pytest.mark.parametrize("kind", ["smooth", "wetdry"])
def test_variants_bitwise_equal_fp32(kind, N):
    from paper_1804_02221_amd import esdg
    if kind == "smooth":
        w = smooth_sweep(5, N, seed=60 + N, rotate_seed=N)
        w.hu = w.hu + 0.05 * np.random.default_rng(N).standard_normal(w.hu.shape)
        kw = dict(av_on=1, limiter_on=1, eps0=0.05, sigma_min=-12.0, sigma_max=-1.0)
    else:
        w = dam_break(6, N, seed=N, rotate_seed=N)
        kw = dict(av_on=1, limiter_on=1, eps0=0.05)
    out = []
    for v in range(esdg.STAGE_VARIANTS):
        s = esdg.solver_for(w, precision=32, **kw)
        s.set_stage_variant(v)
        r = s.rhs()
        s.step(2, 0.0, raise_negmean=False)
        out.append([*r, *s.get_state(), s.get_eps(), np.array(s.get_time())])
        s.close()
    assert (out[0][6] > 0).any()
    for o in out[1:]:
        for a, b in zip(out[0], o):
            assert np.array_equal(a, b)
