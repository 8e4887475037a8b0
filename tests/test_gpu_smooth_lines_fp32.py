"""GPU: the line test that spares smooth elements the modal transform, in single
precision (its own cutoff and rounding), against the oracle's indicator of the
same rounded heights: in the indicator pass and in the stage kernel's
epilogue."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle
from paper_1804_02221_amd.inputs import smooth_sweep
from test_gpu_smooth_lines import heights


@pytest.mark.parametrize("shift", [0.0, -3.0])
@pytest.mark.parametrize("N", range(2, 9))
def test_line_test_keeps_the_indicator_fp32(N, shift):
    """On the ramp (two decades wide) d(eps)/d(sigma) is at most eps0 pi/4 and
    the energy fraction's relative error is twice the mode's: 4 (N+1)^2
    roundings of 2^-24 at the size of the heights (at most twice the mean)
    over the square root of the fraction, at least 10^(sigma_min/2).  From
    4e-5 eps0 (N = 2) to 0.17 eps0 (N = 8, thresholds 1000 times lower)."""
    from paper_1804_02221_amd import esdg
    w = smooth_sweep(13, N, seed=3, rotate_seed=1)
    s0 = -4.0 * np.log10(N) + shift
    h = heights(N, w.mesh.K, 11 * N, s0).astype(np.float32).astype(np.float64)
    z = np.zeros_like(h)
    kw = dict(g=9.81, av_on=1, limiter_on=0, eps0=0.05, sigma_min=s0 - 1.0, sigma_max=s0 + 1.0)
    s = esdg.Solver(0, 32)
    s.upload_mesh(w.mesh)
    s.set_params(esdg.default_params(N, **kw))
    s.set_bathymetry(z)
    s.set_state(h, z, z)
    want = oracle.indicator(oracle.params(N, **kw), N, h)
    swept = s.get_eps()
    s.step(1, 1e-200)   # zero in single precision: the state stays, eps is the stage epilogue's
    assert np.array_equal(s.get_state()[0], h)
    staged = s.get_eps()
    s.close()
    mode = 2.0 * 4.0 * (N + 1) ** 2 * 2.0 ** -24 / 10.0 ** (0.5 * (s0 - 1.0))
    tol = 0.05 * np.pi / 4 * 2.0 * mode / np.log(10.0)
    for got in (swept, staged):
        assert np.abs(got - want).max() <= tol, (np.abs(got - want).max(), tol)
    assert (want == 0).any() and (want > 0).any()
