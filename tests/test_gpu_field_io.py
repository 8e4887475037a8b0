"""GPU: state, right-hand side and gradients in the caller's element order,
through host and through device arrays, on meshes whose last tile is partial
(5 x 5 and 7 x 7 elements, rotated frames, so that the internal order is not
the caller's): the same values bit for bit, whichever way they come out."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1804_02221_amd.inputs import smooth_sweep


@pytest.fixture(scope="module")
def esdg():
    from paper_1804_02221_amd import esdg as m
    m.lib()
    return m


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("N", range(2, 9))
def test_host_and_device_arrays_agree(esdg, N, precision):
    import torch
    n = 5 if N % 2 else 7
    w = smooth_sweep(n, N, seed=3, rotate_seed=2)
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    got = []
    for via_device in (False, True):
        put = dev if via_device else (lambda a: a)
        back = (lambda o: [v.cpu().numpy() for v in o]) if via_device else list
        s = esdg.Solver(0, precision)
        s.upload_mesh(w.mesh)
        s.set_params(esdg.default_params(N, **w.params))
        s.set_bathymetry(put(w.b))
        s.set_state(*(put(v) for v in (w.h, w.hu, w.hv)))
        out = [back(s.get_state(device=via_device)), back(s.rhs(device=via_device)), [s.diagnostics()]]
        if precision == 64:
            s.set_params(esdg.default_params(N, **{**w.params, "av_on": 0}))
            out.append(back(s.rhs_vjp(*(put(v) for v in (w.hu, w.h, w.hv)))))
        t, _ = s.step(2)
        out.append(back(s.get_state(device=via_device)))
        s.set_state(*(put(v) for v in (w.h, w.hu, w.hv)))   # the time starts over
        assert t > 0 and s.get_time() == 0.0
        got.append(out)
        s.close()
    kept = np.float64 if precision == 64 else np.float32
    for v, g in zip((w.h, w.hu, w.hv), got[0][0]):
        assert np.array_equal(v.astype(kept).astype(np.float64), g)
    for a, b in zip(*got):
        for x, y in zip(a, b):
            assert np.array_equal(x, y)


def test_instances_of_an_ensemble_in_their_own_order(esdg):
    ws = [smooth_sweep(n, N, seed=n, rotate_seed=n) for n, N in ((3, 3), (6, 5), (4, 3), (5, 3))]
    en = esdg.Ensemble(0)
    for w in ws:
        en.add_workload(w)
    en.build()
    for k, w in enumerate(ws):
        for v, g in zip((w.h, w.hu, w.hv), en.get_state(k)):
            assert np.array_equal(v, g)
    en.close()
