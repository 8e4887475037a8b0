"""GPU: many contexts alive at once, created, stepped and closed by several
threads in their own order: each reads its own status (time, limited and
viscous counts, diagnostics, the step check's decisions), as a context alone
does, and blocks that closed contexts gave back serve new ones."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_1804_02221_amd.inputs import dam_break, smooth_sweep

KW = dict(av_on=1, limiter_on=1, eps0=0.05, integrator=1, max_dt_retries=3)


def report(esdg, w):
    s = esdg.solver_for(w, **KW)
    out = [s.step(1, raise_negmean=False)[0], s.step(2, raise_negmean=False)[0], s.step_stats(), s.diagnostics()]
    return s, out


def same(a, b):
    return a[:3] == b[:3] and np.array_equal(a[3], b[3])


def test_many_contexts_and_threads():
    from paper_1804_02221_amd import esdg
    ws = [dam_break(3 + k, 3, seed=k, rotate_seed=k) if k % 2 else smooth_sweep(3 + k, 2, seed=k) for k in range(6)]
    want = []
    for w in ws:
        s, out = report(esdg, w)
        want.append(out)
        s.close()
    assert len({o[1] for o in want}) == len(want)
    failures = []

    def work(me):
        try:
            rng = np.random.default_rng(me)
            live = []
            for k in rng.permutation(24):
                s, out = report(esdg, ws[k % 6])
                live.append(s)
                if not same(out, want[k % 6]):
                    failures.append((me, int(k)))
                if len(live) > 18:
                    live.pop(int(rng.integers(len(live)))).close()
            for s in live:
                s.close()
        except Exception as e:   # noqa: BLE001
            failures.append((me, repr(e)))

    for _ in range(2):
        threads = [threading.Thread(target=work, args=(me,)) for me in range(4)]   # up to 72 contexts at once
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not failures, failures
