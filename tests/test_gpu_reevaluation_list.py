"""Mixed block steps of one cluster whose re-evaluation needs more row-sum
waves than the step's own sums: the sum launch's last block writes the
re-evaluation plan while blocks without work may still have to start, and none
of them may take that plan for the step's.  Against the same cluster inside an
ensemble, whose list and plan are made by launches of their own (the two are
bitwise equal by design)."""
import numpy as np
import pytest

from paper_0909_0879_amd import binding, ics
from tests.gpu_util import require_gpu, to_np

pytestmark = pytest.mark.gpu


# all n due: 1025 waves of 8 (16) entries; the flagged ones: one (four) a wave
@pytest.mark.parametrize("prec", [binding.MIXED, binding.MIXED_DS])
@pytest.mark.parametrize("n,ratio,least,most", [(8200, 0.118, 1026, 2047),
                                                (16400, 0.040, 4101, 8191)])
def test_reevaluation_with_more_waves_than_the_step(prec, n, ratio, least, most):
    require_gpu()
    m, x, v, off = ics.ensemble(2, sizes=[n, 64], seed=81)
    steps = 8
    kw = dict(eps=1e-3, precision=prec, dt_shared=1 / 256, level_min=5, level_max=8,
              tuning={"refine_ratio": ratio, "small_log2": -1})
    e = binding.NBody(m, x, v, cluster_offsets=off, **kw)
    before = e.stats()["refined"]
    e.step(steps / 256)
    refined = e.stats()["refined"] - before
    se = {k: to_np(t) for k, t in e.get_state().items()}
    e.close()
    alone = 0
    for c in range(2):
        sl = slice(off[c], off[c + 1])
        g = binding.NBody(m[sl], x[sl], v[sl], **kw)
        before = g.stats()["refined"]
        g.step(steps / 256)
        mine = g.stats()["refined"] - before
        if c == 0:
            print(f"re-evaluated per step: {mine / steps:.0f} of {n}", flush=True)
            assert least * steps <= mine <= most * steps
        alone += mine
        for k, t in g.get_state().items():
            assert np.array_equal(se[k][sl], to_np(t)), (c, k)
        g.close()
    assert alone == refined
