"""The level histogram after a symplectic run, which chooses every level anew:
the next block step ends at the finest step that is present then, not at one
that only the levels before the run needed."""
import numpy as np
import pytest

from paper_0909_0879_amd import binding
from tests.gpu_util import require_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [binding.FP64, binding.MIXED, binding.MIXED_DS])
@pytest.mark.parametrize("clusters", [1, 3])
def test_first_step_after_a_symplectic_run(prec, clusters):
    require_gpu()
    # an eccentric binary (e = 0.6, a = 1, period 2 pi) from its pericentre,
    # where the steps are short, to about its apocentre
    m = np.array([0.5, 0.5])
    x = np.array([[0.2, 0.0, 0.0], [-0.2, 0.0, 0.0]])
    v = np.array([[0.0, 1.0, 0.0], [0.0, -1.0, 0.0]])
    off = None if clusters == 1 else 2 * np.arange(clusters + 1)
    g = binding.NBody(np.tile(m, clusters), np.tile(x, (clusters, 1)), np.tile(v, (clusters, 1)),
                      eps=1e-3, precision=prec, eta=0.01, eta_start=0.01, level_min=3,
                      level_max=20, cluster_offsets=off)
    first = int(to_np(g.get_state()["level"]).max())
    g.step_symplectic(binding.LEAPFROG, 2.0 ** -10, 3200)
    st = {k: to_np(t) for k, t in g.get_state().items()}
    finest = int(st["level"].max())
    print(f"finest level {first} at the pericentre, {finest} at the apocentre", flush=True)
    assert finest < first
    ns, ni = g.step_blocks(4.0, 1)
    assert ns == 1 and ni == 4 * clusters
    after = to_np(g.get_state()["tick"])
    assert np.all(after == st["tick"] + (1 << (20 - finest)))
    # levels counted once each: the state put back takes the same steps
    mid = g.get_state()
    once = g.step(4.0)
    end = {k: to_np(t) for k, t in g.get_state().items()}
    g.set_state(mid)
    assert g.step(4.0) == once
    for k, t in g.get_state().items():
        assert np.array_equal(end[k], to_np(t)), k
    g.close()
