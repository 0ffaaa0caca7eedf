"""A context's tuning goes back in as it came out: every default lies within
the ranges that nbody_set_tuning accepts."""
import pytest

from paper_0909_0879_amd import binding, ics
from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [binding.FP64, binding.MIXED, binding.MIXED_DS])
def test_default_tuning_goes_back_in(prec):
    require_gpu()
    m, x, v = ics.plummer(64, 90)
    g = binding.NBody(m, x, v, precision=prec)
    t = g.get_tuning()
    assert all(1 <= q <= 1 << 20 for q in t["target_items"])
    assert all(1 <= p <= 256 and p & (p - 1) == 0 for p in t["i_slots"])
    g.set_tuning(t)
    assert g.get_tuning() == t
    g.close()
