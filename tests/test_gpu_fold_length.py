"""How many FP64 terms a lane adds before it folds them into its compensated
pair: one LDS tile's share, 256 / (lanes of a slot), in narrow items.  A term
of 1 followed by terms of 2^-55, each of which vanishes against it (half an ulp
of 1 is 2^-53): those that share its fold are lost, the others are kept, so the
loss counts the terms of one fold."""
import numpy as np
import pytest

from paper_0909_0879_amd import binding
from tests.gpu_util import require_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", [16, 64, 128])
@pytest.mark.parametrize("variant", [binding.VARIANT_K1, binding.VARIANT_K2])
def test_narrow_items_fold_every_tile(slots, variant):
    require_gpu()
    n = 4096
    # j at unit distance along x; the i, massless, all at the origin and last
    x = np.zeros((n + slots, 3))
    x[:n, 0] = 1.0
    v = np.zeros_like(x)
    v[:n, 1] = 1.0                     # jerk: m along y, the same sums again
    alone = np.zeros(n + slots)
    alone[0] = 1.0                     # the first record of its lane
    m = alone.copy()
    m[1:n] = 2.0 ** -55
    idx = np.arange(n, n + slots, dtype=np.int32)
    # eps^2 vanishes against 1; distances and eps leave no pair at zero
    g = binding.NBody(m, x, v, eps=1e-9, precision=binding.FP64)
    g.set_tuning({"variant": variant, "acc_variant": variant, "i_slots": [slots] * 25,
                  "target_items": [1] * 25})
    lanes = 256 // slots
    # the lost terms, and the roundings of the lanes' tree and of both results
    tol = 256 / lanes * 2.0 ** -55 + (np.log2(lanes) + 2) * 2.0 ** -53
    want = (n - 1) * 2.0 ** -55
    (a1, j1), (a0, j0) = (g.forces(x, v, q, i_active=idx) for q in (m, alone))
    g.sync()
    for name, one, none in (("acc", a1, a0), ("jerk", j1, j0),
                            ("accel", g.accel(x, m, i_active=idx), g.accel(x, alone, i_active=idx))):
        col = 1 if name == "jerk" else 0
        got = to_np(one)[:, col] - to_np(none)[:, col]
        off = np.abs(got - want).max()
        print(f"{name}: off by {off * 2.0 ** 55:.0f} terms, at most {tol * 2.0 ** 55:.0f}", flush=True)
        assert off <= tol, name
    g.close()
