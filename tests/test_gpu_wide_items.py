"""Edges of the work-item shapes, of the one-launch step head and of the paths
that the host chooses for nbody_forces / nbody_accel: wide items of 256 i-slots
and of 64 whose waves share j (short and long chunks, a last chunk of one
record), active counts around a wave and a tile, compaction blocks around 1024
particles, states replaced in clusters that cross a block's pieces, and the
energy's split sums.  Against the oracle at the parity bars of the other GPU
tests."""
import numpy as np
import pytest

import oracle
from paper_0909_0879_amd import binding, ics
from tests.gpu_util import check_parity, is_mixed, require_gpu, to_np

pytestmark = pytest.mark.gpu

PRECS = [binding.FP64, binding.MIXED, binding.MIXED_DS]


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("variant", [binding.VARIANT_K1, binding.VARIANT_S1, binding.VARIANT_S2])
@pytest.mark.parametrize("n,split,target", [
    (1025, 256, 1 << 20),     # too few items for the chip: waves share j, 256-record chunks
    (4097, 256, 1 << 20),     # 256 slots an item; the last chunk holds one record
    (4097, 1024, 1 << 20),    # waves share j in 1024-record chunks, last one a single record
    (2300, 64, 1),            # one chunk of the whole range
])
def test_wide_item_shapes(prec, variant, n, split, target):
    require_gpu()
    m, x, v = ics.plummer(n, 71)
    m = ics.salpeter_masses(n, 72)
    g = binding.NBody(m, x, v, eps=1e-3, precision=prec)
    g.set_tuning({"variant": variant, "acc_variant": variant, "i_slots": [256] * 25,
                  "target_items": [target] * 25, "min_split_j": split})
    rng = np.random.default_rng(73)
    a_ref, j_ref = oracle.forces(x, v, m, 1e-3)
    for na in (n, 257, 65, 64, 1):
        idx = np.sort(rng.choice(n, na, replace=False)).astype(np.int32)
        acc, jerk = g.forces(x, v, m, i_active=idx)
        only = g.accel(x, m, i_active=idx)
        g.sync()
        check_parity(to_np(acc), to_np(jerk), a_ref[idx], j_ref[idx], is_mixed(prec),
                     f"n {n} na {na} variant {variant}")
        check_parity(to_np(only), to_np(jerk), a_ref[idx], j_ref[idx], is_mixed(prec), "accel")
    g.close()


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("n", [1, 2, 1023, 1024, 1025, 2049])
def test_step_head_around_compaction_blocks(prec, n):
    # block steps (FP64 arithmetic in every precision: small steps) whose
    # levels and times are the oracle's; a replaced state and symplectic steps
    # rebuild the level table that the head reads
    require_gpu()
    m, x, v = ics.plummer(n, 74)
    kw = dict(eta=0.02, eta_start=0.01, level_min=5, level_max=20)
    g = binding.NBody(m, x, v, eps=1e-2, precision=prec, **kw)
    ref = oracle.System(m, x, v, 1e-2, **kw)
    if not is_mixed(prec):
        g.step(1 / 32)
        ref.run(1 / 32)
        st = {k: to_np(t) for k, t in g.get_state().items()}
        assert np.array_equal(st["level"], ref.level) and np.array_equal(st["tick"], ref.tick)
        assert np.abs(st["x"] - ref.x).max() < 1e-11
    else:
        g.step(1 / 32)
    mid = g.get_state()
    g.step(1 / 16)
    once = {k: to_np(t) for k, t in g.get_state().items()}
    g.set_state(mid)
    g.step(1 / 16)
    again = {k: to_np(t) for k, t in g.get_state().items()}
    for k in once:
        assert np.array_equal(once[k], again[k]), k
    g.step_symplectic(binding.LEAPFROG, 2.0 ** -8, 8)
    g.step(1 / 8)
    end = g.get_state()
    assert np.all(to_np(end["tick"]) == 1 << 17)
    g.close()


@pytest.mark.parametrize("sizes", [[300, 5, 700, 1, 256, 1024, 37], [1], [2, 511, 513]])
def test_replaced_state_and_energy_of_uneven_clusters(sizes):
    require_gpu()
    m, x, v, off = ics.ensemble(len(sizes), sizes=sizes, seed=75)
    eps = np.linspace(1e-3, 2e-3, len(sizes))
    kw = dict(precision=binding.FP64, eta=0.02, eta_start=0.01, level_min=5, level_max=20)
    g = binding.NBody(m, x, v, eps=eps, cluster_offsets=off, **kw)
    g.step(1 / 32)
    mid = g.get_state()
    ns, ni = g.step(1 / 16)
    once = {k: to_np(t) for k, t in g.get_state().items()}
    g.set_state(mid)
    assert g.step(1 / 16) == (ns, ni)
    for k, t in g.get_state().items():
        assert np.array_equal(once[k], to_np(t)), k
    e = g.energy()
    for c in range(len(sizes)):
        sl = slice(off[c], off[c + 1])
        r = oracle.energy(once["x"][sl], once["v"][sl], m[sl], eps[c])
        want = np.concatenate([[r["K"], r["W"], r["E"]], r["L"], r["P"]])
        # a few roundings of sums of terms below 1
        assert np.allclose(e[c], want, rtol=1e-13, atol=1e-13), c
    g.close()


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("n,na", [(2000, 2000), (2100, 2100), (2100, 131), (5000, 256),
                                  (5000, 312), (5000, 313)])
def test_routes_agree_with_the_oracle(prec, n, na):
    # tile fill, records in LDS and broadcast records, each side of the rules
    # that choose between them (2^22 pairs, one entry in 16, one wide item)
    require_gpu()
    m, x, v = ics.plummer(n, 76)
    idx = np.sort(np.random.default_rng(77).choice(n, na, replace=False)).astype(np.int32)
    a_ref, j_ref = oracle.forces(x, v, m, 1e-3, idx=idx.astype(np.int64))
    for slots in (64, 256):
        g = binding.NBody(m, x, v, eps=1e-3, precision=prec)
        g.set_tuning({"variant": binding.VARIANT_S1, "i_slots": [slots] * 25})
        acc, jerk = g.forces(x, v, m, i_active=idx)
        g.sync()
        check_parity(to_np(acc), to_np(jerk), a_ref, j_ref, is_mixed(prec), f"slots {slots}")
        g.close()
