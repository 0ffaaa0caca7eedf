"""What a block step starts from, step by step against the oracle: the due
particles (those whose next time is the earliest) and the forces stored for
them.  One cluster around the compaction's blocks of 1024 particles, mixed
steps routed to FP64 and mixed steps that read the j records built with the
list; and a cluster beyond 2^20 particles, whose list, plan and re-evaluation
list come from launches of their own.  The energy's sums over several
workgroups of a cluster."""
import numpy as np
import pytest

import oracle
from paper_0909_0879_amd import binding, ics
from tests.gpu_util import FP64_TOL, check_parity, is_mixed, require_gpu, to_np

pytestmark = pytest.mark.gpu

TICK = 2.0 ** -20


def _state(g):
    return {k: to_np(t) for k, t in g.get_state().items()}


def _one_step(g, m, eps, t_end, sample, label):
    """One block step: its due particles, their forces; returns their number
    and the parity found."""
    s0 = _state(g)
    before = g.stats()
    ns, ni = g.step_blocks(t_end, 1)
    s1 = _state(g)
    due = s0["tick"] + (np.int64(1) << (20 - s0["level"].astype(np.int64)))
    now = due.min()
    act = np.nonzero(due == now)[0]
    n = m.shape[0]
    assert ns == 1 and ni == act.size * n
    assert np.array_equal(np.nonzero(s1["tick"] != s0["tick"])[0], act)
    assert np.all(s1["tick"][act] == now) and g.stats()["t_tick"] == now
    xp, vp = oracle.predict(s0["x"], s0["v"], s0["a"], s0["j"], (now - s0["tick"]) * TICK)
    idx = act if act.size <= sample else \
        np.sort(np.random.default_rng(int(now)).choice(act, sample, False))
    a_ref, j_ref = oracle.forces(xp, vp, m, eps, idx=idx.astype(np.int64))
    st = check_parity(s1["a"][idx], s1["j"][idx], a_ref, j_ref, is_mixed(g.precision),
                      f"{label}: {act.size} of {n} due")
    small = g.stats()["small_step_interactions"] - before["small_step_interactions"]
    return act.size, small == ni, st


@pytest.mark.parametrize("prec,small_log2", [(binding.FP64, 0), (binding.MIXED, 0),
                                              (binding.MIXED_DS, 0), (binding.MIXED, -1),
                                              (binding.MIXED_DS, -1)])
@pytest.mark.parametrize("n", [1023, 1024, 1025, 2049])
def test_due_particles_around_compaction_blocks(prec, small_log2, n):
    require_gpu()
    m, x, v = ics.plummer(n, 93)
    g = binding.NBody(m, x, v, eps=1e-2, precision=prec, eta=0.02, eta_start=0.02, level_min=3,
                      level_max=8, tuning={"small_log2": small_log2} if small_log2 else None)
    sizes = []
    for k in range(12):
        na, small, st = _one_step(g, m, 1e-2, 1 / 8, n, f"step {k}")
        sizes.append(na)
        if is_mixed(prec) and small_log2 == 0:       # evaluated by the FP64 kernel
            assert small and st["acc_max"] <= FP64_TOL and st["jerk_max"] <= FP64_TOL
        elif is_mixed(prec):
            assert not small
    print(f"n {n}: due {sizes}", flush=True)
    assert max(sizes) > 256 and min(sizes) < n
    g.close()


@pytest.mark.parametrize("prec,small_log2", [(binding.FP64, 0), (binding.MIXED, 0),
                                              (binding.MIXED, -1)])
def test_block_steps_beyond_2_20(prec, small_log2):
    require_gpu()
    n = (1 << 20) + 1025
    m, x, v = ics.plummer(n, 94)
    print(f"beyond 2^20: prec {prec} small_log2 {small_log2}", flush=True)
    g = binding.NBody(m, x, v, eps=1e-3, precision=prec, eta=0.01, eta_start=0.01, level_min=10,
                      level_max=14, tuning={"small_log2": small_log2} if small_log2 else None)
    sizes = [_one_step(g, m, 1e-3, 2.0 ** -10, 128, f"step {k}")[0] for k in range(5)]
    refined = g.stats()["refined"]
    g.step(2.0 ** -10)                  # captured steps, the last of all n
    s = _state(g)
    assert np.all(s["tick"] == 1 << 10)
    if prec == binding.MIXED and small_log2 < 0:
        assert g.stats()["refined"] > refined
    print(f"due {sizes}", flush=True)
    assert min(sizes) < n // 16
    g.close()


@pytest.mark.parametrize("sizes", [[300, 2049, 1], [1025], [70000]])
@pytest.mark.parametrize("field", [False, True])
def test_energy_sums_of_several_workgroups(sizes, field):
    # more than 512 particles in the mean cluster: n / (256 C) workgroups each
    require_gpu()
    m, x, v, off = ics.ensemble(len(sizes), sizes=sizes, seed=95)
    f = binding.allen_santillan(length_unit_kpc=1e-3, mass_unit_msun=1e5) if field else None
    if field:
        x = x + np.array([8500.0, 0.0, 0.0])
    g = binding.NBody(m, x, v, eps=1e-3, precision=binding.FP64, cluster_offsets=off, field=f,
                      level_min=5, level_max=20)
    e = g.energy()
    for c in range(len(sizes)):
        sl = slice(off[c], off[c + 1])
        r = oracle.energy(x[sl], v[sl], m[sl], 1e-3, field=f)
        want = np.concatenate([[r["K"], r["W"], r["E"]], r["L"], r["P"]])
        # a few roundings of the largest of the terms that are summed
        scale = max(1.0, np.abs(want).max())
        assert np.abs(e[c] - want).max() <= 1e-13 * scale, c
    g.close()
