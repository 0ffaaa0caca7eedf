"""Workloads of the N-body library for timing, through its public entry points.

`listed()` holds the named workloads, `draw(rng)` gives another one of the same
ranges, `prepare(case, seed)` makes what a program holds before the call,
`run(state)` is one pass, `work(case)` what that pass cannot do without, and
`exact(case, seed)` the same results from plain FP64 torch.

The sizes are those of bench.py and the tests: Plummer, King and Salpeter
systems from 1024 to 2^20 particles and ensembles of clusters of 256 to 16384.
"""
import math

import numpy as np
import torch

from paper_0909_0879_amd import binding, ics

PRECISIONS = {"fp64": binding.FP64, "mixed": binding.MIXED, "mixed_ds": binding.MIXED_DS}
SCHEMES = {"leapfrog": binding.LEAPFROG, "sixth": binding.SYMPLECTIC6}
ETA = 0.01
TICKS = 1 << 20
# Force evaluations per particle and unit of time of a block-step run at
# eta = 0.01 (2.9e11 interactions to t = 1/8 at 65536, 3.3e12 to t = 1/16 at
# 262144): sets work() of those cases only.
EVALS_PER_TIME = 550.0


def listed():
    return [
        # one evaluation of a small cluster by a caller that may not allocate
        # (captured code, tight loops): latency
        dict(name="noalloc-fp64-1024", entry="noalloc", model="plummer", n=1024, active=1024,
             precision="fp64", eps=1e-3),
        # a few due particles of a large system: the split-j regime
        dict(name="forces-fp64-16-of-262144", entry="forces", model="king", n=262144, active=16,
             precision="fp64", eps=1e-4),
        # an ordinary active set, of no round size
        dict(name="forces-mixed-1001-of-262144", entry="forces", model="king", n=262144,
             active=1001, precision="mixed", eps=1e-4),
        # every particle of a middle-sized system
        dict(name="forces-mixed-65536", entry="forces", model="plummer", n=65536, active=65536,
             precision="mixed", eps=1e-3),
        # the double-single form, unequal masses, an odd size
        dict(name="forces-ds-40001", entry="forces", model="salpeter", n=40001, active=40001,
             precision="mixed_ds", eps=1e-4),
        # the paper's drivers: constant steps, acceleration only
        dict(name="leapfrog-mixed-65536", entry="symplectic", model="uniform", n=65536,
             precision="mixed", eps=1e-3, scheme="leapfrog", steps=16),
        dict(name="sixth-fp64-4096", entry="symplectic", model="uniform", n=4096,
             precision="fp64", eps=1e-3, scheme="sixth", steps=16),
        # shared steps of a small cluster: 32 steps of 1/256, then its energy
        dict(name="shared-fp64-1024", entry="shared", model="plummer", n=1024,
             precision="fp64", eps=1e-3),
        # individual time steps over one output interval, then the energy
        dict(name="blocks-fp64-65536", entry="blocks", model="plummer", n=65536,
             precision="fp64", eps=1e-3, level=6),
        dict(name="blocks-mixed-salpeter-262144", entry="blocks", model="salpeter", n=262144,
             precision="mixed", eps=1e-4, level=7),
        # many independent clusters in one context
        dict(name="ensemble-mixed-256", entry="ensemble", model="plummer", clusters=256,
             sizes=5000, precision="mixed", eps=1e-3, level=5),
        # the headline: one block step with all 2^20 particles due
        dict(name="step-mixed-king-1048576", entry="step", model="king", n=1 << 20,
             precision="mixed", eps=1e-4),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    entry = rng.choice(["noalloc", "forces", "forces", "accel", "symplectic", "shared", "blocks",
                        "blocks", "ensemble"])
    case = dict(entry=entry, model=rng.choice(["plummer", "king", "salpeter"]),
                precision=rng.choice(["fp64", "mixed", "mixed_ds"]),
                eps=rng.choice([1e-3, 1e-4]))
    if entry in ("noalloc", "forces", "accel"):
        case["n"] = size(256, 16384 if entry == "noalloc" else 262144)
        case["active"] = case["n"] if rng.random() < 0.5 else size(1, case["n"])
    elif entry == "symplectic":
        case.update(model="uniform", eps=1e-3, n=size(256, 65536),
                    scheme=rng.choice(["leapfrog", "sixth"]), steps=16)
    elif entry == "shared":
        case.update(model="plummer", eps=1e-3, n=size(256, 16384))
    elif entry == "blocks":
        case.update(n=size(1024, 131072), level=7, field=rng.random() < 0.25)
    else:
        case.update(model="plummer", eps=1e-3, clusters=size(4, 256),
                    sizes=rng.randrange(1, 1 << 20), level=5)
    return case


# ------------------------------------------------------------------ inputs

def _king(n, w0, seed):
    """King (1966) model in Henon units, as ics.king, its samples drawn with
    torch (quick at 2^20 particles)."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    g = torch.Generator(device=dev).manual_seed(int(seed))
    prof = ics.king_profile(w0)
    tab = {k: torch.as_tensor(prof[k], device=dev) for k in ("r", "W", "M")}

    def uniform(*shape):
        return torch.rand(*shape, generator=g, device=dev, dtype=torch.float64)

    def interp(u, xs, ys):
        k = torch.searchsorted(xs, u).clamp(1, xs.numel() - 1)
        f = (u - xs[k - 1]) / (xs[k] - xs[k - 1])
        return ys[k - 1] + f * (ys[k] - ys[k - 1])

    def direction(k):
        cz, ph = 2.0 * uniform(k) - 1.0, 2.0 * math.pi * uniform(k)
        sz = (1.0 - cz * cz).clamp(min=0.0).sqrt()
        return torch.stack([sz * ph.cos(), sz * ph.sin(), cz], 1)

    r = interp(uniform(n), tab["M"] / prof["M_t"], tab["r"])
    w = interp(r, tab["r"], tab["W"]).clamp(min=0.0)
    grid = torch.linspace(0.0, 1.0, 65, device=dev, dtype=torch.float64)
    top = torch.zeros(n, device=dev, dtype=torch.float64)
    for u in grid:
        top = torch.maximum(top, u * u * torch.expm1(w * (1.0 - u * u)))
    speed = torch.zeros(n, device=dev, dtype=torch.float64)
    todo = torch.arange(n, device=dev)
    while todo.numel():
        u, y = uniform(todo.numel()), uniform(todo.numel()) * 1.1 * top[todo]
        wt = w[todo]
        ok = y <= u * u * torch.expm1(wt * (1.0 - u * u))
        speed[todo[ok]] = (u * (2.0 * wt).sqrt())[ok]
        todo = todo[~ok]
    lam = -2.0 * prof["pot"] / prof["M_t"] ** 2      # model energy to -1/4
    x = r[:, None] * direction(n) * lam
    v = speed[:, None] * direction(n) / math.sqrt(prof["M_t"] * lam)
    m = torch.full((n,), 1.0 / n, device=dev, dtype=torch.float64)
    return m, x - x.mean(0), v - v.mean(0)


def _system(case, seed):
    """m, x, v (FP64, on the GPU) and, for an ensemble, the cluster offsets."""
    model, off = case["model"], None
    if case["entry"] == "ensemble":
        sizes = ics.ensemble_sizes(case["clusters"], 256, 16384, case["sizes"])
        m, x, v, off = ics.ensemble(sizes=sizes, seed=seed)
    elif model == "king":
        m, x, v = _king(case["n"], 7.0, seed)
    elif model == "salpeter":
        m, x, v = ics.plummer(case["n"], seed, masses=ics.salpeter_masses(case["n"], seed))
    elif model == "uniform":
        m, x, v = ics.uniform_sphere_virial(case["n"], seed)
    else:
        m, x, v = ics.plummer(case["n"], seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    m, x, v = (torch.as_tensor(a, dtype=torch.float64, device=dev) for a in (m, x, v))
    if case.get("field"):
        # on a circular orbit at 8.5 kpc (units of 1e5 M_sun and 1 pc)
        x = x + torch.tensor([8500.0, 0.0, 0.0], dtype=torch.float64, device=dev)
        v = v + torch.tensor([0.0, 10.6, 0.0], dtype=torch.float64, device=dev)
    return m, x, v, off


def _active(case, seed):
    """The due particles' indices, ascending, or None for all of them."""
    if case["active"] == case["n"] and case["entry"] != "noalloc":
        return None
    rng = np.random.default_rng(seed)
    return np.sort(rng.choice(case["n"], case["active"], replace=False)).astype(np.int32)


def _step_args(case):
    """Time-step parameters of a case's context and the time it runs to."""
    if case["entry"] == "shared":
        return dict(dt_shared=1.0 / 256, level_min=3, level_max=8), 1.0 / 8
    if case["entry"] == "step":
        return dict(level_min=10, level_max=10), 2.0 ** -10
    if case["entry"] == "symplectic":
        return dict(level_min=6, level_max=20), case["steps"] * 2.0 ** -10
    return dict(level_min=case.get("level", 3), level_max=20), 2.0 ** -case.get("level", 3)


def prepare(case, seed):
    m, x, v, off = _system(case, seed)
    state = dict(case=case, m=m, x=x, v=v)
    prec = PRECISIONS[case["precision"]]
    if case["entry"] == "noalloc":
        state["ia"] = torch.as_tensor(_active(case, seed), device="cuda")
        state["acc"] = torch.empty((case["active"], 3), dtype=torch.float64, device="cuda")
        state["jerk"] = torch.empty_like(state["acc"])
        return state
    steps, state["t"] = _step_args(case)
    field = (binding.allen_santillan(length_unit_kpc=1e-3, mass_unit_msun=1e5)
             if case.get("field") else None)
    g = binding.NBody(m, x, v, eps=case["eps"], precision=prec, eta=ETA, eta_start=ETA,
                      cluster_offsets=off, field=field, tuning="auto", **steps)
    state["g"] = g
    if case["entry"] in ("forces", "accel"):
        ia = _active(case, seed)
        state["ia"] = None if ia is None else torch.as_tensor(ia, device="cuda")
    else:
        state["checkpoint"] = g.get_state()
    return state


def run(state):
    case, g = state["case"], state.get("g")
    entry = case["entry"]
    if entry == "noalloc":
        binding.nbody_forces_noalloc(PRECISIONS[case["precision"]], case["eps"], state["ia"],
                                     state["x"], state["v"], state["m"], state["acc"],
                                     state["jerk"])
        return state["acc"], state["jerk"]
    if entry == "forces":
        return g.forces(state["x"], state["v"], state["m"], i_active=state["ia"])
    if entry == "accel":
        return g.accel(state["x"], state["m"], i_active=state["ia"])
    # an integration: resume from the checkpoint, run one output interval,
    # diagnose, read the state out
    g.set_state(state["checkpoint"])
    if entry == "symplectic":
        pairs = g.step_symplectic(SCHEMES[case["scheme"]], 2.0 ** -10, case["steps"])
        return dict(g.get_state(), interactions=pairs)
    blocks, pairs = g.step(state["t"])
    out = dict(block_steps=blocks, interactions=pairs)
    if entry != "step":
        out["energy"] = g.energy()
    out.update(g.get_state())
    return out


# ------------------------------------------------------------------ work

def work(case):
    entry = case["entry"]
    if entry in ("noalloc", "forces", "accel"):
        # 41 (20) flops a pair; m, x (and v) read once, indices in, results out
        pair, per_j, per_i = (20, 32, 28) if entry == "accel" else (41, 56, 52)
        return dict(bytes=per_j * case["n"] + per_i * case["active"],
                    flops=pair * case["n"] * case["active"])
    if entry == "ensemble":
        sizes = ics.ensemble_sizes(case["clusters"], 256, 16384, case["sizes"]).astype(float)
    else:
        sizes = np.array([float(case["n"])])
    n, pairs = sizes.sum(), (sizes * sizes).sum()
    flops = 41.0
    if entry == "symplectic":
        evals = 1 + case["steps"] * (7 if case["scheme"] == "sixth" else 1)
        flops = 20.0 + 41.0 / evals
    elif entry == "shared":
        evals = 32
    elif entry == "step":
        evals = 1
    else:
        evals = EVALS_PER_TIME * 2.0 ** -case["level"]
    # the state (x, v, a, jerk, tick, level) in and out, the masses in
    return dict(bytes=n * (2 * 105 + 8), flops=flops * evals * pairs)


# ------------------------------------------------------------------ exact

MOST_PAIRS = 6e10        # about 15 seconds of the sums below


def _pair_sums(xi, vi, xj, vj, mj, eps):
    """Acceleration and jerk on (xi, vi) from the j-particles; a particle's
    own term is zero since eps > 0.  vi None: acceleration only."""
    n, out_a, out_j = mj.numel(), [], []
    chunk = max(1, (1 << 24) // n)
    for b in range(0, xi.shape[0], chunk):
        dx = [xj[None, :, c] - xi[b:b + chunk, None, c] for c in range(3)]
        s = dx[0] * dx[0] + dx[1] * dx[1] + dx[2] * dx[2] + eps * eps
        mr3 = mj / (s * s.sqrt())
        out_a.append(torch.stack([(mr3 * d).sum(1) for d in dx], 1))
        if vi is None:
            continue
        w = [vj[None, :, c] - vi[b:b + chunk, None, c] for c in range(3)]
        al = (dx[0] * w[0] + dx[1] * w[1] + dx[2] * w[2]) * (3.0 / s)
        out_j.append(torch.stack([(mr3 * (w[c] - al * dx[c])).sum(1) for c in range(3)], 1))
    return torch.cat(out_a), (torch.cat(out_j) if out_j else None)


def _energy(m, x, v, eps):
    """K, W, E, L, P of one cluster, as nbody_energy lays them out."""
    n, phi = m.numel(), []
    chunk = max(1, (1 << 24) // n)
    for b in range(0, n, chunk):
        s = sum((x[None, :, c] - x[b:b + chunk, None, c]) ** 2 for c in range(3)) + eps * eps
        t = m / s.sqrt()
        rows = torch.arange(t.shape[0], device=t.device)
        t[rows, rows + b] = 0.0
        phi.append(-t.sum(1))
    k = 0.5 * (m * (v * v).sum(1)).sum()
    w = 0.5 * (m * torch.cat(phi)).sum()
    ang = (m[:, None] * torch.linalg.cross(x, v)).sum(0)
    mom = (m[:, None] * v).sum(0)
    return torch.cat([torch.stack([k, w, k + w]), ang, mom])[None, :].cpu()


def _predict(x, v, a, j, h):
    return (x + h * (v + h * (0.5 * a + h * (j / 6.0))), v + h * (a + h * (0.5 * j)))


def _hermite(m, x, v, eps, t_end, level_min, level_max, dt_shared=0.0):
    """Hermite-4 block steps (or shared steps) to t_end; None when they take
    too many pairs."""
    n = m.numel()
    a, j = _pair_sums(x, v, x, v, m, eps)
    tick = torch.zeros(n, dtype=torch.int64, device=m.device)
    if dt_shared > 0.0:
        level = torch.full_like(tick, round(-math.log2(dt_shared)))
    else:
        dt0 = ETA * a.norm(dim=1) / j.norm(dim=1)
        level = torch.full_like(tick, level_min)
        for k in range(level_min, level_max):
            level += ((level == k) & (2.0 ** -k > dt0)).long()
    end, pairs = round(t_end * TICKS), 0.0
    while True:
        due = tick + (TICKS >> level)
        now = int(due.min())
        if now > end:
            break
        i = torch.nonzero(due == now)[:, 0]
        pairs += float(i.numel()) * n
        if pairs > MOST_PAIRS:
            return None
        h = ((now - tick).double() / TICKS)[:, None]
        xp, vp = _predict(x, v, a, j, h)
        a1, j1 = _pair_sums(xp[i], vp[i], xp, vp, m, eps)
        h, a0, j0 = h[i], a[i], j[i]
        a2 = (-6.0 * (a0 - a1) - h * (4.0 * j0 + 2.0 * j1)) / h ** 2
        a3 = (12.0 * (a0 - a1) + 6.0 * h * (j0 + j1)) / h ** 3
        x[i] = xp[i] + a2 * (h ** 4 / 24.0) + a3 * (h ** 5 / 120.0)
        v[i] = vp[i] + a2 * (h ** 3 / 6.0) + a3 * (h ** 4 / 24.0)
        a[i], j[i], tick[i] = a1, j1, now
        if dt_shared > 0.0:
            continue
        n1, nj, n2, n3 = (q.norm(dim=1) for q in (a1, j1, a2 + h * a3, a3))
        dt = (ETA * (n1 * n2 + nj * nj) / (nj * n3 + n2 * n2)).sqrt()
        lv = level[i]
        step = 2.0 ** -lv.double()
        up = ((dt >= 2.0 * step) & (lv > level_min) & (now % (TICKS >> (lv - 1)) == 0)).long()
        for k in range(level_min, level_max):
            lv = lv + ((lv == k) & (2.0 ** -k > dt)).long()
        level[i] = lv - up
    return dict(x=x, v=v, a=a, j=j, tick=None, level=None)


def exact(case, seed):
    entry = case["entry"]
    if entry in ("ensemble", "step") or case.get("field"):
        return None          # minutes of plain sums
    n = case["n"]
    if entry == "blocks" and EVALS_PER_TIME * 2.0 ** -case["level"] * n * n > MOST_PAIRS:
        return None
    m, x, v, _ = _system(case, seed)
    eps = case["eps"]
    if entry in ("noalloc", "forces", "accel"):
        if float(n) * case["active"] > MOST_PAIRS:
            return None
        ia = _active(case, seed)
        i = torch.arange(n) if ia is None else torch.as_tensor(ia).long()
        i = i.to(m.device)
        a, j = _pair_sums(x[i], None if entry == "accel" else v[i], x, v, m, eps)
        return a if entry == "accel" else (a, j)
    if entry == "symplectic":
        w = [1.0]
        if case["scheme"] == "sixth":
            w1, w2, w3 = -1.17767998417887, 0.235573213359357, 0.784513610477560
            w = [w3, w2, w1, 1.0 - 2.0 * (w1 + w2 + w3), w1, w2, w3]
        if float(n) * n * len(w) * case["steps"] > 2.0 * MOST_PAIRS:
            return None
        a = _pair_sums(x, None, x, v, m, eps)[0]
        for wk in w * case["steps"]:
            c = wk * 2.0 ** -10
            v = v + 0.5 * c * a
            x = x + c * v
            a = _pair_sums(x, None, x, v, m, eps)[0]
            v = v + 0.5 * c * a
        a, j = _pair_sums(x, v, x, v, m, eps)
        return dict(x=x, v=v, a=a, j=j, tick=None, level=None, interactions=None)
    steps, t_end = _step_args(case)
    if entry == "shared" and 33.0 * n * n > MOST_PAIRS:
        return None
    out = _hermite(m, x, v, eps, t_end, **steps)
    if out is None:
        return None
    # every particle sits at t_end: 2^-level_min is the largest step
    energy = _energy(m, out["x"], out["v"], eps)
    return dict(out, energy=energy, block_steps=None, interactions=None)
