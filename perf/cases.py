"""The work a user of this framework has it do, as a list of timed cases.

Each case goes through the public entry points (``Simulation``, ``Batch``) on
Plummer clusters in Henon units, the stand-in the repository uses for the
star clusters of the paper.  Seven kinds:

``run``         a saved state integrated over an interval in individual block
                steps (``Simulation.run``): what a production run consists of;
``batch``       many independent clusters advanced together to a common time
                by replays of a captured batched step (``Batch.replay``);
``force``       prediction of all particles and the force on an active set
                (``Simulation.predict_force``): the call of a program that
                keeps its own integrator;
``neighbours``  prediction and the force split by neighbour spheres with the
                neighbour lists (``Simulation.force_block_nb``): the regular
                force call of an Ahmad-Cohen integrator;
``init``        initial forces and time steps (``Simulation.init``);
``energy``      the energy check of a run (``Simulation.energy``).

``exact`` computes the same outputs in 64 bits with plain torch operations.
"""
import math

import numpy as np
import torch

from paper_1312_1789_amd import Batch, Simulation

TICK_BITS = 40
TICKS = 1 << TICK_BITS
EPS2 = 1e-8
DEV = "cuda:0"
# Operations of one pair interaction without / with its potential (FMA = 2).
PAIR_FLOPS = {4: 41, 6: 78, 8: 125}
# Block steps per particle and time unit of a Plummer cluster (measured with
# Simulation.stats on the listed runs): the interactions of an interval t are
# this times n^2 t.
STEPS_PER_TIME = {4: 300.0, 6: 500.0}


# --------------------------------------------------------------------------
# The cases.

def listed():
    return [
        # a small cluster in full FP64 at order 4: every block step is a few
        # particles against a thousand, so launches and latency are all there is
        {"name": "run_small", "kind": "run", "n": 1024, "order": 4, "precision": "fp64", "binary": False, "k_end": 5},
        # a production run: 80000 stars, order 6, mixed precision; blocks of
        # every size from one particle to thousands
        {"name": "run_large", "kind": "run", "n": 80000, "order": 6, "precision": "mixed", "binary": False,
         "k_end": 9},
        # a galactic nucleus: stars around a black-hole binary with
        # post-Newtonian terms, FP64
        {"name": "run_binary", "kind": "run", "n": 30002, "order": 4, "precision": "fp64", "binary": True, "k_end": 7},
        # an ensemble of clusters of 2^10 to 2^14 stars
        {"name": "batch", "kind": "batch", "clusters": 32, "lo": 10.0, "hi": 14.0, "order": 6, "precision": "mixed",
         "k_end": 8},
        # a block step of the largest system with hardly any active particles
        {"name": "force_few", "kind": "force", "n": 1048576, "n_act": 5, "order": 6, "precision": "mixed",
         "pot": False},
        # a middling active set in FP64 at order 8
        {"name": "force_some", "kind": "force", "n": 100003, "n_act": 201, "order": 8, "precision": "fp64",
         "pot": False},
        # a large block of a large system
        {"name": "force_block", "kind": "force", "n": 262144, "n_act": 3001, "order": 6, "precision": "mixed",
         "pot": False},
        # a synchronised step: every particle active
        {"name": "force_all", "kind": "force", "n": 90000, "n_act": 90000, "order": 6, "precision": "mixed",
         "pot": False},
        # the FP32-only arithmetic, with the potential
        {"name": "force_ds", "kind": "force", "n": 65537, "n_act": 1000, "order": 4, "precision": "ds", "pot": True},
        # a regular-force step of an Ahmad-Cohen integrator
        {"name": "neighbours", "kind": "neighbours", "n": 131072, "n_act": 1024, "precision": "mixed", "max_nb": 128},
        # the start of a run
        {"name": "init", "kind": "init", "n": 40961, "order": 6, "precision": "mixed"},
        # the energy check at each output time
        {"name": "energy", "kind": "energy", "n": 32768},
    ]


def _between(rng, lo, hi):
    """A whole number spread over its logarithm; three in four as it falls,
    one in four a power of two."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return 1 << int(round(math.log2(n))) if rng.random() < 0.25 else n


def draw(rng):
    kind = rng.choice(["run", "run", "batch", "force", "force", "force", "neighbours", "init", "energy"])
    if kind == "run":
        n = _between(rng, 1000, 60000)
        binary = rng.random() < 0.3
        order = 4 if binary else rng.choice([4, 6])
        precision = "fp64" if binary else ("mixed" if order == 6 else rng.choice(["fp64", "mixed"]))
        return {"kind": kind, "n": n, "order": order, "precision": precision, "binary": binary,
                "k_end": 6 + int(3 * math.log2(n / 1000) / 7)}
    if kind == "batch":
        lo = rng.uniform(9.0, 11.0)
        return {"kind": kind, "clusters": rng.randint(8, 48), "lo": lo, "hi": lo + rng.uniform(1.0, 3.0),
                "order": rng.choice([4, 6]), "precision": rng.choice(["mixed", "mixed", "fp64"]), "k_end": 8}
    if kind == "force":
        n = _between(rng, 4096, 1048576)
        n_act = min(_between(rng, 1, n), int(3e9 / n))
        return {"kind": kind, "n": n, "n_act": n_act, "order": rng.choice([4, 6, 6, 8]),
                "precision": rng.choice(["mixed", "mixed", "fp64", "ds"]), "pot": rng.random() < 0.2}
    if kind == "neighbours":
        n = _between(rng, 8192, 262144)
        return {"kind": kind, "n": n, "n_act": min(n, _between(rng, 64, 2048)),
                "precision": rng.choice(["mixed", "fp64"]), "max_nb": rng.choice([96, 128, 256])}
    if kind == "init":
        return {"kind": kind, "n": _between(rng, 1000, 40000), "order": rng.choice([4, 6, 8]),
                "precision": rng.choice(["mixed", "fp64"])}
    return {"kind": kind, "n": _between(rng, 1000, 100000)}


# --------------------------------------------------------------------------
# Inputs, drawn on the GPU from the seed.

def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 13)
    return g


def _directions(g, r):
    n = r.numel()
    c = 2.0 * torch.rand(n, generator=g, device=DEV, dtype=torch.float64) - 1.0
    p = 2.0 * math.pi * torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    s = torch.sqrt(1.0 - c * c)
    return torch.stack([r * s * torch.cos(p), r * s * torch.sin(p), r * c])


def _plummer(n, g):
    """Plummer sphere in Henon units (Aarseth, Henon & Wielen 1974)."""
    X = 1e-9 + 0.999 * torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    r = 1.0 / torch.sqrt(X ** (-2.0 / 3.0) - 1.0)
    q = torch.zeros(n, device=DEV, dtype=torch.float64)
    todo = torch.ones(n, device=DEV, dtype=torch.bool)
    for _ in range(60):   # rejection from q^2 (1 - q^2)^(7/2), about two in five accepted a time
        t = torch.rand((2, n), generator=g, device=DEV, dtype=torch.float64)
        ok = todo & (0.1 * t[1] < t[0] ** 2 * (1.0 - t[0] ** 2) ** 3.5)
        q = torch.where(ok, t[0], q)
        todo &= ~ok
    x = _directions(g, r) * (3.0 * math.pi / 16.0)
    v = _directions(g, q * math.sqrt(2.0) * (1.0 + r * r) ** (-0.25)) * math.sqrt(16.0 / (3.0 * math.pi))
    m = torch.full((n,), 1.0 / n, device=DEV, dtype=torch.float64)
    return m, x - x.mean(1, keepdim=True), v - v.mean(1, keepdim=True)


# Two holes of 0.01 at separation 0.02 on their circular orbit, speed of light 8.
_BH = {"m": 0.01, "sep": 0.02, "c_light": 8.0, "pn_terms": 7}


def _model(case, seed):
    """(m, x, v) of a run; a binary takes indices 0 and 1."""
    n = case["n"]
    if not case.get("binary"):
        return _plummer(n, _generator(seed))
    m, x, v = _plummer(n - 2, _generator(seed))
    s, u = _BH["sep"] / 2, math.sqrt(2 * _BH["m"] / _BH["sep"]) / 2
    pos = torch.tensor([[s, -s], [0.0, 0.0], [0.0, 0.0]], device=DEV, dtype=torch.float64)
    vel = torch.tensor([[0.0, 0.0], [u, -u], [0.0, 0.0]], device=DEV, dtype=torch.float64)
    mass = torch.full((2,), _BH["m"], device=DEV, dtype=torch.float64)
    return torch.cat([mass, m]), torch.cat([pos, x], 1), torch.cat([vel, v], 1)


def _options(case):
    """Keyword arguments of a run's Simulation."""
    o = {"order": case["order"], "precision": case["precision"], "eps2": EPS2, "eta": 0.1 if case["order"] > 4 else 0.01,
         "k_min": 3, "k_max": 20, "dt_rule": 2}
    if case.get("binary"):
        o.update(n_hard=2, c_light=_BH["c_light"], pn_terms=_BH["pn_terms"])
    return o


def _steps(d, o):
    """Levels a run has settled to, from the scheme's step criterion on
    a .. a^(3).  (The first steps after init follow |a| / |jerk|, which is tiny
    where |a| happens to be; a run in mixed precision takes long to leave
    those.)"""
    N = [_norm(a) for a in d[:4]]
    if o["order"] == 4:
        return _level(torch.sqrt(o["eta"] * (N[0] * N[2] + N[1] ** 2) / (N[1] * N[3] + N[2] ** 2)), o)
    return _level(o["eta"] * (torch.sqrt(N[0] * N[2]) + N[1]) / (torch.sqrt(N[1] * N[3]) + N[2]), o)


def _set_steps(s, o, parts):
    """The settled levels into `s`, whose clusters (m, x, v) are `parts`."""
    if o["order"] >= 6:
        s.level.copy_(_steps(s.d, o))
        return
    at = 0
    for p in parts:   # an order-4 state holds no a^(2), a^(3)
        six = Simulation(*_host(*p), order=6, eps2=EPS2, n_hard=o.get("n_hard", 0))
        six.init()
        n = six.n
        s.level[at:at + n] = _steps(six.d, o)
        at += n


def _host(*ts):
    return [t.cpu().numpy() for t in ts]


def _sizes(case):
    k = case["clusters"]
    return [int(round(2.0 ** (case["lo"] + (case["hi"] - case["lo"]) * (c + 0.5) / k))) for c in range(k)]


def _clusters(case, seed):
    g = _generator(seed)
    return [_plummer(n, g) for n in _sizes(case)]


def _block_state(case, seed):
    """A block-step state in mid-run: every particle at a multiple of its own
    step 2^-6 .. 2^-14, derivatives of a cluster's magnitudes, and the time
    its next block step is due."""
    n, order = case["n"], case["order"]
    g = _generator(seed)
    m, x, v = _plummer(n, g)
    d = [torch.randn((3, n), generator=g, device=DEV, dtype=torch.float64) * 10.0 ** k for k in range(order - 2)]
    level = torch.randint(6, 15, (n,), generator=g, device=DEV, dtype=torch.int32)
    T = 3 * (TICKS >> 3) + (TICKS >> 5)
    dt = torch.ones_like(level, dtype=torch.int64) << (TICK_BITS - level.long())
    t = torch.div(T - 1, dt, rounding_mode="floor") * dt
    act = torch.sort(torch.randperm(n, generator=g, device=DEV)[:case["n_act"]])[0].to(torch.int32)
    return m, x, v, d, t, level, T, act


def _radii(x, act, k):
    """h^2 between the k-th and the next nearest particle of each row."""
    h2 = torch.empty(act.numel(), device=DEV, dtype=torch.float64)
    for a in range(0, act.numel(), 64):
        rows = act[a:a + 64].long()
        r2 = sum((x[c][None, :] - x[c][rows][:, None]) ** 2 for c in range(3))
        s = torch.topk(r2, k + 2, largest=False, sorted=True)[0]   # the row itself first
        h2[a:a + 64] = torch.sqrt(s[:, k] * s[:, k + 1])
    return h2


_NEIGHBOURS = 64


def _with_state(case, seed):
    m, x, v, d, t, level, T, act = _block_state(case, seed)
    sim = Simulation(*_host(m, x, v), order=case["order"], precision=case["precision"], eps2=EPS2)
    for to, of in zip(sim.d, d):
        to.copy_(of)
    sim.t_tick.copy_(t)
    sim.level.copy_(level)
    return sim, T, act


def prepare(case, seed):
    kind = case["kind"]
    if kind == "run":
        p, o = _model(case, seed), _options(case)
        sim = Simulation(*_host(*p), **o)
        sim.init()
        _set_steps(sim, o, [p])
        return {"kind": kind, "sim": sim, "saved": [t.clone() for t in _state(sim)], "end": TICKS >> case["k_end"]}
    if kind == "batch":
        parts, o = _clusters(case, seed), _options(case)
        b = Batch([_host(*c) for c in parts], **o)
        b.init()
        b.set_end(TICKS >> case["k_end"])
        b.capture()
        b.synchronize()
        _set_steps(b, o, parts)
        saved = [t.clone() for t in _state(b)]
        torch.cuda.synchronize()
        return {"kind": kind, "b": b, "saved": saved}
    if kind == "force":
        sim, T, act = _with_state(case, seed)
        return {"kind": kind, "sim": sim, "T": T, "act": act, "out": sim.alloc_forces(act.numel()),
                "keys": ["acc", "jrk", "snp", "crk"][:case["order"] // 2] + (["pot"] if case["pot"] else [])}
    if kind == "neighbours":
        case = dict(case, order=4)
        sim, T, act = _with_state(case, seed)
        z = lambda: torch.empty((3, act.numel()), dtype=torch.float64, device=DEV)
        out = {"acc_irr": z(), "jrk_irr": z(), "acc_reg": z(), "jrk_reg": z(),
               "nb_count": torch.empty(act.numel(), dtype=torch.int32, device=DEV),
               "nb_list": torch.full((act.numel(), case["max_nb"]), -1, dtype=torch.int32, device=DEV)}
        xp = _predict(sim.x, sim.v, sim.d, sim.t_tick, T, 4)[0]
        return {"kind": kind, "sim": sim, "T": T, "act": act, "out": out, "h2": _radii(xp, act, _NEIGHBOURS),
                "max_nb": case["max_nb"]}
    m, x, v = _plummer(case["n"], _generator(seed))
    o = {"order": case["order"], "precision": case["precision"]} if kind == "init" else {}
    return {"kind": kind, "sim": Simulation(*_host(m, x, v), eps2=EPS2, **o)}


def _state(s):
    return [s.x, s.v, *s.d, s.t_tick, s.level]


# --------------------------------------------------------------------------
# One pass.

def run(state):
    kind = state["kind"]
    if kind == "run":
        # back to the saved state, as a program does that repeats an interval
        sim = state["sim"]
        for to, of in zip(_state(sim), state["saved"]):
            to.copy_(of)
        sim.run(state["end"])
        return _state(sim)
    if kind == "batch":
        b = state["b"]
        with torch.cuda.stream(b.stream):
            for to, of in zip(_state(b), state["saved"]):
                to.copy_(of)
        live = 1
        while live:   # until every cluster has reached the end
            b.replay(16)
            live, _ = b.poll()
        return _state(b)
    sim = state["sim"]
    if kind == "force":
        out = sim.predict_force(state["T"], state["act"], state["out"], with_pot="pot" in state["keys"])
        return [out[k] for k in state["keys"]]
    if kind == "neighbours":
        sim.predict(state["T"])
        return sim.force_block_nb(state["act"], state["h2"], state["max_nb"], state["out"])
    if kind == "init":
        sim.init()
        return _state(sim)[2:]
    return np.array(sim.energy())


def work(case):
    kind = case["kind"]
    order = case.get("order", 4)
    state = 8 * (3 * order + 2)   # bytes of a particle's stored state: m, x, v, derivatives, time (and level)
    if kind == "run":
        n = case["n"]
        pairs = STEPS_PER_TIME[order] * 2.0 ** -case["k_end"] * n * n
        return {"bytes": 2 * n * state, "flops": pairs * PAIR_FLOPS[order]}
    if kind == "batch":
        pairs = STEPS_PER_TIME[order] * 2.0 ** -case["k_end"] * sum(n * n for n in _sizes(case))
        return {"bytes": 2 * sum(_sizes(case)) * state, "flops": pairs * PAIR_FLOPS[order]}
    n = case["n"]
    if kind == "force":
        outs = 3 * (order // 2) + (1 if case["pot"] else 0)
        return {"bytes": n * state + 8 * outs * case["n_act"],
                "flops": float(n) * case["n_act"] * (PAIR_FLOPS[order] + (2 if case["pot"] else 0))}
    if kind == "neighbours":
        return {"bytes": n * state + case["n_act"] * (12 * 8 + 4 + 4 * _NEIGHBOURS),
                "flops": float(n) * case["n_act"] * PAIR_FLOPS[4]}
    if kind == "init":
        # acceleration and jerk; snap and crackle in a second pass over all pairs
        return {"bytes": n * (56 + 24 * (order - 2) + 12),
                "flops": float(n) * n * (PAIR_FLOPS[4] + (PAIR_FLOPS[8] if order >= 6 else 0))}
    return {"bytes": 56 * n, "flops": 0.5 * n * n * 11}   # each pair once: differences, r^2, 1/r, sum


# --------------------------------------------------------------------------
# The same in 64 bits with plain torch operations.

def _pair_sums(m, x, v, a, j, rows, order, n_hard=0, pot=False, inside=None):
    """Acceleration and its order/2 - 1 derivatives on `rows` (Nitadori &
    Makino 2008), and the potential; inside: h^2 per row, then the sums over
    the neighbours and over the others."""
    n, q = m.numel(), order // 2
    out = [torch.zeros((3 * q + 1, rows.numel()), dtype=torch.float64, device=DEV) for _ in range(2 if inside is not None else 1)]
    step = max(1, (1 << 24) // n)
    for s in range(0, rows.numel(), step):
        i = rows[s:s + step].long()
        dx = [x[c][None, :] - x[c][i][:, None] for c in range(3)]
        dv = [v[c][None, :] - v[c][i][:, None] for c in range(3)]
        r2 = dx[0] ** 2 + dx[1] ** 2 + dx[2] ** 2
        near = r2 < inside[s:s + step][:, None] if inside is not None else None
        hard = (i < n_hard).nonzero().flatten()
        bare = r2[hard, :n_hard]
        r2 = r2 + EPS2
        r2[hard, :n_hard] = bare
        own = torch.arange(i.numel(), device=DEV)
        r2[own, i] = 1.0
        mr = m[None, :] / torch.sqrt(r2)
        mr[own, i] = 0.0
        mu = mr / r2
        A = [mu * dx[c] for c in range(3)]
        parts = A
        if order >= 4:
            al = (dx[0] * dv[0] + dx[1] * dv[1] + dx[2] * dv[2]) / r2
            J = [mu * dv[c] - 3 * al * A[c] for c in range(3)]
            parts = parts + J
        if order >= 6:
            da = [a[c][None, :] - a[c][i][:, None] for c in range(3)]
            be = (sum(dv[c] ** 2 for c in range(3)) + sum(dx[c] * da[c] for c in range(3))) / r2 + al ** 2
            S = [mu * da[c] - 6 * al * J[c] - 3 * be * A[c] for c in range(3)]
            parts = parts + S
        if order >= 8:
            dj = [j[c][None, :] - j[c][i][:, None] for c in range(3)]
            ga = (3 * sum(dv[c] * da[c] for c in range(3)) + sum(dx[c] * dj[c] for c in range(3))) / r2 \
                + al * (3 * be - 4 * al ** 2)
            parts = parts + [mu * dj[c] - 9 * al * S[c] - 9 * be * J[c] - 3 * ga * A[c] for c in range(3)]
        parts = parts + ([mr] if pot else [])
        for k, p in enumerate(parts):
            k = 3 * q if pot and k == len(parts) - 1 else k
            if near is None:
                out[0][k, s:s + step] = p.sum(1)
            else:
                out[0][k, s:s + step] = torch.where(near, p, 0.0).sum(1)
                out[1][k, s:s + step] = torch.where(near, 0.0, p).sum(1)
    res = [[o[3 * k:3 * k + 3] for k in range(q)] + ([-o[3 * q]] if pot else []) for o in out]
    return res[0] if inside is None else res


def _pn(m, x, v, terms, c):
    """Post-Newtonian acceleration and jerk of the pair (0, 1): 1PN, 2PN and
    2.5PN relative acceleration in harmonic coordinates (Blanchet), its rate
    along the pair's Newtonian motion."""
    m1, m2 = m[0], m[1]
    M = m1 + m2
    nu = m1 * m2 / M ** 2

    def rel(X, V):
        r = torch.sqrt((X * X).sum())
        nx, v2, g = X / r, (V * V).sum(), M / r
        rd = (nx * V).sum()
        A = B = torch.zeros((), dtype=torch.float64, device=DEV)
        if terms & 1:
            A = A + (-1.5 * nu * rd ** 2 + (1 + 3 * nu) * v2 - 2 * (2 + nu) * g) / c ** 2
            B = B - 2 * (2 - nu) * rd / c ** 2
        if terms & 2:
            A = A + (15 / 8 * nu * rd ** 4 - 45 / 8 * nu ** 2 * rd ** 4 - 4.5 * nu * rd ** 2 * v2
                     + 6 * nu ** 2 * rd ** 2 * v2 + 3 * nu * v2 ** 2 - 4 * nu ** 2 * v2 ** 2
                     + g * (-2 * rd ** 2 - 25 * nu * rd ** 2 - 2 * nu ** 2 * rd ** 2 - 6.5 * nu * v2
                            + 2 * nu ** 2 * v2) + g ** 2 * (9 + 87 / 4 * nu)) / c ** 4
            B = B + (4.5 * nu * rd ** 3 + 3 * nu ** 2 * rd ** 3 - 7.5 * nu * rd * v2 - 2 * nu ** 2 * rd * v2
                     + g * rd * (2 + 20.5 * nu + 4 * nu ** 2)) / c ** 4
        if terms & 4:
            A = A - 1.6 * nu * g * rd * (17 / 3 * g + 3 * v2) / c ** 5
            B = B + 1.6 * nu * g * (3 * g + v2) / c ** 5
        return -(M / r ** 2) * (A * nx + B * V)

    X, V = x[:, 0] - x[:, 1], v[:, 0] - v[:, 1]
    newton = -M * X / torch.sqrt((X * X).sum()) ** 3
    a, j = torch.func.jvp(rel, (X, V), (V, newton))
    w = torch.stack([m2 / M, -m1 / M])[None, :]
    return a[:, None] * w, j[:, None] * w


def _taylor(D, dt):
    s, f = torch.zeros_like(D[0]), torch.ones_like(dt)
    for k, d in enumerate(D):
        s = s + d * f
        f = f * dt / (k + 1)
    return s


def _predict(x, v, d, t, T, order):
    dt = (T - t).double() / TICKS
    D = [x, v, *d]
    return [_taylor(D[k:order], dt) for k in range(4)] if order >= 6 else [_taylor(D[:4], dt), _taylor(D[1:4], dt), None, None]


def _level(dt, o):
    e = torch.frexp(dt)[1] - 1   # 2^e <= dt < 2^(e+1)
    return torch.clamp(-e, o["k_min"], o["k_max"]).to(torch.int32)


def _norm(a):
    return torch.sqrt((a * a).sum(0))


def _start(m, x, v, o, order):
    """Initial (Newtonian) derivatives of a run."""
    nh = o.get("n_hard", 0)
    rows = torch.arange(m.numel(), device=DEV)
    d = _pair_sums(m, x, v, None, None, rows, 4, nh)
    if order >= 6:
        d = d + _pair_sums(m, x, v, *d, rows, 8, nh)[2:]
    return d + [torch.zeros_like(d[0]) for _ in range(order - 2 - len(d))]


def _interval(m, x, v, o, end):
    """Block steps up to tick `end` from the start of a run."""
    order, nh = o["order"], o.get("n_hard", 0)
    q = order // 2
    x, v = x.clone(), v.clone()
    d = _start(m, x, v, o, 6)
    level = _steps(d, o)
    d = d[:order - 2]
    if o.get("pn_terms"):
        p = _pn(m, x, v, o["pn_terms"], o["c_light"])
        for e in range(2):
            d[e][:, :2] += p[e]
    t = torch.zeros_like(level, dtype=torch.int64)
    ticks = lambda l: torch.ones_like(l, dtype=torch.int64) << (TICK_BITS - l.long())
    CP = {4: [[6, 2], [12, 6]], 6: [[-60, -24, -3], [-360, -168, -24], [-720, -360, -60]]}[order]
    CQ = {4: [[-6, 4], [-12, 6]], 6: [[60, -36, 9], [360, -192, 36], [720, -360, 60]]}[order]
    while True:
        due = t + ticks(level)
        T = int(due.min())
        if T > end:
            break
        act = (due == T).nonzero().flatten()
        xp, vp, ap, jp = _predict(x, v, d, t, T, order)
        F = _pair_sums(m, xp, vp, ap, jp, act, order, nh)
        if o.get("pn_terms") and int(act[0]) < 2:
            p = _pn(m, xp, vp, o["pn_terms"], o["c_light"])
            for k, i in enumerate(act[:2].tolist()):
                if i < 2:
                    for e in range(2):
                        F[e][:, k] += p[e][:, i]
        h = (T - t[act]).double() / TICKS
        A0 = [d[k][:, act] for k in range(q)]
        x0, v0 = x[:, act], v[:, act]
        if order == 4:
            v1 = v0 + h / 2 * (A0[0] + F[0]) + h ** 2 / 12 * (A0[1] - F[1])
            x1 = x0 + h / 2 * (v0 + v1) + h ** 2 / 12 * (A0[0] - F[0])
        else:
            v1 = v0 + h / 2 * (A0[0] + F[0]) + h ** 2 / 10 * (A0[1] - F[1]) + h ** 3 / 120 * (A0[2] + F[2])
            x1 = x0 + h / 2 * (v0 + v1) + h ** 2 / 10 * (A0[0] - F[0]) + h ** 3 / 120 * (A0[1] + F[1])
        high = [sum(CP[e][k] * A0[k] * h ** k + CQ[e][k] * F[k] * h ** k for k in range(q)) / h ** (q + e)
                for e in range(q)]
        new = F[:q] + high
        old, k = level[act], _steps(new, o)
        up = torch.clamp(old - 1, min=o["k_min"])
        k = torch.where(k < old, torch.where(T % ticks(up) == 0, up, old), k)
        x[:, act], v[:, act], level[act], t[act] = x1, v1, k, T
        for e in range(order - 2):
            d[e][:, act] = new[e]
    if order == 6 and o["precision"] == "mixed":
        d[3] = None   # interpolated over h^3: on the shortest steps the rounding of the FP32 pair terms
    return [x, v, *d, None, None]


def exact(case, seed):
    kind = case["kind"]
    if kind == "run":
        return _interval(*_model(case, seed), _options(case), TICKS >> case["k_end"])
    if kind == "batch":
        o = _options(case)
        parts = [_interval(*c, o, TICKS >> case["k_end"]) for c in _clusters(case, seed)]
        return [None if k[0] is None else torch.cat(k, 1) for k in zip(*parts)]
    if kind in ("force", "neighbours"):
        order = case.get("order", 4)
        m, x, v, d, t, _, T, act = _block_state(dict(case, order=order), seed)
        p = _predict(x, v, d, t, T, order)
        if kind == "force":
            return _pair_sums(m, *p, act, order, pot=case["pot"])
        irr, reg = _pair_sums(m, *p, act, 4, inside=_radii(p[0], act, _NEIGHBOURS))
        return {"acc_irr": irr[0], "jrk_irr": irr[1], "acc_reg": reg[0], "jrk_reg": reg[1]}
    m, x, v = _plummer(case["n"], _generator(seed))
    if kind == "init":
        return _start(m, x, v, {}, case["order"]) + [None, None]
    pot = _pair_sums(m, x, v, None, None, torch.arange(case["n"], device=DEV), 2, pot=True)[1]
    return np.array([float(0.5 * (m * (v * v).sum(0)).sum()), float(0.5 * (m * pot).sum())])
