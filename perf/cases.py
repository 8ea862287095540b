"""Measured cases: what a program that uses this framework has it do, through its public
entry points (the Python binding and the serving loop), over the range of sizes, precisions
and options that the tests, the benchmark and the workloads of this repository cover.

A case is a dict of plain values; "kind" names the entry point:

  noalloc      gd_force_noalloc: force of an index list from the caller's arrays
  force        gd_predict(t) and gd_force of an index list on a context
  reinit       gd_reinit: initial force of all particles, first steps, energy; state read back
  energy       gd_energy of a synchronised context
  diagnostics  gd_diagnostics: Lagrange radii, relaxation time, level counts
  integrate    gd_reinit and gd_step_to: a whole integration by block steps; state read back
  pool         PoolServer.serve: clusters integrated side by side by continuous batching
"""
import math

import numpy as np
import torch

from paper_1702_00440_amd import gravidy as g
from paper_1702_00440_amd.serving import PoolServer, Request
from synth_inputs.plummer import plummer, plummer_imf, plummer_with_bh

DEV = "cuda:0"
EPS, EPS_BH, ETA, DT_MAX, DT_MIN = 1e-4, 1e-6, 0.01, 0.125, 2.0 ** -22
FLOPS_PAIR = 60    # one acceleration and jerk pair, by the usual convention
FLOPS_ENERGY = 20  # one potential pair
FRACTIONS = (0.01, 0.05, 0.1, 0.25, 0.5, 0.75, 0.9)


def listed():
    return [
        # Latency of the smallest calls: a loop of a program's own that asks for the force of a
        # handful of bodies, from its own arrays.
        {"name": "noalloc_n256", "kind": "noalloc", "n": 256, "n_act": 256, "mixed": False, "eps": EPS},
        # A small active block of the benchmark sphere, and an ordinary one.
        {"name": "force_n16384_act16", "kind": "force", "n": 16384, "n_act": 16, "mixed": False,
         "eps": EPS, "central": False},
        {"name": "force_n16384_act1000", "kind": "force", "n": 16384, "n_act": 1000, "mixed": False,
         "eps": EPS, "central": False},
        # A large odd-sized block in mixed precision, with a central massive particle.
        {"name": "force_n50021_act9973_mixed_central", "kind": "force", "n": 50021, "n_act": 9973,
         "mixed": True, "eps": EPS, "central": True},
        # Start of a run on the largest sphere that has a complete force here: N = 262144 with a
        # mass spectrum.
        {"name": "reinit_n262144", "kind": "reinit", "n": 262144, "mixed": False},
        # The energy check of every synchronised time.
        {"name": "energy_n16384", "kind": "energy", "n": 16384},
        # Lagrange radii of the benchmark sphere.
        {"name": "diagnostics_n16384", "kind": "diagnostics", "n": 16384},
        # Whole integrations over one largest step: the paper's example size, the benchmark size,
        # an odd size in mixed precision, and stars around a central massive particle.
        {"name": "integrate_n1024", "kind": "integrate", "n": 1024, "mixed": False, "central": False},
        {"name": "integrate_n16384", "kind": "integrate", "n": 16384, "mixed": False, "central": False},
        {"name": "integrate_n5003_mixed", "kind": "integrate", "n": 5003, "mixed": True, "central": False},
        {"name": "integrate_n2049_central", "kind": "integrate", "n": 2049, "mixed": False, "central": True},
        # Serving: independent clusters of 256 to 8192 particles, all waiting at the start.
        {"name": "pool_48", "kind": "pool", "clusters": 48, "n_lo": 256, "n_hi": 8192, "mixed": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["noalloc", "force", "force", "force", "reinit", "energy", "diagnostics",
                       "integrate", "integrate", "integrate", "pool"])
    mixed = rng.random() < 0.35
    if kind == "noalloc":
        n = _log(rng, 100, 30000)
        return {"kind": kind, "n": n, "n_act": _log(rng, 1, n), "mixed": mixed,
                "eps": 0.0 if rng.random() < 0.2 else EPS}
    if kind == "force":
        n = _log(rng, 1000, 262144)
        central = rng.random() < 0.25
        return {"kind": kind, "n": n, "n_act": _log(rng, 1, n), "mixed": mixed,
                "eps": 0.0 if not central and rng.random() < 0.2 else EPS, "central": central}
    if kind == "reinit":
        return {"kind": kind, "n": _log(rng, 2000, 262144), "mixed": mixed}
    if kind == "energy":
        return {"kind": kind, "n": _log(rng, 1000, 262144)}
    if kind == "diagnostics":
        return {"kind": kind, "n": _log(rng, 256, 65536)}
    if kind == "integrate":
        return {"kind": kind, "n": _log(rng, 256, 16384), "mixed": mixed, "central": rng.random() < 0.25}
    return {"kind": kind, "clusters": rng.randint(5, 48), "n_lo": 256, "n_hi": _log(rng, 1024, 8192),
            "mixed": mixed}


def _on_device(mxv):
    return [torch.from_numpy(a).to(DEV) for a in mxv]


def _particles(case, seed):
    n = case["n"]
    if case.get("central"):
        return plummer_with_bh(n - 1, seed)
    if case["kind"] == "reinit":
        return plummer_imf(n, seed)
    return plummer(n, seed)


def _rows(case, seed):
    """n_act distinct particles, in no particular order."""
    rng = np.random.Generator(np.random.PCG64([seed, 1]))
    return np.ascontiguousarray(rng.permutation(case["n"])[:case["n_act"]].astype(np.int32))


def _pool_sizes(case):
    """Cluster sizes, log-spaced over [n_lo, n_hi], in a shuffled order."""
    k, lo, hi = case["clusters"], case["n_lo"], case["n_hi"]
    sizes = [int(round(lo * (hi / lo) ** ((i + 0.5) / k))) for i in range(k)]
    return [sizes[i] for i in np.random.Generator(np.random.PCG64(7)).permutation(k)]


def _options(case):
    central = bool(case.get("central"))
    return dict(eta=ETA, eps=case.get("eps", EPS), dt_max=DT_MAX, dt_min=DT_MIN,
                flags=g.GD_FLAG_MIXED if case.get("mixed") else 0, eps_bh=EPS_BH if central else None,
                bh_index=case["n"] - 1 if central else -1)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "pool":
        sizes = _pool_sizes(case)
        requests = [Request(i, 0.0, *_on_device(plummer(n, seed * 1000 + i)), DT_MAX) for i, n in enumerate(sizes)]
        params = g.make_params(ETA, EPS, DT_MAX, DT_MIN, flags=g.GD_FLAG_MIXED if case["mixed"] else 0)
        server = PoolServer(params, len(sizes), g.gd_pool_arena_bytes(len(sizes), sizes), DEV, keep_state=True)
        return {"kind": kind, "server": server, "requests": requests}
    m, x, v = _on_device(_particles(case, seed))
    n = case["n"]
    s = {"kind": kind, "m": m, "x": x, "v": v}
    if kind in ("noalloc", "force"):
        rows = torch.from_numpy(_rows(case, seed)).to(DEV)
        s.update(idx=rows, acc=torch.empty(len(rows), 3, dtype=torch.float64, device=DEV),
                 jerk=torch.empty(len(rows), 3, dtype=torch.float64, device=DEV))
    if kind == "noalloc":
        s["params"] = g.make_params(**_options(case))
        return s
    s["cluster"] = g.Cluster(m, x, v, device=DEV, **_options(case))
    if kind in ("reinit", "integrate"):
        s["out"] = [torch.empty(n, 3, dtype=torch.float64, device=DEV) for _ in range(2)]
    return s


def run(s):
    kind = s["kind"]
    if kind == "noalloc":
        g.gd_force_noalloc(s["params"], s["m"], s["x"], s["v"], s["idx"], s["acc"], s["jerk"])
        return {"acc": s["acc"], "jerk": s["jerk"]}
    if kind == "pool":
        results = sorted(s["server"].serve(s["requests"]), key=lambda r: r.rid)
        return {"x": torch.cat([r.x for r in results]), "v": torch.cat([r.v for r in results]),
                "e": [float(sum(r.stats[k] for r in results)) for k in ("e0", "e")],
                "steps": [int(sum(r.stats[k] for r in results)) for k in ("block_steps", "particle_steps")]}
    ctx = s["cluster"].ctx
    if kind == "force":
        g.gd_predict(ctx, 0.0)
        g.gd_force(ctx, s["idx"], s["acc"], s["jerk"])
        return {"acc": s["acc"], "jerk": s["jerk"]}
    if kind == "energy":
        return list(g.gd_energy(ctx))
    if kind == "diagnostics":
        return g.gd_diagnostics(ctx, FRACTIONS)
    g.gd_reinit(ctx, s["m"], s["x"], s["v"])
    first, second = s["out"]
    if kind == "reinit":
        g.gd_get_state(ctx, a=first, jerk=second)
        st = g.gd_stats_get(ctx)
        return {"a": first, "jerk": second, "e0": st["e0"]}
    st = g.gd_step_to(ctx, DT_MAX)
    g.gd_get_state(ctx, x=first, v=second)
    return {"x": first, "v": second, "e": [st["e0"], st["e"]], "steps": [st["block_steps"], st["particle_steps"]]}


# Particle steps per particle over one largest step (1/8 time unit) of a Plummer sphere, from
# integrations of 1024 to 16384 particles: the work of an integration is what its block steps
# take.
STEPS_PER_PARTICLE = 45.0


def work(case):
    kind = case["kind"]
    if kind == "pool":
        sizes = _pool_sizes(case)
        return {"bytes": sum(n * 56 + n * 48 for n in sizes),
                "flops": FLOPS_PAIR * (1 + STEPS_PER_PARTICLE) * sum(n * n for n in sizes)}
    n = case["n"]
    if kind in ("noalloc", "force"):
        return {"bytes": n * 56 + case["n_act"] * (4 + 48), "flops": FLOPS_PAIR * n * case["n_act"]}
    if kind == "reinit":
        return {"bytes": n * 56 + n * 48, "flops": FLOPS_PAIR * n * n + FLOPS_ENERGY * n * (n - 1) // 2}
    if kind == "energy":
        return {"bytes": n * 56 + 16, "flops": FLOPS_ENERGY * n * (n - 1) // 2}
    if kind == "diagnostics":
        return {"bytes": n * 32, "flops": 12 * n}
    return {"bytes": n * 56 + n * 48, "flops": FLOPS_PAIR * (1 + STEPS_PER_PARTICLE) * n * n}


def _direct(m, x, v, rows, eps, bh):
    """Acceleration and jerk of the given rows by direct summation in 64 bits. bh: index of the
    central particle (its pairs take EPS_BH), or -1."""
    n = m.shape[0]
    acc = torch.empty(len(rows), 3, dtype=torch.float64, device=m.device)
    jerk = torch.empty_like(acc)
    chunk = max(1, 16_000_000 // n)
    e2 = torch.full((n,), eps * eps, dtype=torch.float64, device=m.device)
    if bh >= 0:
        e2[bh] = EPS_BH * EPS_BH
    for k in range(0, len(rows), chunk):
        r = rows[k:k + chunk]
        d = [x[None, :, c] - x[r][:, c, None] for c in range(3)]
        w = [v[None, :, c] - v[r][:, c, None] for c in range(3)]
        soft = e2[None, :].expand(len(r), n)
        if bh >= 0:
            soft = torch.where((r == bh)[:, None], torch.full_like(soft, EPS_BH * EPS_BH), soft)
        s = d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + soft
        own = torch.arange(len(r), device=m.device)
        s[own, r] = 1.0
        q = s.rsqrt()
        q2 = 1.0 / s
        f = m[None, :] * q * q2
        f[own, r] = 0.0
        b = -3.0 * (d[0] * w[0] + d[1] * w[1] + d[2] * w[2]) * q2
        for c in range(3):
            acc[k:k + chunk, c] = (f * d[c]).sum(1)
            jerk[k:k + chunk, c] = (f * (w[c] + b * d[c])).sum(1)
    return acc, jerk


def _potential(m, x, eps):
    n = m.shape[0]
    total = 0.0
    chunk = max(1, 16_000_000 // n)
    for k in range(0, n, chunk):
        s = sum((x[None, :, c] - x[k:k + chunk, c, None]) ** 2 for c in range(3)) + eps * eps
        p = m[None, :] * s.rsqrt()
        own = torch.arange(p.shape[0], device=m.device)
        p[own, own + k] = 0.0
        total += float((m[k:k + chunk] * p.sum(1)).sum())
    return -0.5 * total


def exact(case, seed):
    kind = case["kind"]
    if kind in ("integrate", "pool"):
        return None  # a whole integration in plain torch takes minutes
    n = case["n"]
    if n * case.get("n_act", n) > 2e10:
        return None
    hm, hx, hv = _particles(case, seed)
    m, x, v = _on_device((hm, hx, hv))
    if kind in ("noalloc", "force"):
        rows = torch.from_numpy(_rows(case, seed)).to(DEV).long()
        acc, jerk = _direct(m, x, v, rows, case["eps"], n - 1 if case.get("central") else -1)
        return {"acc": acc, "jerk": jerk}
    if kind == "diagnostics":
        com = (hm[:, None] * hx).sum(0) / hm.sum()
        r = np.sqrt(((hx - com) ** 2).sum(1))
        order = np.argsort(r, kind="stable")
        cum, total = np.cumsum(hm[order]), np.cumsum(hm)[-1]
        radii = [float(r[order[np.searchsorted(cum, f * total)]]) for f in FRACTIONS]
        r_half = radii[FRACTIONS.index(0.5)]
        t_rh = 0.138 * math.sqrt(n * r_half ** 3 / (total / n)) / math.log(0.1 * n)
        return {"fractions": list(FRACTIONS), "radii": radii, "t_rh": t_rh, "r_half": r_half, "levels": None}
    kinetic = 0.5 * float((m * (v * v).sum(1)).sum())
    potential = _potential(m, x, EPS)
    if kind == "energy":
        return [kinetic, potential]
    acc, jerk = _direct(m, x, v, torch.arange(n, device=DEV), EPS, -1)
    return {"a": acc, "jerk": jerk, "e0": kinetic + potential}
