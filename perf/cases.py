"""Timed cases of the gravity solver: what its users call, over the sizes they use.

A case is one pass through the public entry points (`api.Tree.rebuild` with
`evaluate` or `evaluate_forest`, `api.evaluate_forces_oneshot`,
`session.Session.step`) on a particle set that is already on the GPU:

* entry "step":    a kept tree rebuilt for the particles, then evaluated (a
                   server slot, or a time step driven from outside);
* entry "oneshot": build, evaluate and destroy in one call (a single solve);
* entry "forest":  several small sets solved together, each with its own
                   theta (the server's batches);
* entry "session": leapfrog steps on resident state.

Orders, opening angles, leaf sizes and distributions are those of the
repository's workloads and of its serving trace (N from 1e3 to 5e5, p in
{2, 4, 6}, theta in {0.4, 0.6, 0.8}).  Inputs are drawn on the GPU from the
seed alone.
"""

from __future__ import annotations

import math
import random

import torch

from paper_2107_07166_amd import api, session

EPS = 1e-3
EXACT_MAX_N = 300_000  # the direct sum of a larger set takes too long

# Floating-point operations of one directed far pair (derivatives, contraction) by order.
PAIR_FLOPS = {
    "standard": {1: 40, 2: 90, 4: 362, 6: 1760},
    "conserving": {1: 60, 2: 150, 3: 350, 4: 740, 5: 1900, 6: 4298},
}


def listed():
    return [
        # the smallest solve: 2048 particles in a ball at second order, where launches and waits are all there is
        dict(name="ball-2k", entry="step", kind="ball", n=2048, p=2, theta=0.5, variant="conserving",
             precision="mixed32", n_leaf=64),
        # one small set solved by a single call, nothing kept: a script, or a service's rare request
        dict(name="oneshot-10k", entry="oneshot", kind="plummer", n=10007, p=4, theta=0.6, variant="standard",
             precision="mixed32", n_leaf=64),
        # a small resident system advanced several steps per call
        dict(name="session-5k", entry="session", kind="plummer", n=5000, p=4, theta=0.5, variant="conserving",
             precision="mixed32", n_leaf=64, steps=4),
        # the same in full double precision with small leaves, for reference orbits
        dict(name="fp64-step-20k", entry="step", kind="plummer", n=20011, p=4, theta=0.5, variant="conserving",
             precision="fp64", n_leaf=32),
        # a server's batch of small requests, ragged sizes, each with its own opening angle
        dict(name="forest-16", entry="forest", kind="ball", n=131072, sets=16, p=4, theta=0.6, variant="conserving",
             precision="mixed32", n_leaf=64),
        # an ordinary serving request at high order
        dict(name="slot-100k", entry="step", kind="disk", n=100003, p=6, theta=0.6, variant="conserving",
             precision="mixed32", n_leaf=64),
        # forces and potential, for the energy of a snapshot
        dict(name="potential-262k", entry="step", kind="plummer", n=262144, p=4, theta=0.5, variant="standard",
             precision="mixed32", n_leaf=64, potential=True),
        # double precision at a production size
        dict(name="fp64-262k", entry="step", kind="plummer", n=262139, p=4, theta=0.5, variant="conserving",
             precision="fp64", n_leaf=64),
        # a raised projection scalar: the accurate torque-free force
        dict(name="knob-262k", entry="step", kind="plummer", n=262144, p=4, theta=0.5, variant="conserving",
             precision="mixed32", n_leaf=64, scalar_degree=5),
        # a binary of two polytropes, one leapfrog step of a long run
        dict(name="binary-1m", entry="session", kind="binary", n=1048576, p=4, theta=0.7, variant="conserving",
             precision="mixed32", n_leaf=64, steps=1),
        # the benchmark's headline step
        dict(name="plummer-1m", entry="step", kind="plummer", n=1048576, p=4, theta=0.5, variant="conserving",
             precision="mixed32", n_leaf=64),
        # the largest: the exponential disk at high order and a wide angle
        dict(name="disk-4m", entry="step", kind="disk", n=4194304, p=6, theta=0.8, variant="conserving",
             precision="mixed32", n_leaf=128),
    ]


def draw(rng: random.Random):
    """One more case: the entry, the distribution and the options uniform, the
    size uniform in its logarithm over the range that the entry is used for."""
    entry = rng.choice(["step", "step", "step", "oneshot", "forest", "session"])
    precision = rng.choice(["mixed32", "mixed32", "mixed32", "fp64"])
    lo, hi = {"step": (1e3, 1.2e6), "oneshot": (1e3, 5e5), "forest": (8e3, 2.6e5), "session": (1e3, 1e6)}[entry]
    if precision == "fp64":
        hi = min(hi, 3e5)
    n = int(10 ** rng.uniform(math.log10(lo), math.log10(hi)))
    kind = rng.choice(["plummer", "binary"] if entry == "session" else ["ball", "plummer", "disk"])
    if kind == "binary":
        n += n % 2
    p = rng.choice([2, 4, 6])
    theta = rng.choice([0.4, 0.6, 0.8])
    if p == 2:
        theta = min(theta, 0.6)  # at second order a wide angle is of no use
    if p == 6 and theta < 0.6 and n > 200_000:
        theta = 0.6
    c = dict(entry=entry, kind=kind, n=n, p=p, theta=theta, variant=rng.choice(["standard", "conserving"]),
             precision=precision, n_leaf=rng.choice([32, 64, 64, 128]))
    if entry == "forest":
        c["sets"] = rng.randint(3, 24)
    elif entry == "session":
        c["steps"] = 4 if n < 50_000 else 1
    elif entry == "step" and c["variant"] == "standard" and rng.random() < 0.3:
        c["potential"] = True
    elif entry == "step" and c["variant"] == "conserving" and p <= 4 and n <= 300_000 and rng.random() < 0.25:
        c["scalar_degree"] = p
    return c


# ---- inputs -------------------------------------------------------------------

def _rand(g, n):
    return torch.rand(n, dtype=torch.float64, device="cuda", generator=g)


def _isotropic(g, n):
    v = torch.randn((n, 3), dtype=torch.float64, device="cuda", generator=g)
    return v / v.square().sum(1, keepdim=True).sqrt()


def _draw_set(kind, n, g):
    """Positions, masses and velocities (n, equal masses, total 1)."""
    mass = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
    if kind == "ball":
        pos = _isotropic(g, n) * _rand(g, n).pow(1.0 / 3.0)[:, None]
        return pos, mass, torch.zeros_like(pos)
    if kind == "plummer":
        u = (_rand(g, n) * 0.999).clamp_min(1e-300)
        r = 1.0 / (u.pow(-2.0 / 3.0) - 1.0).sqrt()
        pos = _isotropic(g, n) * r[:, None]
        # speeds of the isotropic equilibrium: q = v / v_esc with density q^2 (1 - q^2)^(7/2)
        q = torch.full((n,), -1.0, dtype=torch.float64, device="cuda")
        for _ in range(40):
            x, y = _rand(g, n), _rand(g, n) * 0.1
            q = torch.where((q < 0) & (y < x * x * (1.0 - x * x).pow(3.5)), x, q)
        q = torch.where(q < 0, torch.full_like(q, 0.4), q)
        vesc = math.sqrt(2.0) * (1.0 + r * r).pow(-0.25)
        return pos, mass, _isotropic(g, n) * (q * vesc)[:, None]
    if kind == "disk":
        u = _rand(g, n) * (1.0 - 11.0 * math.exp(-10.0))
        R = torch.where(u < 0.5, (2.0 * u).sqrt() + 1e-12, torch.full_like(u, 2.0))
        for _ in range(40):
            e = torch.exp(-R)
            R = (R - (1.0 - (1.0 + R) * e - u) / (R * e).clamp_min(1e-300)).clamp(1e-12, 10.0)
        z = (0.05 * torch.atanh((2.0 * _rand(g, n) - 1.0).clamp(-1.0 + 1e-16, 1.0 - 1e-16))).clamp(-0.5, 0.5)
        phi = _rand(g, n) * (2.0 * math.pi)
        pos = torch.stack([R * torch.cos(phi), R * torch.sin(phi), z], dim=1)
        return pos, mass, torch.zeros_like(pos)
    # two n = 1 polytropes of radius 1 at (-2, 0, 0) and (2, 0, 0) on a circular orbit
    h = n // 2
    u = _rand(g, n)
    lo, hi = torch.zeros_like(u), torch.ones_like(u)
    for _ in range(55):
        mid = 0.5 * (lo + hi)
        below = (torch.sin(math.pi * mid) - math.pi * mid * torch.cos(math.pi * mid)) / math.pi < u
        lo, hi = torch.where(below, mid, lo), torch.where(below, hi, mid)
    pos = _isotropic(g, n) * (0.5 * (lo + hi))[:, None]
    vel = torch.zeros_like(pos)
    pos[:h, 0] -= 2.0
    pos[h:, 0] += 2.0
    vel[:h, 1], vel[h:, 1] = -0.25, 0.25
    return pos, mass, vel


def _offsets(case):
    """Ragged set boundaries: the sizes grow about threefold from first to last."""
    n, k = int(case["n"]), int(case["sets"])
    w = [1.0 + 2.0 * i / max(k - 1, 1) for i in range(k)]
    off, acc = [0], 0.0
    for x in w:
        acc += x
        off.append(int(n * acc / sum(w)))
    off[-1] = n
    return off


def _thetas(case):
    return [(0.4, 0.6, 0.8)[i % 3] for i in range(int(case["sets"]))]


DT = 1e-5  # short steps: the system looks the same after many passes


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    n = int(case["n"])
    if case["entry"] != "forest":
        return tuple(t.contiguous() for t in _draw_set(case["kind"], n, g))
    off = _offsets(case)
    parts = [_draw_set(case["kind"], b - a, g) for a, b in zip(off, off[1:])]
    return tuple(torch.cat([q[i] for q in parts]).contiguous() for i in range(3))


def prepare(case, seed):
    pos, mass, vel = _inputs(case, seed)
    s = dict(case=dict(case), pos=pos, mass=mass)
    ctx = api.default_context(0)
    kw = dict(p=case["p"], theta=case["theta"], eps=EPS, variant=case["variant"], precision=case["precision"])
    if case["entry"] == "session":
        s["session"] = session.Session(ctx, pos, vel, mass, n_leaf=case["n_leaf"], **kw)
        return s
    s["out"] = torch.empty_like(pos)
    if case["entry"] == "forest":
        s["offsets"], s["thetas"] = _offsets(case), _thetas(case)
        s["tree"] = api.Tree(ctx, pos, mass, n_leaf=case["n_leaf"], offsets=s["offsets"])
        kw.pop("theta")
    elif case["entry"] == "step":
        s["tree"] = api.Tree(ctx, pos, mass, n_leaf=case["n_leaf"])
        if case.get("potential"):
            s["pot"] = kw["pot"] = torch.empty_like(mass)
        if case.get("scalar_degree"):
            kw["scalar_degree"] = case["scalar_degree"]
    s["kw"] = kw
    return s


def run(s):
    case = s["case"]
    if case["entry"] == "session":
        ses = s["session"]
        ses.step(DT, case["steps"])
        return {"pos": ses.pos, "vel": ses.vel, "force": ses.force}
    if case["entry"] == "oneshot":
        return api.evaluate_forces_oneshot(s["pos"], s["mass"], n_leaf=case["n_leaf"], out=s["out"], **s["kw"])
    if case["entry"] == "forest":
        s["tree"].rebuild(s["pos"], s["mass"], offsets=s["offsets"])
        return s["tree"].evaluate_forest(s["thetas"], out=s["out"], **s["kw"])
    s["tree"].rebuild(s["pos"], s["mass"])
    f = s["tree"].evaluate(out=s["out"], **s["kw"])
    return {"force": f, "pot": s["pot"]} if case.get("potential") else f


def work(case):
    """One read of the particles and one write of the results; the pair
    operations of near and far lists, whose lengths follow from the opening
    angle (a leaf is near what lies within about 1 / theta of its size)."""
    n, th = int(case["n"]), float(case["theta"])
    steps = int(case.get("steps", 1))
    size = n / case["sets"] if case["entry"] == "forest" else n
    leaf = 0.4 * case["n_leaf"]
    around = (1.0 + 2.0 / th) ** 3
    near = 20.0 * n * min(size, around * leaf)
    order = max(case["p"], case.get("scalar_degree", 0) + 1 if case.get("scalar_degree") else 0)
    far = PAIR_FLOPS[case["variant"]][order] * (1.2 * n / leaf) * min(1.2 * size / leaf, 2.5 * around)
    words = 7 + (1 if case.get("potential") else 0) + (6 if case["entry"] == "session" else 0)
    return {"bytes": 8.0 * words * n * steps, "flops": (near + far) * steps}


# ---- the direct sum -----------------------------------------------------------

def _direct(pos, mass, want_pot=False):
    """Softened direct forces (and potential) in double precision."""
    n = pos.shape[0]
    f = torch.empty_like(pos)
    pot = torch.empty_like(mass)
    rows = max(1, min(n, (1 << 26) // n))
    x = pos.t().contiguous()
    for a in range(0, n, rows):
        b = min(n, a + rows)
        d = [x[k][None, :] - x[k][a:b, None] for k in range(3)]
        r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + EPS * EPS
        ri = r2.rsqrt()
        w = mass[None, :] * ri
        if want_pot:
            pot[a:b] = mass[a:b] / EPS - w.sum(1)
        w = w * ri * ri
        for k in range(3):
            f[a:b, k] = (w * d[k]).sum(1)
    return f * mass[:, None], pot


def exact(case, seed):
    """The same outputs from the direct sum over all pairs (for sets small enough)."""
    if int(case["n"]) > EXACT_MAX_N or int(case["n"]) * int(case.get("steps", 1)) > 4 * EXACT_MAX_N:
        return None
    pos, mass, vel = _inputs(case, seed)
    if case["entry"] == "forest":
        off = _offsets(case)
        return torch.cat([_direct(pos[a:b].contiguous(), mass[a:b])[0] for a, b in zip(off, off[1:])])
    if case["entry"] == "session":
        f = _direct(pos, mass)[0]
        for _ in range(int(case["steps"])):
            vel = vel + f / mass[:, None] * (0.5 * DT)
            pos = pos + vel * DT
            f = _direct(pos, mass)[0]
            vel = vel + f / mass[:, None] * (0.5 * DT)
        return {"pos": pos, "vel": vel, "force": f}
    f, pot = _direct(pos, mass, bool(case.get("potential")))
    return {"force": f, "pot": pot} if case.get("potential") else f
