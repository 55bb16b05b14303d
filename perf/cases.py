"""Performance cases: the calls that programs built on this package make.

A program here advances batches of micro-domains (``Micro.step``,
``Micro.step_subset``), the macro solver (``Sph.step``), both together
(``Coupled.step``, ``Hybrid.step``), and evaluates or trains the stress
surrogate (``Surrogate.forward``, ``Surrogate.train_step``).  ``listed``
names twelve such workloads from the smallest call to the benchmark's batch,
``draw`` makes more of the same ranges, ``prepare`` builds what a program
holds before the call, ``run`` makes the call, ``work`` states what it cannot
do without, and ``exact`` recomputes its outputs in double precision from the
equations alone.

Micro-domains start from a jittered lattice (chains as random walks through
it) with Maxwell velocities, every number representable in single precision.
"""
import math
import os

import numpy as np
import torch

from paper_2512_13267_amd import lhmm, micro, surrogate

N_IN, HIST = 129, 32  # surrogate features: 32 gradient samples of 4 components, and the polymer fraction
EXACT_MOST = 1.0e9  # ordered pair updates beyond which exact() would take too long


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def _micro(**over):
    """Micro-domains; subset: how many of the boxes are advanced (0: all); rate: simple shear, or the range of random
    in-plane gradients when random_grad; restart: each pass starts from the snapshot, as replays do."""
    c = dict(kind="micro", n_boxes=1, edge_lo=10.0, edge_hi=10.0, planar=False, afbc=False, chain_len=10, phi=0.1,
             random_grad=False, rate=0.1, steps=20, subset=0, restart=False, fp64=False, components=False,
             graphs=True, state=False)
    c.update(over)
    return c


def listed():
    return [
        # the parity and rheometry unit: one 3000-particle box in simple shear, advanced and written to a checkpoint
        dict(_micro(state=True), name="one box"),
        # verification runs are made in double precision: three small boxes of odd sizes, 25 steps (the smoke run)
        dict(_micro(n_boxes=3, edge_lo=4.2, edge_hi=6.3, phi=0.2, random_grad=True, rate=0.3, steps=25, fp64=True,
                    restart=True, state=True), name="three boxes fp64"),
        # the surrogate's fallback: a few micro-domains of many are restored and relive their gradient history
        dict(_micro(n_boxes=96, edge_lo=11.006, edge_hi=11.006, random_grad=True, rate=0.3, steps=50, subset=5,
                    restart=True), name="replay of 5 boxes"),
        # rheometry of the planar melt in its micro-domain with boundary regions
        dict(_micro(n_boxes=8, edge_lo=76.0, edge_hi=76.0, planar=True, afbc=True, chain_len=8, phi=1.0, rate=0.05,
                    steps=20), name="planar melt, boundary regions"),
        # stress by force type (kept by the engine when asked) of a middle-sized batch
        dict(_micro(n_boxes=40, edge_lo=8.0, edge_hi=14.0, phi=0.2, random_grad=True, rate=0.5, steps=20,
                    components=True, restart=True), name="stress components"),
        # the benchmark's batch: 256 boxes of 1.5k to 12k particles under their own gradients
        dict(_micro(n_boxes=256, edge_lo=8.0, edge_hi=16.0, phi=0.2, random_grad=True, rate=0.5, steps=20,
                    restart=True), name="batch of 256"),
        # macro solver alone: one exchange interval of 8 steps on the cylinder array with wall particles
        dict(kind="sph", nx=64, ny=64, cylinder=True, lucy=False, steps=8, stress=True, name="macro steps, cylinders"),
        # the coupled reverse-Poiseuille run with plain micro-DPD: one exchange interval
        dict(kind="couple", nx=16, ny=64, lucy=False, particles=4000, planar=False, m_bar=1, k_micro=50,
             name="coupled interval"),
        # the macro step with the surrogate in the loop while its gate stays quiet (most steps are)
        dict(kind="hybrid", n=64, particles=500, steps=4, name="surrogate in the loop"),
        # the ensemble's in-loop inference for every mobile particle of the cylinder array
        dict(kind="forward", rows=3572, members=5, hidden=256, static=False, name="forward 3572 rows"),
        # the smallest inference: a coarse macro lattice, odd row count
        dict(kind="forward", rows=217, members=5, hidden=256, static=True, name="forward 217 rows"),
        # training: a stretch of Adam steps at the training configuration, then the weights are read
        dict(kind="train", rows=4096, members=5, hidden=256, steps=24, name="training steps"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["one", "fp64", "replay", "melt", "batch", "batch", "sph", "couple", "hybrid", "forward",
                       "forward", "train"])
    edge = round(rng.uniform(4.3, 14.0), 3)
    if kind == "one":
        return _micro(n_boxes=rng.randint(1, 4), edge_lo=edge, edge_hi=edge, phi=round(rng.uniform(0.0, 0.3), 3),
                      rate=round(rng.uniform(0.01, 0.3), 4), steps=rng.randint(10, 40), state=True)
    if kind == "fp64":
        return _micro(n_boxes=rng.randint(1, 8), edge_lo=round(rng.uniform(4.2, 6.0), 3),
                      edge_hi=round(rng.uniform(6.0, 10.0), 3), phi=round(rng.uniform(0.0, 0.3), 3), random_grad=True,
                      rate=0.3, steps=rng.randint(10, 30), fp64=True, restart=True, state=True,
                      graphs=rng.random() < 0.5)
    if kind == "replay":
        n = rng.randint(16, 96)
        e = round(rng.uniform(8.0, 12.0), 3)
        return _micro(n_boxes=n, edge_lo=e, edge_hi=e, random_grad=True, rate=0.3, steps=rng.randint(20, 50),
                      subset=max(1, int(_log(rng, 1.0, n))), restart=True)
    if kind == "melt":
        af = rng.random() < 0.5
        e = round(rng.uniform(20.0, 76.0), 3)
        return _micro(n_boxes=rng.randint(2, 16), edge_lo=e, edge_hi=e, planar=True, afbc=af,
                      chain_len=rng.choice([4, 8, 16, 32]), phi=1.0, rate=round(rng.uniform(0.01, 0.5), 4),
                      steps=rng.randint(10, 30))
    if kind == "batch":
        return _micro(n_boxes=int(_log(rng, 12.0, 256.0)), edge_lo=round(rng.uniform(6.0, 9.0), 3),
                      edge_hi=round(rng.uniform(9.0, 16.0), 3), phi=round(rng.uniform(0.1, 0.3), 3), random_grad=True,
                      rate=0.5, steps=rng.randint(10, 20), restart=True, components=rng.random() < 0.25)
    if kind == "sph":
        cyl, lucy = rng.random() < 0.5, rng.random() < 0.3
        nx = rng.randint(20, 72)
        return dict(kind="sph", nx=nx, ny=nx if cyl else rng.randint(20, 72), cylinder=cyl, lucy=lucy,
                    steps=rng.randint(1, 8), stress=rng.random() < 0.5)
    if kind == "couple":
        lucy = rng.random() < 0.5
        return dict(kind="couple", nx=rng.randint(12, 20), ny=rng.randint(14, 40), lucy=lucy,
                    particles=int(_log(rng, 300.0, 4000.0)), planar=rng.random() < 0.3,
                    m_bar=rng.choice([1, 2, 8]), k_micro=rng.randint(10, 50))
    if kind == "hybrid":
        return dict(kind="hybrid", n=rng.randint(24, 64), particles=rng.randint(220, 600), steps=rng.randint(1, 6))
    if kind == "forward":
        rows, members, hidden = int(_log(rng, 20.0, 5000.0)), rng.choice([3, 5, 5, 8]), rng.choice([64, 128, 256, 256])
        fits = rows * (members * (4 * hidden + 128) + 320) < 30 << 20  # the static entry point's scratch
        return dict(kind="forward", rows=rows, members=members, hidden=hidden, static=fits and rng.random() < 0.25)
    return dict(kind="train", rows=int(_log(rng, 200.0, 4096.0)), members=rng.choice([3, 5, 5]),
                hidden=rng.choice([64, 128, 256, 256]), steps=rng.randint(8, 24))


# ---------------------------------------------------------------------------
# inputs, the same for prepare and exact
# ---------------------------------------------------------------------------

SOLVENT = dict(a=25.0, gamma=4.5, sigma=3.0, kBT=1.0, mass=1.0, rc=1.0, dt=0.01, H=30.0, R0=1.5)
MELT = dict(a=25.0, gamma=4.5, sigma=3.0, kBT=1.0, mass=1.0, rc=1.0, dt=0.005, H=50.0, R0=1.5)
PLANAR_Z = 3.5  # z edge of a planar cell
DEV = "cuda"


def _fluid(rng, h, n_boxes, n, n_chains, chain_len, planar):
    """n_boxes boxes of n particles in the cell h: fractional coordinates and velocities, (n_boxes, n, 3) float32."""
    dims = 2 if planar else 3
    ext = np.linalg.norm(h, axis=0)[:dims]
    per = (n / np.prod(ext)) ** (1.0 / dims)
    m = np.maximum(np.floor(ext * per).astype(int), 1)
    while np.prod(m) < n:
        m[np.argmin(m / ext)] += 1
    sites = np.stack(np.meshgrid(*[np.arange(k) for k in m], indexing="ij"), -1).reshape(-1, dims)
    sites = sites[rng.permutation(len(sites))[:n]]
    s = np.zeros((n_boxes, n, 3), dtype=np.float32)
    s[..., :dims] = (sites + 0.2 + 0.6 * rng.random((n_boxes, n, dims), dtype=np.float32)) / m
    if n_chains:
        u = rng.standard_normal((n_boxes, n_chains, chain_len - 1, 3), dtype=np.float32)
        if planar:
            u[..., 2] = 0.0
        u *= 0.9 / np.linalg.norm(u, axis=-1, keepdims=True)
        walk = np.concatenate([np.zeros_like(u[:, :, :1]), np.cumsum(u, axis=2)], axis=2) @ np.linalg.inv(h).T
        nb = n_chains * chain_len
        s[:, :nb] = (s[:, 0:nb:chain_len][:, :, None] + walk).reshape(n_boxes, nb, 3)
    s -= np.floor(s)
    s[s >= 1.0] = 0.0
    c = rng.standard_normal((n_boxes, n, 3), dtype=np.float32)
    if planar:
        c[..., 2] = 0.0
    c -= c.mean(axis=1, keepdims=True)
    return s, c


def _boxes(case, seed):
    """The micro-domains of a "micro" case: parameters, sizes (n, chains), cells, state, gradients, advanced boxes."""
    rng = np.random.default_rng([seed, 1])
    shape = np.random.default_rng([case["n_boxes"], int(1000 * case["edge_hi"])])  # sizes go by the case alone
    planar, nb = case["planar"], case["n_boxes"]
    p = dict(MELT if planar else SOLVENT, chain_len=case["chain_len"], seed=int(rng.integers(1 << 62)))
    density = 4.0 if planar else 3.0
    sizes, hs, ss, cs = [], [], [], []
    for _ in range(nb):
        e = float(shape.uniform(case["edge_lo"], case["edge_hi"])) if case["edge_hi"] > case["edge_lo"] else case["edge_lo"]
        h = np.diag([e, e, PLANAR_Z if planar else e])
        if case["random_grad"] and not case["afbc"]:
            h[0, 1] = e * rng.uniform(-0.45, 0.45)  # a phase of the sheared lattice (det = e^3)
        n = int(round(density * e ** (2 if planar else 3)))
        n_ch = int(round(case["phi"] * n / p["chain_len"])) if not planar else int(case["phi"] * n) // p["chain_len"]
        s, c = _fluid(rng, h, 1, n, n_ch, p["chain_len"], planar)
        sizes.append((n, n_ch))
        hs.append(h)
        ss.append(s[0])
        cs.append(c[0])
    L = np.zeros((nb, 3, 3))
    if case["random_grad"]:
        g = rng.uniform(-case["rate"], case["rate"], size=(nb, 3))
        L[:, 0, 0], L[:, 0, 1], L[:, 1, 0], L[:, 1, 1] = g[:, 0], g[:, 1], g[:, 2], -g[:, 0]
    else:
        L[:, 0, 1] = case["rate"]
    sel = np.arange(nb)
    if case["subset"]:
        sel = np.sort(rng.permutation(nb)[:case["subset"]])
    regions = np.tile([case["edge_lo"] * 12.0 / 76.0, case["edge_lo"] * 25.0 / 76.0], (nb, 1)) if case["afbc"] else None
    return p, sizes, np.stack(hs), np.concatenate(ss), np.concatenate(cs), L, sel.astype(np.int32), regions


def _macro(case, seed):
    """SPH parameters, positions, velocities and micro stresses of a macro problem."""
    rng = np.random.default_rng([seed, 2])
    nx, ny = (case["n"], case["n"]) if case["kind"] == "hybrid" else (case["nx"], case["ny"])
    lucy = case.get("lucy", False)
    cyl = case["kind"] == "hybrid" or case.get("cylinder", False)
    dh = 1.0 / nx if cyl else 2.0 / ny
    xs, ys = np.meshgrid((np.arange(nx) + 0.5) * dh, (np.arange(ny) + 0.5) * dh, indexing="ij")
    r = np.stack([xs.ravel(), ys.ravel()], axis=1)
    n_fixed, Lx, Ly = 0, nx * dh, ny * dh
    if cyl:
        inside = np.hypot(r[:, 0] - 0.5, r[:, 1] - 0.5) < 0.2
        r = np.concatenate([r[~inside], r[inside]])
        n_fixed = int(inside.sum())
    nm = len(r) - n_fixed
    r[:nm] += rng.uniform(-0.1, 0.1, size=(nm, 2)) * dh
    r[:nm] -= np.floor(r[:nm] / [Lx, Ly]) * [Lx, Ly]
    v = np.zeros_like(r)
    ph = rng.uniform(0.0, 2.0 * math.pi, size=4)
    v[:nm, 0] = 0.05 * np.sin(2 * math.pi * r[:nm, 1] / Ly + ph[0]) + 0.02 * np.sin(2 * math.pi * r[:nm, 0] / Lx + ph[1])
    v[:nm, 1] = 0.03 * np.sin(2 * math.pi * r[:nm, 0] / Lx + ph[2]) + 0.02 * np.cos(2 * math.pi * r[:nm, 1] / Ly + ph[3])
    F = 1.0 if cyl else 0.2
    gap = 0.6 if cyl else 1.0
    vmax = F * gap * gap / 1.6
    length = 0.2 if cyl else 1.0
    c = max(10.0 * vmax, math.sqrt(2.0 * vmax / length), math.sqrt(10.0 * F * length))
    q = dict(rho0=1.0, eta=0.1, zeta=0.0, c=c, theta=0.5, F=F, h=(4.0 if lucy else 3.0) * dh, dt=1e-3,
             mass=dh * dh, Lx=Lx, Ly=Ly, lambda_star=0.2, alpha=0.07, n_fixed=n_fixed, force_mode=1 if cyl else 0,
             kernel=1 if lucy else 0, micro_dim=2 if case.get("planar") else 3)
    sigma = None
    if case.get("stress"):
        sigma = np.zeros((len(r), 6))
        sigma[:nm] = 0.3 * rng.standard_normal((nm, 6)) - np.array([20.0, 20.0, 20.0, 0.0, 0.0, 0.0])
    return q, r, v, sigma


def _domains(case, seed, n_boxes):
    """One micro-domain per mobile macro particle."""
    rng = np.random.default_rng([seed, 3])
    planar, n = case.get("planar", False), case["particles"]
    p = dict(MELT if planar else SOLVENT, chain_len=8 if planar else 10, seed=int(rng.integers(1 << 62)))
    e = (n / 4.0) ** 0.5 if planar else (n / 3.0) ** (1.0 / 3.0)
    h = np.diag([e, e, PLANAR_Z if planar else e])
    n_ch = n // 8 if planar else int(round(0.1 * n / 10))
    s, c = _fluid(rng, h, n_boxes, n, n_ch, p["chain_len"], planar)
    return p, (n, n_ch), h, s.reshape(-1, 3), c.reshape(-1, 3)


def _members(case, seed):
    """Weights of the ensemble, in float32 values (float64 arrays)."""
    rng = np.random.default_rng([seed, 4])
    nh, out = case["hidden"], []
    for _ in range(case["members"]):
        w = {"W1": rng.normal(scale=math.sqrt(2.0 / N_IN), size=(N_IN, nh)), "b1": rng.normal(scale=0.1, size=nh),
             "W2": rng.normal(scale=math.sqrt(2.0 / nh), size=(nh, nh)), "b2": rng.normal(scale=0.1, size=nh),
             "W3": rng.normal(scale=math.sqrt(1.0 / nh), size=(nh, 3)), "b3": rng.normal(scale=0.1, size=3)}
        out.append({k: x.astype(np.float32).astype(np.float64) for k, x in w.items()})
    return out


def _rows(case, seed):
    """Feature rows (gradient histories, correlated in time, and a polymer fraction) and stress targets, float32."""
    steps = case.get("steps", 1)
    g = torch.Generator(device="cpu").manual_seed(seed * 7 + 5)
    n = case["rows"] * steps
    x = torch.empty((n, N_IN))
    z = torch.randn((n, 4), generator=g)
    noise = torch.randn((HIST, n, 4), generator=g)
    for k in range(HIST):
        z = 0.9 * z + math.sqrt(1.0 - 0.81) * noise[k]
        x[:, 4 * k:4 * k + 4] = z
    x[:, N_IN - 1] = torch.rand(n, generator=g) * 2.0 - 1.0
    t = 0.5 * z[:, :3] + 0.3 * torch.randn((n, 3), generator=g)
    return x, t


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------

def _engine(p, specs, s, c, fp64=False, components=False, graphs=True):
    m = micro.Micro(p, specs, precision="fp64" if fp64 else "fp32", graphs=graphs, components=components)
    m.set_state(s, c, None, 0)
    return m


def prepare(case, seed):
    st = {"case": case}
    kind = case["kind"]
    if kind == "micro":
        p, sizes, hs, s, c, L, sel, regions = _boxes(case, seed)
        m = micro.Micro(p, [(n, k, h) for (n, k), h in zip(sizes, hs)],
                        precision="fp64" if case["fp64"] else "fp32", graphs=case["graphs"],
                        components=case["components"])
        if regions is not None:
            m.set_afbc(regions)
        m.set_state(s, c, None, 0)
        if case["restart"]:
            m.snapshot()
        if not case["subset"]:
            m.prepare(case["steps"])
        st.update(m=m, sel=sel, G=torch.from_numpy(L.reshape(-1, 9)).to(DEV),
                  out=torch.empty((len(sizes), 6), dtype=torch.float64, device=DEV))
    elif kind in ("sph", "couple", "hybrid"):
        q, r, v, sigma = _macro(case, seed)
        st["sph"] = lhmm.Sph(q, r, v)
        n, nm = len(r), len(r) - q["n_fixed"]
        if kind == "sph":
            st["sigma"] = None if sigma is None else torch.from_numpy(sigma).to(DEV)
            st["gradL"] = torch.empty((n, 9), dtype=torch.float64, device=DEV)
            return st
        p, (k, n_ch), h, s, c = _domains(case, seed, nm)
        st["m"] = _engine(p, [(k, n_ch, h)] * nm, s, c)
        if kind == "couple":
            st["m"].prepare(case["k_micro"])
            st["cp"] = lhmm.Coupled(st["sph"], st["m"])
        else:
            members, nh, gs, ss = surrogate.load_trained()
            sur = surrogate.Surrogate(members, N_IN, nh, 3, max_batch=nm)
            # a threshold at which no particle falls back to its micro-domain
            st["hy"] = lhmm.Hybrid(st["sph"], st["m"], sur, phi=np.full(nm, -1.0, dtype=np.float32), k_micro=50, hold=10,
                                   replay=10, threshold=50.0, floor=1.0, grad_scale=gs, stress_scale=ss)
    else:
        members = _members(case, seed)
        x, t = _rows(case, seed)
        rows = case["rows"]
        st["sur"] = surrogate.Surrogate(members, N_IN, case["hidden"], 3, max_batch=rows)
        if kind == "forward":
            st["x"] = x.to(DEV)
            st["y"] = torch.empty((case["members"], rows, 3), dtype=torch.float32, device=DEV)
        else:
            st["x"] = [b.contiguous().to(DEV) for b in x.split(rows)]
            st["t"] = [b.contiguous().to(DEV) for b in t.split(rows)]
            st["loss"] = torch.zeros(case["members"], dtype=torch.float32, device=DEV)
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "micro":
        m, out = state["m"], state["out"]
        if case["restart"]:
            m.restore(state["sel"])
        if case["subset"]:
            m.step_subset(state["G"], case["steps"], state["sel"], out=out)
        else:
            m.step(state["G"], case["steps"], out=out)
        got = {"stress": out}
        if case["components"]:
            got["parts"] = m.components()
        if case["state"]:
            s, c, h, _ = m.get_state()
            got.update(s=s, c=c, h=h)
        return got
    if kind == "sph":
        for k in range(case["steps"]):
            state["sph"].step(state["sigma"], state["gradL"] if k + 1 == case["steps"] else None)
        return state["gradL"]
    if kind == "couple":
        state["cp"].step(case["k_micro"], m_bar=case["m_bar"])
        sigma, grad = state["cp"].coupling_state()
        return {"sigma": sigma, "grad": grad}
    if kind == "hybrid":
        for _ in range(case["steps"]):
            state["hy"].step()
        sigma, on = state["hy"].state()
        return {"sigma": sigma, "on": on.astype(np.int64)}
    sur = state["sur"]
    if kind == "forward":
        return sur.forward_static(state["x"], state["y"]) if case["static"] else sur.forward(state["x"], out=state["y"])
    for x, t in zip(state["x"], state["t"]):
        sur.train_step(x, t, 3e-4, state["loss"])
    return {"loss": state["loss"], "weights": sur.get_weights()}


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------

NEIGHBOURS = 4.0 / 3.0 * math.pi * 3.0  # within the cutoff; 4 pi in the planar melt is the same number
PAIR_FLOPS = 73.0  # FP32 operations of one unordered pair, the random integers not counted


def _micro_work(n, steps, boxes, real):
    # positions, velocities and forces in and out once, gradients in, stresses out
    return {"bytes": 18.0 * n * real + 120.0 * boxes, "flops": steps * n * (0.5 * NEIGHBOURS * PAIR_FLOPS + 40.0)}


def _sph_work(n, steps, lucy):
    near = math.pi * (16.0 if lucy else 9.0)
    # per step two density and two force sums and, at the end, the gradients; state and stresses in and out once
    return {"bytes": n * (8.0 * 8 + 48.0 + 72.0), "flops": n * near * (steps * 2.0 * (25.0 + 70.0) + 45.0)}


def _mlp_flops(case, rows):
    return 2.0 * case["members"] * rows * (N_IN * case["hidden"] + case["hidden"] ** 2 + 3 * case["hidden"])


def work(case):
    kind = case["kind"]
    if kind == "micro":
        nb = case["subset"] or case["n_boxes"]
        lo, hi = case["edge_lo"], case["edge_hi"]
        dims, density = (2, 4.0) if case["planar"] else (3, 3.0)
        mean = sum((lo + (hi - lo) * (k + 0.5) / 16) ** dims for k in range(16)) / 16
        return _micro_work(nb * density * mean, case["steps"], nb, 8.0 if case["fp64"] else 4.0)
    if kind == "sph":
        return _sph_work(case["nx"] * case["ny"], case["steps"], case["lucy"])
    if kind == "couple":
        n = case["nx"] * case["ny"]
        a, b = _micro_work(n * case["particles"], case["k_micro"], n, 4.0), _sph_work(n, case["m_bar"], case["lucy"])
        return {k: a[k] + b[k] for k in a}
    if kind == "hybrid":
        n = case["n"] ** 2
        nm = n * (1.0 - math.pi * 0.04)
        net = dict(members=5, hidden=256)
        a, b = _sph_work(n, case["steps"], False), _mlp_flops(net, nm)
        return {"bytes": a["bytes"] + case["steps"] * (nm * 4 * N_IN + 2.0e6), "flops": a["flops"] + case["steps"] * b}
    weights = case["members"] * (N_IN * case["hidden"] + case["hidden"] ** 2 + 5 * case["hidden"])
    rows = case["rows"]
    if kind == "forward":
        return {"bytes": rows * (4.0 * N_IN + 12.0 * case["members"]) + 2.0 * weights, "flops": _mlp_flops(case, rows)}
    # forward, input gradients of two layers and weight gradients; Adam reads and writes three words a weight
    return {"bytes": case["steps"] * (rows * 4.0 * (N_IN + 3) + 28.0 * weights),
            "flops": case["steps"] * (3.0 * _mlp_flops(case, rows) - 2.0 * case["members"] * rows * N_IN * case["hidden"])}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _philox(x, k0, k1):
    """Philox4x32-10 of the counters x (four int64 tensors of 32-bit words)."""
    x0, x1, x2, x3 = x
    mask = 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = 0xD2511F53 * x0, 0xCD9E8D57 * x2  # the low 64 bits
        x0, x1, x2, x3 = ((p1 >> 32) & mask) ^ x1 ^ k0, p1 & mask, ((p0 >> 32) & mask) ^ x3 ^ k1, p0 & mask
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return x0, x1


def _normals(x, key):
    w0, w1 = _philox(x, key & 0xFFFFFFFF, key >> 32)
    u0, u1 = ((w0 >> 9).double() + 0.5) * 2.0 ** -23, ((w1 >> 9).double() + 0.5) * 2.0 ** -23
    r = torch.sqrt(-2.0 * torch.log(u0))
    return r * torch.cos(2 * math.pi * u1), r * torch.sin(2 * math.pi * u1)


def _expm(L, t):
    a, k2 = 0.5 * (L[0, 0] - L[1, 1]), 0.25 * (L[0, 0] - L[1, 1]) ** 2 + L[0, 1] * L[1, 0]
    k = math.sqrt(abs(k2))
    f0, f1 = (math.cosh(k * t), math.sinh(k * t) / k) if k2 > 0 else (math.cos(k * t), math.sin(k * t) / k) if k2 < 0 else (1.0, t)
    E = np.eye(3) * f0
    E[2, 2] = 1.0
    E[0, 0] += f1 * a
    E[1, 1] -= f1 * a
    E[0, 1], E[1, 0] = f1 * L[0, 1], f1 * L[1, 0]
    return E


def _mat(M, x):
    return (M * x[:, None, :]).sum(-1)


def _reduce(h):
    """Lagrange-Gauss reduction of the in-plane columns: the new cell and U with h_new = h U."""
    h, U = h.copy(), np.eye(3)
    for _ in range(64):
        b1, b2 = h[:2, 0], h[:2, 1]
        if b2 @ b2 < b1 @ b1:
            T = np.array([[0.0, -1.0, 0.0], [1.0, 0.0, 0.0], [0.0, 0.0, 1.0]])
        else:
            m = math.floor((b1 @ b2) / (b1 @ b1) + 0.5)
            if m == 0:
                break
            T = np.array([[1.0, -m, 0.0], [0.0, 1.0, 0.0], [0.0, 0.0, 1.0]])
        h, U = h @ T, U @ T
    return h, U


class _Dpd:
    """Micro-domains advanced in double precision; the pairs of a skin-enlarged list are kept for a few steps."""

    SKIN, KEEP = 0.5, 7

    def __init__(self, p, sizes, hs, s, c, rng_ids, regions=None, zeta=10.0):
        self.p, self.nb = p, len(sizes)
        n = np.array([k for k, _ in sizes])
        self.off = torch.from_numpy(np.concatenate([[0], np.cumsum(n)]))
        T = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.float64, device=DEV)  # noqa: E731
        self.T = T
        self.s, self.c, self.h = T(s), T(c), [h.copy() for h in hs]
        self.box = torch.repeat_interleave(torch.arange(self.nb), torch.from_numpy(n)).to(DEV)
        self.rng = torch.from_numpy(np.asarray(rng_ids, dtype=np.int64)).to(DEV)[self.box]
        self.id = torch.arange(int(self.off[-1]), device=DEV) - self.off[:-1].to(DEV)[self.box]
        bonds = [int(self.off[b]) + np.arange(k * p["chain_len"]).reshape(k, -1)[:, :-1].ravel() for b, (_, k) in enumerate(sizes)]
        self.bi = torch.from_numpy(np.concatenate(bonds).astype(np.int64)).to(DEV)
        self.age, self.pairs = 10 ** 9, None
        self.step, self.f = 0, None
        self.L = np.zeros((self.nb, 3, 3))
        self.regions = regions
        if regions is not None:
            self.hc, self.hb = T(regions[:, 0])[self.box], T(regions[:, 1])[self.box]
            self.damp = math.exp(-0.5 * zeta * p["dt"])
            self.amp = math.sqrt(p["kBT"] / p["mass"] * (1.0 - math.exp(-zeta * p["dt"])))

    def _list(self):
        out = []
        cut2 = (self.p["rc"] + self.SKIN) ** 2
        for b in range(self.nb):
            o, e = int(self.off[b]), int(self.off[b + 1])
            s, h = self.s[o:e].float().T.contiguous(), self.h[b]
            rows = max(1, int(1.0e8 // (e - o)))
            for k in range(0, e - o, rows):
                x, y, z = (a[k:k + rows, None] - a[None, k:] for a in s)  # j >= k holds every j > i
                for a in (x, y, z):
                    a -= torch.round(a)
                r2 = (x * h[0, 0] + y * h[0, 1]).square_() + (x * h[1, 0] + y * h[1, 1]).square_() + (z * h[2, 2]).square_()
                ij = torch.nonzero(r2 < cut2) + k
                out.append(ij[ij[:, 0] < ij[:, 1]] + o)
        self.pairs, self.age = torch.cat(out).T.contiguous(), 0

    def _core(self, a, e, hc):
        """Share of the segments a + t e inside |x|, |y| <= hc."""
        t0, t1 = torch.zeros_like(hc), torch.ones_like(hc)
        for k in range(2):
            flat = e[:, k] == 0
            ek = torch.where(flat, torch.ones_like(hc), e[:, k])
            ta, tb = (-hc - a[:, k]) / ek, (hc - a[:, k]) / ek
            lo, hi = torch.minimum(ta, tb), torch.maximum(ta, tb)
            inside = a[:, k].abs() <= hc
            t0 = torch.maximum(t0, torch.where(flat, torch.where(inside, 0.0, 2.0), lo))
            t1 = torch.minimum(t1, torch.where(flat, torch.where(inside, 1.0, -1.0), hi))
        return (t1 - t0).clamp(min=0.0)

    def _centred(self, s):
        H = self.T(np.stack(self.h))[self.box]
        return _mat(H[:, :2, :2], s[:, :2] - 0.5)

    def _per_box(self, x):
        """Sums of a per-particle array over each box."""
        run = torch.cat([torch.zeros_like(x[:1]), torch.cumsum(x, 0)])[self.off]
        return run[1:] - run[:-1]

    def _sum(self, i, d, g):
        """Per box, the sums of d (x) g over rows that belong to the particles i."""
        w = torch.stack([d[:, 0] * g[:, 0], d[:, 1] * g[:, 1], d[:, 2] * g[:, 2], d[:, 0] * g[:, 1], d[:, 0] * g[:, 2],
                         d[:, 1] * g[:, 2]], -1)
        return self._per_box(torch.zeros((len(self.s), 6), dtype=torch.float64, device=DEV).index_add_(0, i, w))

    def forces(self, counter):
        p = self.p
        if self.age >= self.KEEP:
            self._list()
        self.age += 1
        H, Lt = self.T(np.stack(self.h)), self.T(self.L)
        i, j = self.pairs
        ds = self.s[i] - self.s[j]
        d = _mat(H[self.box[i]], ds - torch.round(ds))
        near = ((d * d).sum(-1) < p["rc"] ** 2).nonzero()[:, 0]
        i, j, d = i[near], j[near], d[near]
        b = self.box[i]
        r = d.norm(dim=-1)
        e = d / r[:, None]
        w = 1.0 - r / p["rc"]
        v = self.c[i] - self.c[j] + _mat(Lt[b], d)
        ev = (e * v).sum(-1)
        one = torch.ones_like(self.id[i])
        th, _ = _normals((torch.minimum(self.id[i], self.id[j]), torch.maximum(self.id[i], self.id[j]), one * counter, self.rng[i]), p["seed"])
        parts = [w * p["a"], -p["gamma"] * w * w * ev, w * p["sigma"] / math.sqrt(p["dt"]) * th]
        g = sum(parts)[:, None] * e
        f = torch.zeros_like(self.s).index_add_(0, i, g).index_add_(0, j, -g)
        wd = d
        if self.regions is not None:
            x = self._centred(self.s)
            wd = d * self._core(x[i], -d[:, :2], self.hc[i])[:, None]
        self.vir_parts = [self._sum(i, wd, q[:, None] * e) for q in parts]
        k = self.bi
        ds = self.s[k] - self.s[k + 1]
        d = _mat(H[self.box[k]], ds - torch.round(ds))
        g = -p["H"] * d / (1.0 - (d * d).sum(-1) / p["R0"] ** 2).clamp(min=0.01)[:, None]
        f.index_add_(0, k, g).index_add_(0, k + 1, -g)
        wd = d
        if self.regions is not None:
            wd = d * self._core(x[k], -d[:, :2], self.hc[k])[:, None]
        self.fene = self._sum(k, wd, g)
        self.f = f

    def _ring(self, half):
        if self.regions is None:
            return
        x = self._centred(self.s)
        far = x.abs().max(dim=-1).values
        ring = ((far >= self.hc) & (far < self.hb)).nonzero()[:, 0]
        one = torch.ones_like(ring)
        n0, n1 = _normals((self.id[ring], one * (0xFFFFFFF0 + half), one * self.step, self.rng[ring]), self.p["seed"])
        u = _mat(self.T(self.G)[self.box[ring]][:, :2, :2], x[ring])
        self.c[ring, :2] = u + (self.c[ring, :2] - u) * self.damp + self.amp * torch.stack([n0, n1], -1)

    def begin(self, L):
        """A call under the gradients L: zero mean velocities; first forces if there are none."""
        if self.regions is not None:
            self.G, L = L, np.zeros_like(L)
        self.L = L
        self.c -= (self._per_box(self.c) / self.off.diff().to(DEV)[:, None])[self.box]
        if self.f is None:
            self.forces(self.step)

    def advance(self, L, steps):
        """Mean stresses over the steps: (kinetic, conservative, dissipative, random, FENE), (n_boxes, 5, 6)."""
        self.begin(L)
        p = self.p
        dt, m = p["dt"], p["mass"]
        Lb = self.T(self.L)[self.box]
        acc = 0.0
        kick = lambda: 0.5 * dt * (self.f / m - _mat(Lb, self.c))  # noqa: E731
        for _ in range(steps):
            self.step += 1
            hmi, U = [], []
            for b in range(self.nb):
                hmi.append(np.linalg.inv(_expm(self.L[b], 0.5 * dt) @ self.h[b]))
                self.h[b], u = _reduce(_expm(self.L[b], dt) @ self.h[b])
                U.append(np.linalg.inv(u))
            self.c += kick()
            self._ring(0)
            s = self.s + dt * _mat(self.T(np.stack(hmi))[self.box], self.c)
            s = _mat(self.T(np.stack(U))[self.box], s)
            self.s = s - torch.floor(s)
            self.forces(self.step)
            self.c += kick()
            self._ring(1)
            c, keep = self.c, torch.arange(len(self.s), device=DEV)
            vol = [np.linalg.det(h) for h in self.h]
            if self.regions is not None:
                x = self._centred(self.s)
                keep = (x.abs().max(dim=-1).values < self.hc).nonzero()[:, 0]
                c = self.c.clone()
                c[:, :2] -= _mat(self.T(self.G)[self.box][:, :2, :2], x)
                vol = [4.0 * self.regions[b, 0] ** 2 * self.h[b][2, 2] for b in range(self.nb)]
            kin = m * self._sum(keep, c[keep], c[keep])
            acc = acc - torch.stack([kin, *self.vir_parts, self.fene], 1) / self.T(vol)[:, None, None]
        return acc / steps


def _exact_micro(case, seed):
    p, sizes, hs, s, c, L, sel, regions = _boxes(case, seed)
    n_all = len(sizes)
    sel = sel.astype(np.int64)
    off = np.concatenate([[0], np.cumsum([n for n, _ in sizes])])
    pick = np.concatenate([np.arange(off[b], off[b + 1]) for b in sel])
    if len(pick) * case["steps"] * NEIGHBOURS > EXACT_MOST:
        return None
    d = _Dpd(p, [sizes[b] for b in sel], hs[sel], s[pick].astype(np.float64), c[pick].astype(np.float64), sel,
             None if regions is None else regions[sel])
    if case["restart"]:  # the snapshot's forces were taken at rest
        d.forces(0)
    parts = d.advance(L[sel], case["steps"])
    stress = torch.zeros((n_all, 6), dtype=torch.float64, device=DEV)
    stress[torch.from_numpy(sel).to(DEV)] = parts.sum(1)
    got = {"stress": stress}
    if case["components"]:
        got["parts"] = parts.cpu().numpy()
    if case["state"]:
        got.update(s=d.s.cpu().numpy(), c=d.c.cpu().numpy(), h=np.stack(d.h))
    return got


class _Macro:
    """The macro solver in double precision, all pairs."""

    def __init__(self, q, r, v):
        self.q = q
        T = lambda a: torch.as_tensor(a, dtype=torch.float64, device=DEV)  # noqa: E731
        self.r, self.v = T(r), T(v)
        self.n, self.nm = len(r), len(r) - q["n_fixed"]
        self.L = T([q["Lx"], q["Ly"]])

    def _pairs(self):
        d = self.r[:, None] - self.r[None]
        d = d - self.L * torch.round(d / self.L)
        rr = d.norm(dim=-1)
        i, j = (rr < self.q["h"]).nonzero().T
        return i, j, d[i, j], rr[i, j]

    def _kernel(self, r):
        h = self.q["h"]
        if self.q["kernel"] == 1:
            u = 1.0 - r / h
            return 5.0 / (math.pi * h * h) * (1.0 + 3.0 * r / h) * u ** 3, 60.0 / (math.pi * h ** 4) * u ** 2
        x, k = 3.0 * r / h, 63.0 / (478.0 * math.pi * h * h)
        t = [(b - x).clamp(min=0.0) for b in (3.0, 2.0, 1.0)]
        W = k * (t[0] ** 5 - 6.0 * t[1] ** 5 + 15.0 * t[2] ** 5)
        return W, k * 3.0 / h * (5.0 * t[0] ** 4 - 30.0 * t[1] ** 4 + 75.0 * t[2] ** 4) / r.clamp(min=1e-300)

    def _add(self, i, x):
        return torch.zeros((self.n,) + x.shape[1:], dtype=torch.float64, device=DEV).index_add_(0, i, x)

    def _state(self):
        i, j, d, r = self._pairs()
        W, F = self._kernel(r)
        dens = self._add(i, W)
        off = i != j
        return i[off], j[off], d[off], r[off], F[off], dens

    def _accel(self, pi):
        q = self.q
        i, j, d, r, F, dens = self._state()
        B = q["c"] ** 2 * q["rho0"] / 7.0
        pr = B * ((q["mass"] * dens / q["rho0"]) ** 7 - 1.0) + q["theta"] * B
        i2 = 1.0 / dens ** 2
        e, v = d / r[:, None], self.v[i] - self.v[j]
        f = ((pr * i2)[i] + (pr * i2)[j])[:, None] * F[:, None] * d
        av, bv = 2.0 * q["eta"] - q["zeta"], 4.0 * q["zeta"] + 2.0 * q["eta"]
        f = f - (av * v + bv * (v * e).sum(-1, keepdim=True) * e) * (F / (dens[i] * dens[j]))[:, None]
        if pi is not None:
            s = pi * i2[:, None, None]
            f = f - _mat(s[i] + s[j], d) * F[:, None]
        a = self._add(i, f) / q["mass"]
        sign = torch.ones_like(self.r[:, 1]) if q["force_mode"] == 1 else torch.where(self.r[:, 1] >= 0.5 * q["Ly"], 1.0, -1.0)
        a[:, 0] += q["F"] * sign
        a[self.nm:] = 0.0
        return a

    def step(self, sigma):
        q = self.q
        pi = None
        if sigma is not None:
            iso = (sigma[:, 0] + sigma[:, 1]) / 2 if q["micro_dim"] == 2 else sigma[:, :3].sum(1) / 3
            pi = torch.stack([sigma[:, 0] - iso, sigma[:, 3], sigma[:, 3], sigma[:, 1] - iso], -1).reshape(-1, 2, 2)
            pi = pi * (q["alpha"] / q["lambda_star"])
            pi[self.nm:] = 0.0
        self.v = self.v + 0.5 * q["dt"] * self._accel(pi)
        r = self.r[:self.nm] + q["dt"] * self.v[:self.nm]
        self.r = torch.cat([r - self.L * torch.floor(r / self.L), self.r[self.nm:]])
        self.v = self.v + 0.5 * q["dt"] * self._accel(pi)

    def gradients(self):
        i, j, d, _, F, dens = self._state()
        v = self.v[i] - self.v[j]
        G = self._add(i, (F / dens[j])[:, None, None] * d[:, :, None] * v[:, None, :])
        G = G - 0.5 * torch.diagonal(G, dim1=1, dim2=2).sum(-1)[:, None, None] * torch.eye(2, dtype=torch.float64, device=DEV)
        out = torch.zeros((self.n, 3, 3), dtype=torch.float64, device=DEV)
        out[:, :2, :2] = self.q["lambda_star"] * G.transpose(1, 2)
        out[self.nm:] = 0.0
        return out


def _mlp(w, x):
    gelu = lambda z: 0.5 * z * (1.0 + torch.erf(z / math.sqrt(2.0)))  # noqa: E731
    return gelu(gelu(x @ w["W1"] + w["b1"]) @ w["W2"] + w["b2"]) @ w["W3"] + w["b3"]


def _tensors(members):
    return [{k: torch.as_tensor(x, dtype=torch.float64, device=DEV) for k, x in w.items()} for w in members]


def _exact_hybrid(case, seed):
    q, r, v, _ = _macro(case, seed)
    path = os.path.join(os.path.dirname(surrogate.__file__), "weights", "surrogate_e5_h256.npz")
    z = np.load(path, allow_pickle=False)
    members = _tensors([{k: z["m%d_%s" % (e, k)] for k in ("W1", "b1", "W2", "b2", "W3", "b3")} for e in range(int(z["n_members"]))])
    mac = _Macro(q, r, v)
    sigma = torch.zeros((mac.n, 6), dtype=torch.float64, device=DEV)
    hist = torch.zeros((mac.nm, HIST, 4), dtype=torch.float64, device=DEV)
    for _ in range(case["steps"]):
        mac.step(sigma)
        g = mac.gradients()[:mac.nm, :2, :2].reshape(-1, 1, 4) * float(z["grad_scale"])
        hist = torch.cat([hist[:, 1:], g], 1)
        x = torch.cat([hist.reshape(mac.nm, -1), torch.full((mac.nm, 1), -1.0, dtype=torch.float64, device=DEV)], 1)
        y = sum(_mlp(w, x) for w in members) / len(members) * float(z["stress_scale"])
        sigma[:mac.nm, 0], sigma[:mac.nm, 1], sigma[:mac.nm, 3] = y[:, 0], y[:, 2], y[:, 1]
        sigma[:mac.nm, 2] = -(y[:, 0] + y[:, 2])
    return {"sigma": sigma.cpu().numpy(), "on": None}


def _exact_train(case, seed):
    members = _tensors(_members(case, seed))
    x, t = _rows(case, seed)
    loss, out = [], []
    for w in members:
        w = {k: a.requires_grad_(True) for k, a in w.items()}
        m, s = {k: torch.zeros_like(a) for k, a in w.items()}, {k: torch.zeros_like(a) for k, a in w.items()}
        for n, (xb, tb) in enumerate(zip(x.split(case["rows"]), t.split(case["rows"])), 1):
            e = ((_mlp(w, xb.double().to(DEV)) - tb.double().to(DEV)) ** 2).mean()
            grads = torch.autograd.grad(e, list(w.values()))
            with torch.no_grad():
                for (k, a), g in zip(w.items(), grads):
                    m[k].mul_(0.9).add_(0.1 * g)
                    s[k].mul_(0.999).add_(0.001 * g * g)
                    a -= 3e-4 * (m[k] / (1 - 0.9 ** n)) / (torch.sqrt(s[k] / (1 - 0.999 ** n)) + 1e-8)
        loss.append(e.detach())
        out.append({k: a.detach().cpu().numpy() for k, a in w.items()})
    return {"loss": torch.stack(loss), "weights": out}


def exact(case, seed):
    kind = case["kind"]
    if kind == "micro":
        return _exact_micro(case, seed)
    if kind == "hybrid":
        return _exact_hybrid(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "forward":
        x = _rows(case, seed)[0].double().to(DEV)
        return torch.stack([_mlp(w, x) for w in _tensors(_members(case, seed))])
    q, r, v, sigma = _macro(case, seed)
    mac = _Macro(q, r, v)
    if kind == "sph":
        sigma = None if sigma is None else torch.as_tensor(sigma, device=DEV)
        for _ in range(case["steps"]):
            mac.step(sigma)
        return mac.gradients().reshape(-1, 9)
    if mac.n * case["particles"] * case["k_micro"] * NEIGHBOURS > EXACT_MOST:
        return None
    for _ in range(case["m_bar"]):
        mac.step(torch.zeros((mac.n, 6), dtype=torch.float64, device=DEV))
    grad = mac.gradients().cpu().numpy()
    p, size, h, s, c = _domains(case, seed, mac.nm)
    d = _Dpd(p, [size] * mac.nm, [h] * mac.nm, s.astype(np.float64), c.astype(np.float64), np.arange(mac.nm))
    stress = d.advance(grad[:mac.nm], case["k_micro"]).sum(1)
    return {"sigma": stress.cpu().numpy(), "grad": grad}
