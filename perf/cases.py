"""Workloads that the library's speed is followed on.

Every case is what a program that uses the library does: it makes a case (or a
serving batch), gives it initial fields, advances it by some steps and reads
phi, P and u back, through the Python binding.  A pass is the advance and the
read-back; the case goes on from where the last pass left it.  The read-back is
the binding's FP64 arrays; where the case computes in FP32 a pass keeps its
snapshot in FP32, which holds those values exactly.

Sizes are the repository's own: its named workloads, its benchmark and its
serving stream's ranges (2D 128..1024, 3D 32..192 a side), or generic ragged
ones.  Inputs follow the same geometries, moved by the seed.
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch

from paper_2512_01027_amd import binding as B

STORE_BYTES = {"fp64": 8, "fp32": 4, "fp16": 2, "bf16": 2}


def _case(name, kind, nx, ny, nz, store, steps, q=None, collision="filter"):
    """One case: kind says geometry and boundaries, nz = 1 means 2D."""
    c = {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "store": store, "steps": steps,
         "q_hydro": (9 if nz == 1 else 27) if q is None else q, "collision": collision}
    return c if name is None else {"name": name, **c}


def listed():
    return [
        # the smallest call: the 2D static droplet in FP64 watched at short
        # intervals (4,096 nodes: launches and latency)
        _case("droplet_64sq_fp64", "droplet", 64, 64, 1, "fp64", 20),
        # the 2D rising bubble of the paper's Table I (walls on all sides)
        _case("table1_200x400_fp32", "table1", 200, 400, 1, "fp32", 500),
        # one request of the serving stream's small 3D end, run alone
        _case("bubble_48cube_fp16", "bubble", 48, 48, 48, "fp16", 300),
        # an odd-sized box with walls on every face in full precision (parity
        # and reference runs)
        _case("dam_101x53x45_fp64", "dam", 101, 53, 45, "fp64", 50),
        # BGK collision on an odd-sized periodic box
        _case("droplet_90x75x70_fp32_bgk", "droplet", 90, 75, 70, "fp32", 100, collision="bgk"),
        # the 128^3 translated droplet (the ordinary 3D run)
        _case("droplet_128cube_fp32", "droplet", 128, 128, 128, "fp32", 200),
        # a 3D rising bubble in BF16 storage
        _case("bubble_128cube_bf16", "bubble", 128, 128, 128, "bf16", 200),
        # a dam break against a block under an open top, ragged in every axis
        # (half the resolution of the 585 x 182 x 182 run)
        _case("block_293x91x91_fp16", "block", 293, 91, 91, "fp16", 200),
        # head-on droplet collision on the paper's D3Q19 lattice
        _case("collision_256x192x192_fp32", "collision", 256, 192, 192, "fp32", 150, q=19),
        # the benchmark's dam break, walls on all faces: the largest
        _case("dam_512x256x256_fp16", "dam", 512, 256, 256, "fp16", 200),
        # the serving batch: ten small requests of the stream's range (2D and
        # 3D, droplets and bubbles), admitted, advanced together and taken
        {"name": "serving_10_small_fp16", "kind": "serving", "store": "fp16", "requests": 10, "steps": 400,
         "largest_2d": 320, "largest_3d": 64},
    ]


def draw(rng):
    """A case of the same ranges: 4,096 to 8 M nodes (log-uniform), 2D or 3D,
    every storage precision, both 3D hydro lattices, both collisions."""
    if rng.random() < 0.12:
        return {"kind": "serving", "store": rng.choice(["fp16", "fp16", "fp32"]), "requests": rng.randint(4, 12),
                "steps": rng.randint(100, 500), "largest_2d": rng.randint(160, 400),
                "largest_3d": rng.randint(40, 80)}
    two_d = rng.random() < 0.3
    nodes = math.exp(rng.uniform(math.log(4096), math.log(6e5 if two_d else 8e6)))
    store = rng.choice(["fp16", "fp16", "fp32", "fp32", "bf16", "fp64"])
    if two_d:
        nx = max(48, int(round(math.sqrt(nodes) * math.exp(rng.uniform(-0.4, 0.4)))))
        ny, nz = max(48, int(round(nodes / nx))), 1
        kind, q = rng.choice(["droplet", "bubble", "table1", "dam"]), 9
    else:
        nodes = max(nodes, 24 * 24 * 24)
        e = nodes ** (1 / 3)
        nx = max(24, int(round(e * math.exp(rng.uniform(-0.2, 0.6)))))
        ny = max(24, int(round(math.sqrt(nodes / nx) * math.exp(rng.uniform(-0.2, 0.2)))))
        nz = max(24, int(round(nodes / nx / ny)))
        kind, q = rng.choice(["droplet", "bubble", "dam", "collision"]), rng.choice([27, 27, 19])
        if kind == "collision":
            nx, q = max(nx, 48), 19
    # between about 10 and 500 steps, fewer on larger grids and in FP64
    per = 2.0e8 / (nx * ny * nz) / (2.0 if store == "fp64" else 1.0)
    steps = max(10, min(500, int(per * math.exp(rng.uniform(-0.7, 0.7)))))
    collision = "bgk" if kind == "droplet" and rng.random() < 0.25 else "filter"
    return _case(None, kind, nx, ny, nz, store, steps, q, collision)


# ------------------------------------------------------------------ inputs


def _rng(case, seed):
    return np.random.Generator(np.random.PCG64([int(seed), case["kind"].encode()[0], int(case.get("nx", 0))]))


_U = 0.06  # relative velocity of the colliding droplets


def _diameter(cfg):
    return min(min(cfg["ny"], cfg["nz"]) / 3.0, cfg["nx"] / 4.0)


def _params(case):
    """Case parameters of the binding (the repository's workload parameters)."""
    dim = 2 if case["nz"] == 1 else 3
    cfg = {"dim": dim, "nx": case["nx"], "ny": case["ny"], "nz": case["nz"], "q_hydro": case["q_hydro"],
           "q_phase": 9 if dim == 2 else 19, "wall": (0, 0, 0), "delta_theta": 1, "rho_heavy": 1000.0,
           "rho_light": 1.0, "nu_heavy": 0.05, "nu_light": 0.05, "sigma": 0.005, "W": 4.0, "M": 0.166,
           "lambda_bulk": 1.0 / 6.0, "gravity": (0.0, 0.0, 0.0), "store": case["store"],
           "collision": case["collision"]}
    down = (lambda g: (0.0, -g, 0.0)) if dim == 2 else (lambda g: (0.0, 0.0, -g))
    kind = case["kind"]
    if kind == "droplet":
        if case["collision"] == "bgk":  # needs the larger viscosity at this density ratio
            cfg.update(nu_heavy=0.1, nu_light=0.1)
        elif dim == 2:
            cfg.update(sigma=0.01, nu_heavy=0.1, nu_light=0.1)
    elif kind == "bubble":
        cfg.update(sigma=0.01, nu_heavy=0.02, nu_light=0.2, W=5.0, wall=(0, 1, 0) if dim == 2 else (0, 0, 1),
                   gravity=down(1e-6), rho_heavy=100.0)
    elif kind == "table1":
        cfg.update(wall=(1, 1, 0), gravity=down(1.36e-8), rho_heavy=2.2, rho_light=0.22, nu_heavy=7.3e-3 / 2.2,
                   nu_light=7.3e-4 / 0.22, sigma=3.0e-5)
    elif kind == "dam":
        cfg.update(wall=(1, 1, 0) if dim == 2 else (1, 1, 1), gravity=down(2e-6), nu_heavy=0.01, nu_light=0.05)
    elif kind == "block":
        nx, ny, nz = case["nx"], case["ny"], case["nz"]
        x0, by = int(0.231 * nx), int(0.403 * ny)
        y0, bx, bz = (ny - by) // 2, max(2, int(0.05 * nx)), max(2, int(0.161 * nz))
        cfg.update(wall=(1, 1, 2), gravity=(0.0, 0.0, -(0.0289 ** 2) / (2.0 * 0.55 * nz)), p_top=0.0,
                   rho_heavy=815.6, nu_heavy=4e-3, nu_light=0.0513, sigma=0.003,
                   block=((x0, y0, 0), (x0 + bx, y0 + by, bz)))
    elif kind == "collision":
        # We = 58.4 and the paper's viscosity ratio; Re as far as stability lets it
        nu = 2.3e-3
        cfg.update(nu_heavy=nu, nu_light=15.1 * nu, sigma=1000.0 * _U ** 2 * _diameter(cfg) / 58.4)
    return cfg


def _axes(cfg):
    ax = [torch.arange(n, dtype=torch.float64) for n in (cfg["nx"], cfg["ny"], cfg["nz"])]
    return ax[0][None, None, :], ax[1][None, :, None], ax[2][:, None, None]


def _tanh(d, W):
    return torch.tanh(d * (2.0 / W)).mul_(0.5).add_(0.5)


def _fields(case, cfg, seed):
    """Initial phi, P, u as host FP64 arrays."""
    r = _rng(case, seed)
    x, y, z = _axes(cfg)
    dim, nx, ny, nz, W = cfg["dim"], cfg["nx"], cfg["ny"], cfg["nz"], cfg["W"]
    shape = (nz, ny, nx)
    P = torch.zeros(shape, dtype=torch.float64)
    u = torch.zeros((dim,) + shape, dtype=torch.float64)
    least = min(nx, ny) if dim == 2 else min(nx, ny, nz)
    shift = r.uniform(-0.04, 0.04, 3) * least

    def ball(c, R):
        r2 = (x - c[0] - shift[0]) ** 2 + (y - c[1] - shift[1]) ** 2
        if dim == 3:
            r2 = r2 + (z - c[2] - shift[2]) ** 2
        return (R - r2.expand(shape).sqrt())

    kind = case["kind"]
    if kind == "droplet":
        R = least * r.uniform(0.18, 0.25)
        phi = _tanh(ball((nx / 2, ny / 2, nz / 2), R), W)
        if dim == 3:
            for a, v in enumerate((0.05, 0.02, 0.0)):
                u[a] += v * r.uniform(0.8, 1.2)
    elif kind in ("bubble", "table1"):
        R = least * (r.uniform(0.15, 0.18) if kind == "bubble" else r.uniform(0.23, 0.27))
        c = (nx / 2, ny / 4, 0) if dim == 2 else (nx / 2, ny / 2, nz / 4)
        phi = _tanh(-ball(c, R), W)
    elif kind in ("dam", "block"):
        up, n_up = (y, ny) if dim == 2 else (z, nz)
        if kind == "dam":
            dx = (nx * r.uniform(0.22, 0.28) - 0.5) - x
            top = n_up * r.uniform(0.45, 0.55) - 0.5
        else:
            dx = x - (nx * r.uniform(0.73, 0.77) - 0.5)
            top = 0.55 * n_up * r.uniform(0.95, 1.05) - 0.5
        dz = top - up
        d = torch.where((dx < 0) & (dz < 0), -torch.sqrt(dx * dx + dz * dz), torch.minimum(dx, dz))
        phi = _tanh(d, W).expand(shape).clone()
        if kind == "block":  # hydrostatic pressure under the open top
            g = -cfg["gravity"][2]
            rho = cfg["rho_light"] + phi * (cfg["rho_heavy"] - cfg["rho_light"])
            w = rho + torch.cat([rho[1:], torch.zeros_like(rho[:1])])
            P = 0.5 * g * torch.flip(torch.cumsum(torch.flip(w, [0]), 0), [0])
            (x0, y0, _), (x1, y1, z1) = cfg["block"]
            phi[:z1, y0:y1, x0:x1] = 0.0
            P[:z1, y0:y1, x0:x1] = 0.0
    else:  # collision
        U, D = _U, _diameter(cfg)
        R, gap = D / 2 * r.uniform(0.95, 1.05), 8.0 * D / 64.0
        p1 = _tanh(ball((nx / 2 - D / 2 - gap, ny / 2, nz / 2), R), W)
        p2 = _tanh(ball((nx / 2 + D / 2 + gap, ny / 2, nz / 2), R), W)
        phi = p1 + p2
        P += (2.0 * cfg["sigma"] / R) * phi
        u[0] += 0.5 * U * r.uniform(0.9, 1.1) * (p1 - p2)
    return phi.contiguous().numpy(), P.contiguous().numpy(), u.numpy()


def _requests(case, seed):
    """The requests of a serving case: sizes, kinds and steps belong to the
    case, the fields to the seed."""
    sizes = np.random.Generator(np.random.PCG64(case["requests"] * 1000 + case["largest_2d"]))
    out = []
    for k in range(case["requests"]):
        if k % 4 == 3:
            n = int(round(math.exp(sizes.uniform(math.log(128), math.log(case["largest_2d"])))))
            c = _case(None, "droplet" if k % 8 == 3 else "bubble", n, n, 1, case["store"], case["steps"])
        else:
            n = int(round(math.exp(sizes.uniform(math.log(32), math.log(case["largest_3d"])))))
            c = _case(None, "droplet" if k % 2 == 0 else "bubble", n, n, n, case["store"], case["steps"])
        cfg = _params(c)
        out.append((cfg, _fields(c, cfg, seed * 100 + k), int(case["steps"] * sizes.uniform(0.6, 1.0))))
    return out


# --------------------------------------------------------------- measured


def prepare(case, seed):
    if case["kind"] == "serving":
        reqs = _requests(case, seed)
        return {"batch": B.Batch(4 << 30, store=case["store"], max_slots=64), "requests": reqs}
    cfg = _params(case)
    c = B.Case(cfg)
    c.init_fields(*_fields(case, cfg, seed))
    return {"case": c, "steps": case["steps"], "single": case["store"] != "fp64"}


def _snapshot(fields, single):
    t = [torch.from_numpy(f) for f in fields]
    phi, P, u = [f.to(torch.float32) for f in t] if single else t
    return {"phi": phi, "P": P, "u": u}


def run(state):
    if "batch" in state:
        return _serve(state["batch"], state["requests"])
    c = state["case"]
    c.step(state["steps"])
    return _snapshot(c.read_fields(), state["single"])


def _serve(batch, requests, k=50):
    """Admit every request, advance the batch and take each as it finishes."""
    slot_of = {}
    for i, (cfg, fields, steps) in enumerate(requests):
        slot_of[batch.admit(cfg, *fields, steps)] = i
    out = [None] * len(requests)
    while slot_of:
        batch.advance(k)
        for s in batch.poll():
            out[slot_of.pop(s)] = _snapshot(batch.take(s), True)
    return out


def _work_of(nodes, q, steps, dim, store):
    """Bytes and operations of `steps` steps and one read-back: a step reads
    and writes the populations and the pressure and velocity carried with
    them; about 40 operations per population (equilibria, collisions, moments
    and stencils)."""
    sb, ab = STORE_BYTES[store], 8 if store == "fp64" else 4
    pops = q + (9 if dim == 2 else 19)
    step = 2 * (pops * sb + (1 + dim) * ab)
    return nodes * (steps * step + (2 + dim) * 8), nodes * steps * pops * 40


def work(case):
    if case["kind"] == "serving":
        parts = [_work_of(c["nx"] * c["ny"] * c["nz"], c["q_hydro"], n, c["dim"], c["store"])
                 for c, _, n in _requests(case, 0)]
    else:
        parts = [_work_of(case["nx"] * case["ny"] * case["nz"], case["q_hydro"], case["steps"],
                          2 if case["nz"] == 1 else 3, case["store"])]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


# ------------------------------------------------------ the step in 64 bits


def exact(case, seed):
    """phi, P, u after the pass's steps from a plain FP64 form of the step
    (whole-grid arrays); None where the grid is too large for it, and for the
    block and the open top."""
    if case["kind"] == "serving":
        return [dict(zip(("phi", "P", "u"), _reference(cfg, f, n))) if cfg["nx"] ** cfg["dim"] * n < 6e7 else None
                for cfg, f, n in _requests(case, seed)]
    nodes = case["nx"] * case["ny"] * case["nz"]
    if case["kind"] == "block" or (nodes + 150000) * case["steps"] > 5e8:
        return None
    cfg = _params(case)
    return dict(zip(("phi", "P", "u"), _reference(cfg, _fields(case, cfg, seed), case["steps"])))


_T = 1.0 / 3.0
_W = {(2, 9): (4 / 9, 1 / 9, 1 / 36, 0), (3, 19): (1 / 3, 1 / 18, 1 / 36, 0), (3, 27): (8 / 27, 2 / 27, 1 / 54, 1 / 216)}


def _lattice(dim, q):
    w = _W[dim, q]
    cs = [c + (0,) * (3 - dim) for c in itertools.product((0, 1, -1), repeat=dim)]
    return [(c, w[sum(map(abs, c))]) for c in cs if w[sum(map(abs, c))]]


def _reference(cfg, fields, steps):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    dim, wall, grav = cfg["dim"], cfg["wall"], cfg["gravity"]
    n = (cfg["nx"], cfg["ny"], cfg["nz"])
    G, H = _lattice(dim, cfg["q_hydro"]), _lattice(dim, cfg["q_phase"])
    ra, rw = cfg["rho_light"], cfg["rho_heavy"]
    ta, tw = cfg["nu_light"] / _T + 0.5, cfg["nu_heavy"] / _T + 0.5
    tau_phi, theta0 = cfg["M"] / _T + 0.5, cfg["M"] / (_T * cfg["W"])
    sigma, W, lam = cfg["sigma"], cfg["W"], cfg["lambda_bulk"]
    pairs = [(c, w) for c, w in G if c > (0, 0, 0)]  # one of each opposite pair

    def pad(f, sign=1.0, add=None):
        """One ghost layer on the last three axes: the other end's nodes, or
        beyond a wall the nearest node's value times sign (plus add)."""
        for a in range(3):
            ax, m = f.dim() - 1 - a, n[a]
            lo, hi = f.narrow(ax, m - 1, 1), f.narrow(ax, 0, 1)
            if wall[a]:
                lo, hi = hi * sign, lo * sign
                if add is not None:
                    lo, hi = lo + add, hi + add
            f = torch.cat([lo, f, hi], ax)
        return f

    def at(fp, c, s=1):
        for a in range(3):
            fp = fp.narrow(fp.dim() - 1 - a, 1 + s * c[a], n[a])
        return fp

    def grad(fp, lap_of=None):
        """Central gradient (and Laplacian) of padded fields."""
        g = [0.0] * dim
        lap = 0.0
        for c, w in pairs:
            p, m = at(fp, c), at(fp, c, -1)
            d = (p - m) * (w / _T)
            for a in range(dim):
                if c[a]:
                    g[a] = g[a] + c[a] * d
            if lap_of is not None:
                lap = lap + (p + m - 2.0 * lap_of) * (2.0 * w / _T)
        return g, lap

    zero = torch.zeros((n[2], n[1], n[0]), dtype=torch.float64, device=dev)
    # g . (ghost - mirror) on the ghost frame: the hydrostatic part of P there
    off = torch.zeros([v + 2 for v in zero.shape], dtype=torch.float64, device=dev)
    for a in range(3):
        if wall[a]:
            off.narrow(2 - a, 0, 1).sub_(grav[a])
            off.narrow(2 - a, n[a] + 1, 1).add_(grav[a])
    walled = any(wall)

    def props(phi):
        pc = phi.clamp(0.0, 1.0)
        return ra + pc * (rw - ra), ta + pc * (tw - ta)

    def reconstruct(h, g):
        phi = sum(h.values())
        rho, _ = props(phi)
        J = torch.stack([sum(c[a] * g[c] for c, _ in G if c[a]) for a in range(dim)])
        Ps = ra * _T * sum(g.values())
        Pp = pad(Ps)
        Jp = pad(J, -1.0, torch.tensor([2.0 * v for v in grav[:dim]], device=dev, dtype=torch.float64).reshape(-1, 1, 1, 1)
                 if walled else None)
        sk, su = 0.0, 0.0
        for c, w in pairs:
            sk = sk + w * (at(Pp, c) + at(Pp, c, -1) - 2.0 * Ps)
            if walled:
                sk = sk + w * rho * (at(off, c) + at(off, c, -1))
            d = at(Jp, c, -1) - at(Jp, c)
            su = su + w * sum(c[a] * d[a] for a in range(dim) if c[a])
        P = Ps + sk + (rho - ra) * su
        Pp = pad(P)
        u = [J[a] for a in range(dim)]
        for c, w in pairs:
            d = at(Pp, c) - at(Pp, c, -1)
            if walled:
                d = d + rho * (at(off, c) - at(off, c, -1))
            d = d * (w / _T) / rho
            for a in range(dim):
                if c[a]:
                    u[a] = u[a] - c[a] * d
        return phi, P, torch.stack(u)

    def dot(c, v):
        t = [v[a] if c[a] > 0 else -v[a] for a in range(dim) if c[a]]
        return sum(t) if t else 0.0

    def collide(h, g, phi, P, u):
        """Post-collision populations (equilibria where h is None) and the
        force part of g's equilibrium over w_i c_i."""
        rho, tau = props(phi)
        gphi, lap = grad(pad(phi), phi)
        grho, _ = grad(pad(rho))
        gu, _ = grad(pad(u, -1.0))  # gu[b][a] = d u_a / d x_b
        gn = torch.sqrt(sum(v * v for v in gphi))
        nv = [v / (gn + 1e-10) for v in gphi]
        theta = theta0 * (1.0 - 4.0 * (phi - 0.5) ** 2)
        if cfg["delta_theta"]:
            s = lap / (lap.abs() + 1e-10)
            ramp = lambda v: (v * 1e4).clamp(0.0, 1.0)  # noqa: E731
            y1 = torch.minimum(ramp(phi - 0.8), ramp(1.0 - phi))
            y2 = torch.minimum(ramp(phi), ramp(0.2 - phi))
            theta = theta - 22.5 * theta0 * gn * ((1.0 + s) * y1 + (1.0 - s) * y2)
        u2 = sum(u[a] * u[a] for a in range(dim))
        nu = _T * (tau - 0.5)
        mu = (48.0 * sigma / W) * phi * (phi - 1.0) * (phi - 0.5) - 1.5 * sigma * W * lap
        F = [rho * grav[a] + mu * gphi[a] for a in range(dim)]
        div = sum(gu[a][a] for a in range(dim))
        bulk = rho * (2.0 / 3.0) * (lam - nu) * div
        av = []
        for a in range(dim):
            sg = sum(rho * nu * (gu[b][a] + gu[a][b]) * grho[b] for b in range(dim)) + bulk * grho[a]
            av.append(u[a] + F[a] / rho + sg / (rho * rho))
        Bd = ((2.0 / 3.0) * (nu - lam) + _T / 2.0) * div
        hs, gs = {}, {}
        for c, w in H:
            cu = dot(c, u)
            eq = w * (phi * (1.0 + cu / _T + cu * cu / (2 * _T * _T) - u2 / (2 * _T)) + theta * dot(c, nv))
            hs[c] = eq if h is None else h[c] + (eq - h[c]) / tau_phi
        if h is not None and cfg["collision"] == "filter":
            kf = (1.0 - 1.0 / tau) / (2.0 * _T * _T)
            Pi = {}
            for a in range(dim):
                for b in range(a, dim):
                    m = sum(c[a] * c[b] * g[c] for c, _ in G if c[a] * c[b])
                    Pi[a, b] = kf * (m - u[a] * u[b] - (Bd if a == b else 0.0))
            tr = _T * sum(Pi[a, a] for a in range(dim))
        for c, w in G:
            cu = dot(c, u)
            e = cu * cu / (2 * _T * _T) - u2 / (2 * _T) + Bd / _T + dot(c, av) / _T
            eq = w * e
            if c == (0, 0, 0):
                eq = eq - Bd / _T + P / (ra * _T)
            if h is None:
                gs[c] = eq
            elif cfg["collision"] == "filter":
                ph = -tr
                for a in range(dim):
                    for b in range(a, dim):
                        if c[a] * c[b]:
                            ph = ph + (1 if a == b else 2) * c[a] * c[b] * Pi[a, b]
                gs[c] = eq + w * ph
            else:
                gs[c] = g[c] + (eq - g[c]) / tau
        return hs, gs, [v * (2.0 / _T) / rho for v in F]

    leaves = {}
    if walled:
        for c, _ in G + H:
            m = torch.zeros(zero.shape, dtype=torch.bool, device=dev)
            for a in range(3):
                if wall[a] and c[a]:
                    m.narrow(2 - a, 0 if c[a] < 0 else n[a] - 1, 1).fill_(True)
            leaves[c] = m if bool(m.any()) else None

    def stream(f, lat, F):
        out = {}
        for c, w in lat:
            o = (-c[0], -c[1], -c[2])
            v = torch.roll(f[c], (c[2], c[1], c[0]), (0, 1, 2)) if any(c) else f[c]
            if walled and leaves[o] is not None:
                # what left through a wall along o comes back along c, with the
                # force part of its equilibrium kept
                v = torch.where(leaves[o], f[o] - w * dot(o, F) if F is not None else f[o], v)
            out[c] = v
        return out

    phi, P, u = (torch.from_numpy(np.ascontiguousarray(f)).to(dev) for f in fields)
    h, g, _ = collide(None, None, phi, P, u)
    for _ in range(steps):
        phi, P, u = reconstruct(h, g)
        hs, gs, F2 = collide(h, g, phi, P, u)
        h, g = stream(hs, H, None), stream(gs, G, F2 if walled else None)
    return reconstruct(h, g)
