"""Measured cases of the library: what a user's program calls, with the sizes it calls them at.

A case is a plain dict; ``listed()`` names the fixed ones, ``draw(rng)`` makes one more of the same
ranges.  ``prepare(case, seed)`` builds the inputs and the handles a program keeps (network, table,
tree), ``run(state)`` is one pass through the public entry points, ``work(case)`` the bytes and
operations the path cannot do without, ``exact(case, seed)`` the same outputs in 64 bits from plain
torch (GPU memory if there is any), or None where that would take too long or has no meaning.

Loads are the ones of the tests, the simulation driver and the benchmark: the stereographic cylinder
load (flat mass density, surface density falling as (1 + r^2/R0^2)^-2), the same with Plummer clumps,
and the displaced load that time steps start from.
"""
import math
import os

import numpy as np
import torch

import paper_2602_20787_amd as sc

L = 1.0
R0, CHI_MAX = 0.5, 0.9 * math.pi  # scale and compact edge of the load
R_EDGE = R0 * math.tan(0.5 * CHI_MAX)
NET = os.path.join(os.path.dirname(os.path.abspath(sc.__file__)), "data", "correction_net.bin")
RHO_MAX, N_RHO, N_DELTA, N_FAR = 6.4, 144, 128, 1024


def listed():
    return [
        # a handful of particles, the nearest images: a unit test's or an interactive call, all latency
        {"name": "exact_tiny", "path": "exact", "N": 500, "n_img": 2, "pot": True, "load": "plain"},
        # the accuracy configuration: 4096 particles, every particle checked against the reference
        {"name": "exact_4k", "path": "exact", "N": 4096, "n_img": 8, "pot": True, "load": "plain"},
        # a time step's forces (no potential) of a medium run, a size that divides by nothing
        {"name": "exact_odd", "path": "exact", "N": 30011, "n_img": 4, "pot": False, "load": "displaced"},
        # the clustered configuration: 64 Plummer clumps in 262,144 particles
        {"name": "exact_clumps", "path": "exact", "N": 262144, "n_img": 8, "pot": True, "load": "clumps"},
        # spot check of a run: some targets against every particle, per-target sums
        {"name": "targets", "path": "targets", "N": 262144, "n_tgt": 4096, "n_img": 8, "pot": True,
         "load": "displaced"},
        # direct sum with the paper's band table, CIC, as a time step calls it
        {"name": "table_cic", "path": "table", "N": 131072, "order": 1, "complete": False, "pot": False,
         "load": "displaced"},
        # the complete table with TSC and the potential, ragged size
        {"name": "table_tsc", "path": "table", "N": 20011, "order": 2, "complete": True, "pot": True,
         "load": "plain"},
        # learned correction, the accuracy configuration
        {"name": "learned_4k", "path": "learned", "N": 4096, "pot": False, "load": "plain"},
        # learned correction of a medium run, ragged size
        {"name": "learned_64k", "path": "learned", "N": 65573, "pot": False, "load": "displaced"},
        # octree forces at the benchmark's size
        {"name": "tree_1m", "path": "tree", "N": 1048576, "theta": 0.5, "quad": False, "order": 1,
         "load": "plain"},
        # one kick-drift-kick step of an octree run with quadrupoles
        {"name": "kdk_tree", "path": "kdk", "N": 100003, "theta": 0.5, "quad": True, "order": 1,
         "load": "displaced"},
        # a stretch of the correction network's training at the batch the trainer uses
        {"name": "train", "path": "train", "batch": 8192, "steps": 100, "n_train": 65536},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["exact", "exact", "exact", "table", "table", "learned", "learned", "targets", "tree", "tree",
                       "kdk", "train"])
    load = rng.choice(["plain", "displaced", "clumps"])
    pot = rng.random() < 0.5
    if path == "exact":
        return {"path": path, "N": _log_int(rng, 500, 200000), "n_img": rng.choice([1, 2, 4, 8, 8]), "pot": pot,
                "load": load}
    if path == "table":
        return {"path": path, "N": _log_int(rng, 2000, 131072), "order": rng.choice([1, 2]),
                "complete": rng.random() < 0.5, "pot": pot, "load": load}
    if path == "learned":
        return {"path": path, "N": _log_int(rng, 2000, 65536), "pot": pot, "load": load}
    if path == "targets":
        return {"path": path, "N": _log_int(rng, 8192, 262144), "n_tgt": _log_int(rng, 256, 8192),
                "n_img": rng.choice([1, 4, 8]), "pot": pot, "load": load}
    if path in ("tree", "kdk"):
        return {"path": path, "N": _log_int(rng, 20000, 1048576 if path == "tree" else 262144),
                "theta": rng.choice([0.4, 0.5, 0.6, 0.7]), "quad": rng.random() < 0.5, "order": rng.choice([1, 1, 2]),
                "load": load}
    return {"path": path, "batch": rng.choice([1024, 2048, 4096, 8192]), "steps": rng.randrange(20, 101),
            "n_train": rng.choice([32768, 65536])}


def _load(case, seed):
    """Positions (3, N), masses and softening lengths of the case's load, as numpy arrays."""
    N, kind = case["N"], case["load"]
    rng = np.random.default_rng(seed)

    def radius(n):
        return R0 * np.tan(0.5 * np.arccos(1.0 - rng.random(n) * (1.0 - math.cos(CHI_MAX))))

    per = int(round(0.005 * N)) if kind == "clumps" else 0
    n_bg = N - 64 * per
    z, phi, r = rng.random(n_bg) * L, rng.random(n_bg) * (2.0 * math.pi), radius(n_bg)
    pos = np.stack([r * np.cos(phi), r * np.sin(phi), z])
    if per:
        # Plummer spheres of scale 0.005 around 64 centres of the load
        phi, r = rng.random(64) * (2.0 * math.pi), radius(64)
        mid = np.repeat(np.stack([r * np.cos(phi), r * np.sin(phi), rng.random(64) * L]), per, axis=1)
        rad = 0.005 / np.sqrt((0.999 * (1.0 - rng.random(64 * per))) ** (-2.0 / 3.0) - 1.0)
        way = rng.standard_normal((3, 64 * per))
        pos = np.concatenate([pos, mid + rad * way / np.linalg.norm(way, axis=0)], axis=1)
    m = (1.0 + (pos[0] ** 2 + pos[1] ** 2) / R0 ** 2) ** 2
    m /= m.sum()
    if kind == "displaced":
        # 3D rms of half the mean spacing
        spacing = (math.pi * R_EDGE ** 2 * L / N) ** (1.0 / 3.0)
        pos = pos + 0.5 * spacing / math.sqrt(3.0) * rng.standard_normal((3, N))
    pos[2] -= L * np.floor(pos[2] / L)
    return np.ascontiguousarray(pos), m, 0.01 * np.cbrt(m / m.min())


def _targets(case, seed):
    rng = np.random.default_rng(seed + 1)
    return np.sort(rng.choice(case["N"], size=case["n_tgt"], replace=False)).astype(np.int64)


def _rho0():
    return 1.0 / (math.pi * R_EDGE ** 2 * L)


def _first_params(seed):
    """Initial network parameters: uniform weights by fan-in, a small output layer."""
    rng = np.random.default_rng(seed)
    flat = []
    for o, i in ((64, 2), (64, 64), (64, 64), (64, 64), (2, 64)):
        a = 0.1 * math.sqrt(3.0 / i) if o == 2 else math.sqrt(6.0 / i)
        flat += [rng.uniform(-a, a, o * i), rng.uniform(-0.1, 0.1, o) * (o > 2)]
    return np.concatenate(flat).astype(np.float32)


def _training_inputs(n, seed):
    """(|d|/L, rho/L): uniform and log-uniform over the network's domain."""
    rng = np.random.default_rng(seed)
    return np.stack([0.5 * rng.random(n), 0.05 * np.exp(math.log(400.0) * rng.random(n))])


def prepare(case, seed):
    dev = torch.device("cuda:0")
    path = case["path"]
    s = {"case": case}
    if path == "train":
        s["p0"] = _first_params(seed)
        s["net"] = sc.Mlp.create(s["p0"])
        s["inputs"] = torch.from_numpy(_training_inputs(case["n_train"], seed)).to(dev)
        return s
    pos, mass, eps = _load(case, seed)
    s["pos"] = torch.from_numpy(pos).to(dev)
    s["mass"] = torch.from_numpy(mass).to(dev)
    s["eps"] = torch.from_numpy(eps).to(dev)
    if path == "targets":
        s["targets"] = torch.from_numpy(_targets(case, seed)).to(dev)
    elif path == "table":
        s["table"] = (sc.CorrectionTable.ewald(N_DELTA, N_RHO, RHO_MAX, 2.0, 5, 12) if case["complete"]
                      else sc.CorrectionTable(N_DELTA, N_RHO, RHO_MAX, N_FAR))
    elif path == "learned":
        s["net"] = sc.Mlp.load(NET)
    elif path in ("tree", "kdk"):
        s["table"] = sc.CorrectionTable.ewald(N_DELTA, N_RHO, RHO_MAX, 2.0, 5, 12)
        s["tree"] = sc.Octree(16, quadrupole=case["quad"])
        rng = np.random.default_rng(seed + 3)
        s["shift"], s["angle"] = float(rng.random() * L), float(rng.random() * 2.0 * math.pi)
        s["R"] = 1.02 * float(np.hypot(pos[0], pos[1]).max())
    if path == "kdk":
        # forces in hand at the start of the step: the homogeneous cylinder's, with some structure
        rng = np.random.default_rng(seed + 4)
        g = -2.0 * math.pi * _rho0()
        acc = np.stack([g * pos[0], g * pos[1], 0.0 * pos[2]])
        acc += 0.05 * abs(g) * rng.standard_normal(acc.shape)
        H0 = math.sqrt(8.0 * math.pi * _rho0() / 0.9)
        s["snap"] = (s["pos"].clone(), torch.zeros_like(s["pos"]), torch.from_numpy(acc.astype(np.float32)).to(dev))
        s["mom"] = torch.zeros_like(s["pos"])
        s["acc"] = torch.empty_like(s["snap"][2])
        s["params"] = sc.kdk_params(0.5, 0.53, H0, 0.3, 0.7, R_cyl=s["R"], rho0=_rho0(), table=s["table"],
                                    table_order=case["order"], tree=s["tree"], theta=case["theta"],
                                    tree_shift=s["shift"], tree_angle=s["angle"])
    return s


def run(s):
    case = s["case"]
    path = case["path"]
    if path == "exact":
        return sc.steps_cyl_forces(s["pos"], s["mass"], s["eps"], L, case["n_img"], potential=case["pot"])
    if path == "targets":
        return sc.steps_cyl_forces_ex(s["pos"], s["mass"], s["eps"], L, case["n_img"], targets=s["targets"],
                                      potential=case["pot"])
    if path == "table":
        return sc.steps_cyl_forces_table(s["pos"], s["mass"], s["eps"], L, s["table"], order=case["order"],
                                         potential=case["pot"])
    if path == "learned":
        return sc.steps_cyl_forces_learned(s["pos"], s["mass"], s["eps"], L, s["net"], potential=case["pot"])
    if path == "tree":
        return sc.steps_cyl_tree_forces(s["tree"], s["pos"], s["mass"], s["eps"], L, s["R"], s["table"],
                                        case["order"], case["theta"], s["shift"], s["angle"])
    if path == "kdk":
        # the step from the snapshot: its state is copied into the run's arrays first
        for a, b in zip((s["pos"], s["mom"], s["acc"]), s["snap"]):
            a.copy_(b)
        sc.steps_cyl_kdk_step(s["pos"], s["mom"], s["mass"], s["eps"], L, s["params"], s["acc"])
        return {"pos": s["pos"], "mom": s["mom"], "acc": s["acc"]}
    s["net"].set_params(s["p0"])
    s["net"].train(s["inputs"], case["steps"], case["batch"], lr=2e-3, lr_min=1e-5, seed=1)
    return s["net"].params()


def work(case):
    path = case["path"]
    if path == "train":
        n = case["steps"] * case["batch"]
        return {"bytes": 16 * case["n_train"] + 8 * sc.STEPS_MLP_PARAMS, "flops": n * 6 * 12800}
    N = case["N"]
    pairs = N * (N - 1) // 2  # every unordered pair once: the term and its two applications
    out = {"bytes": 40 * N + (16 if case.get("pot") else 12) * N}
    if path == "exact":
        out["flops"] = pairs * (37 + 20 * case["n_img"])
    elif path == "targets":
        out["flops"] = case["n_tgt"] * N * (28 + 20 * case["n_img"])
        out["bytes"] = 40 * N + 24 * case["n_tgt"]
    elif path == "table":
        out["flops"] = pairs * (57 + (30 if case["order"] == 1 else 60))
    elif path == "learned":
        out["flops"] = pairs * (57 + 60 + 2 * 12544 + 4 * 256)
    else:
        # interactions per particle grow as log N and about as theta^-2 (2900 at 2^20 particles, theta 0.5)
        per = 2900.0 * math.log2(N) / 20.0 * (0.5 / case["theta"]) ** 2
        out["flops"] = int(N * per * (78 + (180 if case["quad"] else 0)))
        if path == "kdk":
            out["bytes"] = 16 * N + 2 * 60 * N
    return out


# ------------------------------------------------------------------ the same sums in 64 bits


def _spline(r, h):
    """F/r and -P of the cubic-spline law where r < h, else Newton."""
    u = r / h
    w = 1.0 - u
    u2 = u * u
    core = u < 0.5
    f_in = (32.0 / 3.0 + u2 * (-38.4 + 32.0 * u)) / h ** 3
    p_in = (2.8 - u2 * (16.0 / 3.0 + u2 * (-9.6 + 6.4 * u))) / h
    rs = torch.clamp(r, min=1e-300)
    f_mid = (1.0 - w ** 4 * (16.0 - w * (25.6 - 32.0 / 3.0 * w))) / rs ** 3
    p_mid = (3.2 - 1.0 / (15.0 * torch.clamp(u, min=1e-300))
             - u2 * (32.0 / 3.0 + u * (-16.0 + u * (9.6 - 32.0 / 15.0 * u)))) / h
    out = r >= h
    f = torch.where(out, 1.0 / rs ** 3, torch.where(core, f_in, f_mid))
    q = torch.where(out, 1.0 / rs, torch.where(core, p_in, p_mid))
    return f, q


def _direct(load, tgt, n_img, far, dev):
    """Accelerations and potentials of targets tgt with images |n| <= n_img and far(rho, d) -> (Rz, Rrho)."""
    pos, m, h = (torch.from_numpy(a).to(dev) for a in load)
    x, y, z = pos
    assert 2.0 * float(h.max()) <= 0.5 * L  # then only the image n = 0 is ever softened
    tgt = torch.arange(len(m), device=dev) if tgt is None else torch.from_numpy(tgt).to(dev)
    acc = torch.empty((3, len(tgt)), dtype=torch.float64, device=dev)
    pot = torch.empty(len(tgt), dtype=torch.float64, device=dev)
    step = max(1, ((1 << 22) if far is not None else (1 << 26)) // len(m))
    for a in range(0, len(tgt), step):
        t = tgt[a:a + step]
        dx, dy = x[t, None] - x[None], y[t, None] - y[None]
        d = z[t, None] - z[None]
        d -= L * torch.floor(d / L + 0.5)
        rho2 = dx * dx + dy * dy
        S, Q = _spline(torch.sqrt(rho2 + d * d), h[t, None] + h[None])
        F = S * d
        for n in range(-n_img, n_img + 1):
            if n == 0:
                continue
            u = d - n * L
            q = torch.rsqrt(rho2 + u * u)
            Q += q
            q3 = q * q * q
            S += q3
            F += u.mul_(q3)
        if far is not None:
            rho = torch.sqrt(rho2)
            Rz, Rr = far(rho / L, d / L)
            S -= Rr / (L * L) / torch.clamp(rho, min=1e-300)
            F -= Rz / (L * L)
        own = torch.arange(len(t), device=dev)
        for v in (S, F, Q):
            v[own, t] = 0.0
        S *= m
        acc[0, a:a + step] = -(S * dx).sum(1)
        acc[1, a:a + step] = -(S * dy).sum(1)
        acc[2, a:a + step] = -(F @ m)
        pot[a:a + step] = -(Q @ m)
    return acc, pot


def _band(rho, d, n_far):
    """The images 2 <= |n| <= n_far of one unit mass, (F_z, F_rho) at separations rho, d (units of L)."""
    fz, fr = torch.zeros_like(rho), torch.zeros_like(rho)
    r2 = rho * rho
    for n in range(n_far, 1, -1):
        for u in (d - n, d + n):
            q3 = (r2 + u * u) ** -1.5
            fz -= u * q3
            fr -= rho * q3
    return fz, fr


def _complete(rho, d):
    """Every image |n| >= 2: 400 images a side, beyond them rods with the midpoint rule's end term
    (the next one is below 1e-14)."""
    fz, fr = _band(rho, d, 400)
    r2 = rho * rho
    for s in (1.0, -1.0):
        u = s * 400.5 - d  # axial distance of the rod's end
        q = (r2 + u * u) ** -0.5
        fz += s * q + s * (r2 - 2.0 * u * u) * q ** 5 / 24.0
        fr += -rho * q * q / (1.0 + s * u * q) + s * 3.0 * rho * u * q ** 5 / 24.0
    return fz, fr


def _table_far(case, dev):
    i = torch.arange(-1, N_DELTA + 2, dtype=torch.float64, device=dev) / (2.0 * N_DELTA)
    j = torch.arange(-1, N_RHO + 2, dtype=torch.float64, device=dev) * (RHO_MAX / N_RHO)
    r, dl = torch.meshgrid(j, i, indexing="ij")
    nodes = _complete(r, dl) if case["complete"] else _band(r, dl, N_FAR)
    tab = torch.stack(nodes, -1).reshape(-1, 2)
    w = N_DELTA + 3

    def far(rho, d):
        a, b = d.abs() * (2.0 * N_DELTA), rho * (N_RHO / RHO_MAX)
        t = torch.zeros(rho.shape + (2,), dtype=torch.float64, device=dev)
        if case["order"] == 1:
            ia, ib = a.floor().clamp(0, N_DELTA - 1), b.floor().clamp(0, N_RHO - 1)
            fa, fb = a - ia, b - ib
            wa, wb, off = (1.0 - fa, fa), (1.0 - fb, fb), 0
        else:
            ia, ib = a.round().clamp(0, N_DELTA), b.round().clamp(0, N_RHO)
            fa, fb = a - ia, b - ib
            wa = (0.5 * (0.5 - fa) ** 2, 0.75 - fa * fa, 0.5 * (0.5 + fa) ** 2)
            wb = (0.5 * (0.5 - fb) ** 2, 0.75 - fb * fb, 0.5 * (0.5 + fb) ** 2)
            off = -1
        base = (ib.long() + 1 + off) * w + ia.long() + 1 + off
        for q, v in enumerate(wb):
            for k, u in enumerate(wa):
                t += (u * v)[..., None] * tab[base + q * w + k]
        Rz, Rr = torch.where(d > 0, t[..., 0], torch.where(d < 0, -t[..., 0], 0.0 * d)), t[..., 1].contiguous()
        k = torch.nonzero(rho.reshape(-1) > RHO_MAX)[:, 0]  # beyond the table
        if len(k):
            a, b = rho.reshape(-1)[k], d.reshape(-1)[k]
            ez, er = _complete(a, b) if case["complete"] else _band(a, b, N_FAR)
            Rz.view(-1)[k] = ez
            Rr.view(-1)[k] = er
        return Rz, Rr

    return far


def _learned_far(dev):
    flat = np.frombuffer(open(NET, "rb").read(), dtype=np.float32, count=sc.STEPS_MLP_PARAMS, offset=16)
    flat = torch.from_numpy(flat.copy()).to(dev)
    W, B, at = [], [], 0
    for o, i in ((64, 2), (64, 64), (64, 64), (64, 64), (2, 64)):
        W.append(flat[at:at + o * i].reshape(o, i).bfloat16().double())
        B.append(flat[at + o * i:at + o * i + o].double())
        at += o * i + o

    def far(rho, d):
        dl = d.abs()
        inside = (rho >= 0.05) & (rho <= 20.0)
        r = torch.where(inside, rho, torch.ones_like(rho))
        v = torch.stack([4.0 * dl - 1.0, 2.0 * torch.log(r / 0.05) / math.log(400.0) - 1.0], -1).reshape(-1, 2)
        for k in range(4):
            v = v @ W[k].T + B[k]
            v = v / (1.0 + torch.exp2(-v))
        v = (v @ W[4].T + B[4]).reshape(rho.shape + (2,))
        scale = 0.02 / (1.0 + r * r)
        bz, br = torch.zeros_like(r), torch.zeros_like(r)
        for s in (1.0, -1.0):
            for e, sign in ((1.5, 1.0), (1024.5, -1.0)):
                u = s * e - dl
                q = (r * r + u * u) ** -0.5
                bz += sign * s * q
                br += sign * s * u * q / r
            u = s * 1.5 - dl
            q5 = (r * r + u * u) ** -2.5
            bz += s * (r * r - 2.0 * u * u) * q5 / 24.0
            br += s * 3.0 * r * u * q5 / 24.0
        Rz, Rr = bz + scale * v[..., 0], br + scale * v[..., 1]
        Rz = torch.where(d > 0, Rz, torch.where(d < 0, -Rz, torch.zeros_like(Rz)))
        k = torch.nonzero(~inside.reshape(-1))[:, 0]
        ez, er = _band(rho.reshape(-1)[k], d.reshape(-1)[k], N_FAR)
        Rz.view(-1)[k] = ez
        Rr.view(-1)[k] = er
        return Rz, Rr

    return far


def exact(case, seed):
    dev = torch.device("cuda:0" if torch.cuda.is_available() else "cpu")
    fast = 1.0 if dev.type == "cuda" else 0.01
    path = case["path"]
    far, tgt, n_img = None, None, 1
    if path == "exact":
        n_img = case["n_img"]
        if float(case["N"]) ** 2 * (4 + n_img) > 6e10 * fast:
            return None
    elif path == "targets":
        n_img, tgt = case["n_img"], _targets(case, seed)
        if float(case["N"]) * case["n_tgt"] * (4 + n_img) > 6e10 * fast:
            return None
    elif path == "table":
        if float(case["N"]) ** 2 > 1.5e9 * fast:
            return None
        far = _table_far(case, dev)
    elif path == "learned":
        if float(case["N"]) ** 2 > 4e7 * fast:
            return None
        far = _learned_far(dev)
    else:
        return None
    acc, pot = _direct(_load(case, seed), tgt, n_img, far, dev)
    return acc, (pot if case["pot"] else None)
