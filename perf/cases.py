"""Performance cases: what a program does with this library, over the sizes it does it at.

Four kinds of work, each through the Python binding as a program calls it (default tile and
variant, as the README's example):

  steps     a run of the lattice with its point forces: n forced steps, then the density and
            velocity fields, the particle positions and the interpolated velocities
  fields    set-up and read-out without steps: equilibrium of a given field, moments, velocity
            at arbitrary points, FP64 diagnostics
  network   one training iteration of the mobility network and its value on held-out samples

Fields of FP32-arithmetic runs are kept in FP32, the precision such a run computes them in (a
program that writes snapshots does the same); FP64 runs and particle positions stay FP64.

`exact` repeats a case in FP64 with plain torch: spreading and interpolation with Peskin's
four-point kernel, the forced multiple-relaxation-time collision on D3Q19, propagation, the
colloid update, springs, the fluctuating collision with its Philox draws, and the network.
"""
import json
import math
import os

import numpy as np
import torch

from paper_0707_1299_amd import lbm, mobility

DEV = "cuda"


# ---- cases ----------------------------------------------------------------------------------

def _case(kind="steps", nx=32, ny=32, nz=32, nboxes=1, storage="fp32", collision="projected", kT=0.0, points="static",
          n=1, network=False, steps=10, **more):
    return dict(kind=kind, nx=nx, ny=ny, nz=nz, nboxes=nboxes, storage=storage, collision=collision, kT=kT,
                points=points, n=n, network=network, steps=steps, **more)


def listed():
    return [
        # validation run: one point force in a 32^3 box in FP64 (latency: 32768 nodes per step)
        _case(name="stokeslet_32_fp64", storage="fp64", steps=200),
        # the paper's sedimentation study at its own scale: 321 colloids in a small box
        _case(name="suspension_48", nx=48, ny=48, nz=48, points="colloids", n=321, steps=100),
        # fixed point singularities in a 128^3 box, the flow-field runs
        _case(name="singularities_128", nx=128, ny=128, nz=128, n=149, steps=50),
        # general collision operator on a box with no round size
        _case(name="mrt_ragged", nx=101, ny=75, nz=62, collision="mrt", n=40, steps=50),
        # fluctuating fluid with Brownian colloids
        _case(name="brownian_128", nx=128, ny=128, nz=128, kT=1e-5, points="colloids", n=1000, steps=40),
        # mobility labels: many independent 32^3 boxes with a fixed colloid each
        _case(name="label_boxes_512", nboxes=512, points="boxes", n=512, steps=40),
        # polymers: 2048 bead-spring chains of 32 markers in 256^3
        _case(name="chains_256", nx=256, ny=256, nz=256, points="chains", n=65536, steps=15),
        # sedimenting suspension, 10^4 colloids in 256^3
        _case(name="sediment_256", nx=256, ny=256, nz=256, points="colloids", n=10000, steps=20),
        # the same with ten moments per node stored instead of nineteen populations
        _case(name="moments_256", nx=256, ny=256, nz=256, storage="mom32", points="colloids", n=10000, steps=20),
        # the largest: 10^5 colloids in 512^3, FP16 storage, the network in the colloid update
        _case(name="sediment_512_net", nx=512, ny=512, nz=512, storage="fp16", points="colloids", n=100000,
              network=True, steps=10),
        # set-up and read-out of a field with points in it
        _case(name="fields_128", kind="fields", nx=128, ny=96, nz=80, n=20000, steps=0),
        # a training iteration of the mobility network at its usual sample count
        _case(name="network_1024", kind="network", n=1024, points="none", steps=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["steps"] * 6 + ["boxes", "fields", "network"])
    if what == "network":
        return _case(kind="network", n=_log_int(rng, 100, 40000), points="none", steps=1)
    if what == "boxes":
        L, nb = _log_int(rng, 16, 48), _log_int(rng, 16, 512)
        return _case(nx=L, ny=L, nz=L, nboxes=nb, storage=rng.choice(["fp32", "fp32", "fp16", "mom32"]), points="boxes",
                     n=nb, steps=rng.randint(4, 60))
    # boxes of 9^3 (the paper's smallest) to 256^3, one axis in four of its own length
    L = _log_int(rng, 9, 256)
    n3 = [L if rng.random() < 0.75 else max(6, min(320, int(L * rng.uniform(0.5, 1.6)))) for _ in range(3)]
    N = n3[0] * n3[1] * n3[2]
    most = max(1, min(20000, N // 64))
    if what == "fields":
        return _case(kind="fields", nx=n3[0], ny=n3[1], nz=n3[2], storage=rng.choice(["fp32", "fp64", "fp16", "mom32"]),
                     n=_log_int(rng, 1, 30000), steps=0)
    storage = rng.choice(["fp32", "fp32", "fp32", "fp16", "fp64", "mom32"])
    collision = "projected" if storage == "mom32" else rng.choice(["projected", "projected", "projected", "bgk", "mrt"])
    kT = 1e-5 if storage != "mom32" and rng.random() < 0.2 else 0.0
    points = rng.choice(["static", "colloids", "colloids", "chains", "none"])
    n = 0 if points == "none" else _log_int(rng, 1, most)
    if points == "chains":
        n = 8 * max(1, n // 8)
    return _case(nx=n3[0], ny=n3[1], nz=n3[2], storage=storage, collision=collision, kT=kT, points=points, n=n,
                 network=points == "colloids" and rng.random() < 0.3,
                 steps=max(4, min(200, int(rng.uniform(0.3, 1.0) * 3.0e8 / max(N, 1.5e6)))))


# ---- inputs, from the seed alone (host) -----------------------------------------------------

RHO0 = 1.0
INV_A, INV_AL = 1.0 / 0.684, 0.77     # colloid radius and lattice radius
CHAIN, SPRING, REST = 8, 1e-3, 1.0    # markers per chain, spring constant and rest length


def _chain_len(case):
    return 32 if case["n"] % 32 == 0 else CHAIN


def _taus(case, g):
    if case["points"] == "boxes":
        return g.uniform(0.6, 1.5, case["nboxes"])
    return np.full(case["nboxes"], 0.8 if case["points"] == "chains" else 0.5)


def _rates(case):
    """bulk relaxation time (None: tau) and ghost eigenvalue of the general operator"""
    return (1.0, 1.5) if case["collision"] == "mrt" else (None, 2.0)


def _flows(case):
    """cases that start from a given flow: set-up and read-out, and runs without forces (a decaying flow)"""
    return case["kind"] == "fields" or case["points"] == "none"


def _unit(g, n):
    v = g.normal(size=(n, 3))
    return v / np.linalg.norm(v, axis=1, keepdims=True)


def _inputs(case, seed):
    g = np.random.default_rng([7, int(seed)])
    ext = np.array([case["nx"], case["ny"], case["nz"]], dtype=np.float64)
    n, d = case["n"], dict(tau=_taus(case, g), zero_net=case["points"] in ("colloids", "boxes", "chains"))
    if case["kind"] == "fields" or case["points"] == "static":
        # force pairs (stresslets) of separation 2 along a random axis; an odd last one is a single force
        m = n if case["kind"] == "steps" else max(1, n // 100)
        c, a, s = g.uniform(0, 1, (m, 3)) * ext, _unit(g, m), g.uniform(-1e-5, 1e-5, (m, 1))
        h = m // 2
        d["pos"] = np.concatenate([c[:h] + a[:h], c[:h] - a[:h], c[2 * h:]]) % ext
        d["frc"] = np.concatenate([s[:h] * a[:h], -s[:h] * a[:h], s[2 * h:] * a[2 * h:]])
    elif case["points"] == "colloids":
        d["pos"] = g.uniform(0, 1, (n, 3)) * ext
        d["frc"] = np.tile([0.0, 0.0, -1e-6], (n, 1))
    elif case["points"] == "boxes":
        d["pos"] = ext / 2 + g.uniform(0, 1, (n, 3))
        d["frc"] = np.tile([0.0, 0.0, -1e-6], (n, 1))
        d["box"] = np.arange(n, dtype=np.int32)
    elif case["points"] == "chains":
        m = _chain_len(case)
        start = g.uniform(0, 1, (n // m, 1, 3)) * ext
        walk = np.cumsum(_unit(g, n - n // m).reshape(n // m, m - 1, 3), axis=1)
        d["pos"] = np.concatenate([start, start + walk], axis=1).reshape(n, 3) % ext
        d["frc"] = np.tile([0.0, 0.0, -1e-6], (n, 1))
    if _flows(case):
        # a smooth flow: mean velocity, shear waves along each axis, a density wave
        k = 2 * np.pi / ext
        d["mean"], d["amp"], d["phase"] = g.uniform(0.5e-3, 1e-3, 3), g.uniform(-1e-3, 1e-3, (3, 3)), g.uniform(0, 6, (4, 3))
        d["k"] = k
    if case["kind"] == "fields":
        d["at"] = g.uniform(0, 1, (n, 3)) * ext
    return d


def _flow(case, d):
    """density [nz, ny, nx] and velocity [3, nz, ny, nx] that a case starts from (FP64, device)"""
    ax = [torch.arange(case[a], dtype=torch.float64, device=DEV) for a in ("nx", "ny", "nz")]
    wave = [[torch.sin(ax[a] * d["k"][a] + d["phase"][c][a]) for a in range(3)] for c in range(4)]
    view = [(1, 1, -1), (1, -1, 1), (-1, 1, 1)]
    shape = (case["nz"], case["ny"], case["nx"])
    u = torch.empty((3,) + shape, dtype=torch.float64, device=DEV)
    for c in range(3):
        u[c] = d["mean"][c]
        for a in range(3):
            u[c] += d["amp"][c][a] * wave[c][a].view(view[a])
    rho = RHO0 * 1.001 + 1e-3 * (wave[3][0].view(view[0]) * wave[3][1].view(view[1]) * wave[3][2].view(view[2]))
    return rho.contiguous(), u


def _network_inputs(case, seed):
    g = np.random.default_rng([11, int(seed)])
    n = case["n"]
    parts = []
    for shape in ((64, 4), (64,), (64, 64), (64,), (1, 64), (1,)):
        lim = math.sqrt(6.0 / sum(shape)) if len(shape) == 2 else 0.05
        parts.append(g.uniform(-lim, lim, shape).ravel())
    off, tau = g.uniform(0, 1, (n + max(1, n // 4), 3)), g.uniform(0.5, 1.5, n + max(1, n // 4))
    x = np.concatenate([2 * off - 1, (tau[:, None] - 1.05) / 0.45], axis=1).astype(np.float32)
    y = (np.cos(2 * np.pi * off).sum(1) / 3 * (0.5 + 0.5 * tau) + g.normal(scale=0.02, size=len(off))).astype(np.float32)
    m = g.normal(scale=1e-3, size=4545)
    v = (np.abs(m) + 1e-3) ** 2 * g.uniform(0.5, 2.0, 4545)
    return dict(master=np.concatenate(parts).astype(np.float32), m=m.astype(np.float32), v=v.astype(np.float32),
                x=x[:n], y=y[:n], xt=x[n:])


T0, LR, B1, B2, EPS = 200, 1e-3, 0.9, 0.999, 1e-8


# ---- what a program has in hand, and one pass ------------------------------------------------

def _dev(a, dtype=torch.float64):
    return torch.tensor(a, dtype=dtype, device=DEV)


def prepare(case, seed):
    if case["kind"] == "network":
        d = _network_inputs(case, seed)
        s = {k: _dev(v, torch.float32) for k, v in d.items()}
        s["w16"] = torch.zeros(lbm.LBML_NPARAM, dtype=torch.int16, device=DEV)
        lbm.lbml_round_bf16(s["master"], s["w16"])
        s["grad"] = torch.empty(lbm.LBML_NPARAM, dtype=torch.float32, device=DEV)
        s["loss"] = torch.empty(1, dtype=torch.float32, device=DEV)
        s["yt"] = torch.empty(len(d["xt"]), dtype=torch.float32, device=DEV)
        s["work"] = torch.empty(lbm.lbml_work_floats(case["n"]), dtype=torch.float32, device=DEV)
        s["t"], s["case"] = T0, case
        return s
    d = _inputs(case, seed)
    s = dict(case=case)
    tau_bulk, ghost = _rates(case)
    lat = lbm.Lattice((case["nz"], case["ny"], case["nx"]), case["storage"], nboxes=case["nboxes"], tau=d["tau"],
                      zero_net_force=d["zero_net"], max_points=len(d.get("pos", ())), collision=case["collision"],
                      tau_bulk=tau_bulk, ghost_rate=ghost, kT=case["kT"], seed=int(seed) + 1,
                      fp16_exponent=16 if _flows(case) else 0)   # a flow of 1e-2: |df / w| 2^16 far below 65504
    s["lat"] = lat
    if "pos" in d:
        pos, frc = _dev(d["pos"]), _dev(d["frc"])
        s["vel"] = torch.zeros_like(pos)
        if case["points"] == "colloids":
            model = dict(inv_a=INV_A, inv_aL=INV_AL, vel_out=s["vel"])
            if case["network"]:
                model = mobility.load(mobility.DEFAULT_NET).model(INV_A, vel_out=s["vel"])
                lat.add_point_forces(pos, frc, None, lbm.LB_COLLOIDS, model)
            else:
                lat.add_point_forces(pos, frc, None, lbm.LB_COLLOIDS, lbm.PointModel(**model))
            s["pos"] = pos
        elif case["points"] == "boxes":
            lat.add_point_forces(pos, frc, _dev(d["box"], torch.int32), lbm.LB_FORCES_STATIC,
                                 lbm.PointModel(vel_sum=s["vel"]))
        elif case["points"] == "chains":
            s["bond"] = lat.add_chains(pos, _chain_len(case), SPRING, REST, ext=frc, vel_out=s["vel"])
            s["pos"] = pos
        else:
            lat.add_point_forces(pos, frc, None, lbm.LB_FORCES_STATIC)
            del s["vel"]
    if _flows(case):
        rho, u = _flow(case, d)
        s["rho"], s["u"] = rho[None].contiguous(), u[None].contiguous()
    if case["kind"] == "fields":
        s["at"] = _dev(d["at"])
    else:
        if _flows(case):
            lat.set_equilibrium(s["rho"], s["u"])
        lat.prepare_steps(case["steps"])   # graphs captured once, as a program does before its time loop
    return s


def _kept(case, t):
    return t if case["storage"] == "fp64" else t.float()


def run(state):
    case = state["case"]
    if case["kind"] == "network":
        s = state
        lbm.lbml_loss_grad(s["w16"], s["x"], s["y"], s["grad"], s["loss"], s["work"])
        lbm.lbml_adam_step(s["master"], s["m"], s["v"], s["grad"], s["w16"], s["t"], lr=LR, beta1=B1, beta2=B2, eps=EPS)
        lbm.lbml_forward(s["w16"], s["xt"], s["yt"])
        s["t"] += 1
        return dict(loss=s["loss"], grad=s["grad"], master=s["master"], m=s["m"], v=s["v"],
                    weights=s["w16"].view(torch.bfloat16), held_out=s["yt"])
    lat = state["lat"]
    if case["kind"] == "fields":
        lat.set_equilibrium(state["rho"], state["u"])
        rho, u = lat.moments()
        at = lat.interp_velocity(state["at"])
        _, diag = lat.diagnostics()
        return dict(rho=_kept(case, rho), u=_kept(case, u), at=_kept(case, at), mass=diag[:, 0].astype(np.float32),
                    momentum=diag[:, 1:4].astype(np.float32), force=diag[:, 4:7].astype(np.float32),
                    umax=diag[:, 10].astype(np.float32), bad=diag[:, 11:13].astype(np.int64))
    lat.step(case["steps"])
    rho, u = lat.moments()
    out = dict(rho=_kept(case, rho), u=_kept(case, u))
    if "pos" in state:
        out["pos"] = state["pos"]
    if "vel" in state:
        out["vel"] = _kept(case, state["vel"])
    return out


# ---- the least work of a pass ---------------------------------------------------------------

VALUES = {"fp64": 19 * 8, "fp32": 19 * 4, "fp16": 19 * 2, "mom32": 10 * 4}    # bytes of one node's state


def work(case):
    if case["kind"] == "network":
        n, held = case["n"], max(1, case["n"] // 4)
        return dict(bytes=4 * (5 * n + 5 * held) + 4545 * (2 + 4 + 6 * 4 + 2),
                    flops=2 * 4545 * (3 * n + held))
    N = case["nx"] * case["ny"] * case["nz"] * case["nboxes"]
    b, out = VALUES[case["storage"]], 8 if case["storage"] == "fp64" else 4
    if case["kind"] == "fields":
        # the field in, the state out and read again by each read-out, the field back
        return dict(bytes=N * (32 + b + 2 * b + 4 * out) + case["n"] * (24 + 3 * out), flops=N * 350 + case["n"] * 64 * 40)
    # each step reads and writes the state (far over the caches in the larger cases) and its points
    node = 250 + (600 if case["kT"] > 0 else 0) + (100 if case["collision"] != "projected" else 0)
    return dict(bytes=case["steps"] * (2 * b * N + 150 * case["n"]) + N * (b + 4 * out),
                flops=case["steps"] * (node * N + case["n"] * (64 * 20 + (8800 if case["network"] else 0))))


# ---- the same in 64 bits --------------------------------------------------------------------

C = [(0, 0, 0)] + [(x, y, z) for x in (-1, 0, 1) for y in (-1, 0, 1) for z in (-1, 0, 1) if 0 < x * x + y * y + z * z < 3]
W = [1 / 3 if c == (0, 0, 0) else (1 / 18 if sum(v * v for v in c) == 1 else 1 / 36) for c in C]


class _Stencil:
    """Peskin weights and node indices of points; flat index over (box, z, y, x)"""

    def __init__(self, case, pos, box):
        ext = [case["nx"], case["ny"], case["nz"]]
        idx, wgt = [], []
        for a in range(3):
            x = pos[:, a] % ext[a]
            b = torch.floor(x)
            r = torch.abs((x - b)[:, None] - torch.arange(-1.0, 3.0, dtype=torch.float64, device=DEV)[None])
            near = (3 - 2 * r + torch.sqrt(torch.clamp(1 + 4 * r - 4 * r * r, min=0))) / 8
            far = (5 - 2 * r - torch.sqrt(torch.clamp(-7 + 12 * r - 4 * r * r, min=0))) / 8
            wgt.append(torch.where(r < 1, near, far))
            idx.append((b.long()[:, None] + torch.arange(-1, 3, device=DEV)[None]) % ext[a])
        i = (idx[2][:, :, None, None] * ext[1] + idx[1][:, None, :, None]) * ext[0] + idx[0][:, None, None, :]
        if box is not None:
            i = i + box.long()[:, None, None, None] * (ext[0] * ext[1] * ext[2])
        self.i = i.reshape(-1)
        self.w = (wgt[2][:, :, None, None] * wgt[1][:, None, :, None] * wgt[0][:, None, None, :]).reshape(len(pos), 64)

    def spread(self, frc, total):
        g = torch.zeros((3, total), dtype=torch.float64, device=DEV)
        for a in range(3):
            g[a].index_add_(0, self.i, (self.w * frc[:, a:a + 1]).reshape(-1))
        return g

    def interp(self, u):
        return torch.stack([(u[a][self.i].view(-1, 64) * self.w).sum(1) for a in range(3)], dim=1)


def _springs(case, pos, ext_force):
    m = _chain_len(case)
    L = torch.tensor([case["nx"], case["ny"], case["nz"]], dtype=torch.float64, device=DEV)
    p = pos.view(-1, m, 3)
    d = p[:, 1:] - p[:, :-1]
    d = d - L * torch.round(d / L)
    r = d.norm(dim=2, keepdim=True)
    f = SPRING * (r - REST) * d / r
    F = torch.zeros_like(p)
    F[:, :-1] += f
    F[:, 1:] -= f
    return F.view(-1, 3) + ext_force


def _philox(c, k):
    """Philox4x32-10 (Salmon et al. 2011) on int64 tensors of 32-bit words"""
    M = 0xFFFFFFFF

    def mul(a, b):     # high and low words of a 32 x 32 product, in pieces that fit 63 bits
        t = a * (b & 0xFFFF)
        u = a * (b >> 16)
        lo = t + ((u & 0xFFFF) << 16)
        return (lo >> 32) + (u >> 16), lo & M
    k0, k1 = k
    for _ in range(10):
        h0, l0 = mul(c[0], 0xD2511F53)
        h1, l1 = mul(c[2], 0xCD9E8D57)
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return c


def _normals(first, second, t, j, key):
    one = torch.ones_like(first)
    v = _philox([first, one * second, one * (t & 0xFFFFFFFF), one * (((t >> 32) & 0x0FFFFFFF) << 4 | j)], key)
    u = [(x.double() + 0.5) * 2.0 ** -32 for x in v]
    out = []
    for a in (0, 2):
        r = torch.sqrt(-2 * torch.log(u[a]))
        out += [r * torch.cos(2 * math.pi * u[a + 1]), r * torch.sin(2 * math.pi * u[a + 1])]
    return out


def _mode(k, c):
    """the orthogonal basis of Duenweg, Schiller and Ladd (2007), without mass and momentum"""
    x, y, z = c
    q = x * x + y * y + z * z
    return [q - 1, 3 * x * x - q, y * y - z * z, x * y, x * z, y * z, (3 * q - 5) * x, (3 * q - 5) * y, (3 * q - 5) * z,
            (y * y - z * z) * x, (z * z - x * x) * y, (x * x - y * y) * z, 3 * q * q - 6 * q + 1,
            (2 * q - 3) * (3 * x * x - q), (2 * q - 3) * (y * y - z * z)][k]


def _net(w, x):
    """4 -> 64 tanh -> 64 tanh -> 1; returns the layers' values"""
    W1, b1, W2, b2, W3, b3 = (w[0:256].view(64, 4), w[256:320], w[320:4416].view(64, 64), w[4416:4480], w[4480:4544], w[4544])
    h1 = torch.tanh(x @ W1.T + b1)
    h2 = torch.tanh(h1 @ W2.T + b2)
    return h1, h2, h2 @ W3 + b3


def _trained():
    path = os.path.join(os.path.dirname(os.path.abspath(lbm.__file__)), "mobility_net.json")
    with open(path) as f:
        d = json.load(f)
    w = (np.asarray(d["w16"], dtype=np.uint32) << 16).view(np.float32).astype(np.float64)
    return _dev(w), d["mu_plain"], d["out_scale"]


def _moments(f, g):
    rho = f.sum(0)
    j = [0, 0, 0]
    for i, c in enumerate(C):
        for a in range(3):
            if c[a]:
                j[a] = j[a] + c[a] * f[i]
    u = [(j[a] + 0.5 * g[a]) / (RHO0 + rho) for a in range(3)]
    return rho, j, u


def _collide(case, f, g, tau, t, key):
    """post-collision populations in place of f, and u; per-box tau as [nboxes, 1]"""
    tau_bulk, ghost = _rates(case)
    tb = tau if tau_bulk is None else torch.full_like(tau, tau_bulk)
    kappa = (1 - 0.5 / tau) / (1 + 0.5 / tau) if case["collision"] == "bgk" else torch.full_like(tau, (1 - ghost / 2) / (1 + ghost / 2))
    om, omb = 1 / (tau + 0.5), 1 / (tb + 0.5)
    shape = f[0].shape
    nb = case["nboxes"]
    box = lambda v: v.expand(nb, shape[0] // nb).reshape(-1) if nb > 1 else float(v)   # noqa: E731
    tau, tb, om, omb, kappa = (box(v) for v in (tau, tb, om, omb, kappa))
    drho, j, u = _moments(f, g)
    rho = RHO0 + drho
    pairs = [(0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2)]
    S, D = [], []
    for a, b in pairs:
        s = sum(c[a] * c[b] * f[i] for i, c in enumerate(C) if c[a] * c[b])
        s = s - drho / 3 if a == b else s
        S.append(s)
        D.append(s - rho * u[a] * u[b] - tau * (u[a] * g[b] + g[a] * u[b]))
    tr = (D[0] + D[1] + D[2]) / 3
    trb = sum(S[a] - rho * u[a] * u[a] - 2 * tb * u[a] * g[a] for a in range(3)) / 3
    B = [S[q] - om * (D[q] - tr if q < 3 else D[q]) - (omb * trb if q < 3 else 0) for q in range(6)]
    del D
    keep = bool((torch.as_tensor(kappa) != 0).any())
    noise = None
    if case["kT"] > 0:
        node = torch.arange(shape[0], device=DEV)
        z = [q for k in range(4) for q in _normals(node, 0, t, k, key)]
        gam = [1 - omb] + [1 - om] * 5 + [kappa] * 9
        noise = []
        for k in range(15):
            norm = sum(w * _mode(k, c) ** 2 for w, c in zip(W, C))
            noise.append(torch.sqrt(3 * case["kT"] * rho * (1 - gam[k] ** 2) / norm) * z[k])
    for i, c in enumerate(C):
        q = [c[a] * c[b] - (1 / 3 if a == b else 0) for a, b in pairs]
        new = drho + 3 * sum(c[a] * (j[a] + g[a]) for a in range(3) if c[a])
        new = new + 4.5 * sum((1 if k < 3 else 2) * q[k] * B[k] for k in range(6) if q[k])
        if keep:
            old = drho + 3 * sum(c[a] * j[a] for a in range(3) if c[a])
            old = old + 4.5 * sum((1 if k < 3 else 2) * q[k] * S[k] for k in range(6) if q[k])
            new = new + kappa * (f[i] / W[i] - old)
        if noise is not None:
            new = new + sum(_mode(k, c) * noise[k] for k in range(15) if _mode(k, c))
        f[i] = W[i] * new
    return u


def _exact_network(case, seed):
    d = {k: _dev(v) for k, v in _network_inputs(case, seed).items()}
    b16 = lambda v: v.float().bfloat16().double()   # noqa: E731
    w, n = b16(d["master"]), case["n"]
    h1, h2, y = _net(w, d["x"])
    r = y - d["y"]
    dy = 2 * r / n
    W2, W3 = w[320:4416].view(64, 64), w[4480:4544]
    z2 = dy[:, None] * W3[None] * (1 - h2 * h2)
    z1 = (z2 @ W2) * (1 - h1 * h1)
    grad = torch.cat([(z1.T @ d["x"]).reshape(-1), z1.sum(0), (z2.T @ h1).reshape(-1), z2.sum(0), dy @ h2, dy.sum()[None]])
    m = B1 * d["m"] + (1 - B1) * grad
    v = B2 * d["v"] + (1 - B2) * grad * grad
    master = d["master"] - LR * (m / (1 - B1 ** T0)) / (torch.sqrt(v / (1 - B2 ** T0)) + EPS)
    return dict(loss=(r * r).mean()[None], grad=grad, master=master, m=m, v=v, weights=b16(master),
                held_out=_net(b16(master), d["xt"])[2])


def exact(case, seed):
    if case["kind"] == "network":
        return _exact_network(case, seed)
    d = _inputs(case, seed)
    nb, shape = case["nboxes"], (case["nboxes"], case["nz"], case["ny"], case["nx"])
    N = case["nx"] * case["ny"] * case["nz"]
    key = ((int(seed) + 1) & 0xFFFFFFFF, (int(seed) + 1) >> 32)
    tau = _dev(d["tau"])[:, None]
    f = torch.zeros((19, nb * N), dtype=torch.float64, device=DEV)
    pos = frc = box = st = None
    if "pos" in d:
        pos, frc = _dev(d["pos"]), _dev(d["frc"])
        box = _dev(d["box"], torch.int64) if "box" in d else None
    L = torch.tensor([case["nx"], case["ny"], case["nz"]], dtype=torch.float64, device=DEV)
    net = _trained() if case["network"] else None
    moving = case["points"] in ("colloids", "chains")
    g = [torch.zeros(1, dtype=torch.float64, device=DEV)] * 3

    def field():
        F = _springs(case, pos, frc) if case["points"] == "chains" else frc
        s = _Stencil(case, pos, box)
        G = s.spread(F, nb * N)
        if d["zero_net"]:
            for a in range(3):
                net_f = torch.zeros(nb, dtype=torch.float64, device=DEV)
                net_f.index_add_(0, box if box is not None else torch.zeros(len(pos), dtype=torch.int64, device=DEV), F[:, a])
                G[a].view(nb, N).sub_((net_f / N)[:, None])
        return s, G, F

    if _flows(case):
        rho, u = _flow(case, d)
        for i, c in enumerate(C):
            cu = sum(c[a] * u[a] for a in range(3) if c[a]) if any(c) else torch.zeros_like(rho)
            uu = (u * u).sum(0)
            eq = (rho - RHO0) + 3 * rho * cu + 4.5 * rho * (cu * cu - uu / 3)
            if case["storage"] == "mom32":      # that storage takes it as the state before propagation
                eq = torch.roll(eq, (c[2], c[1], c[0]), (0, 1, 2))
            f[i] = W[i] * eq.reshape(-1)
    if case["kind"] == "fields":
        st, g, _ = field()
        drho, j, u = _moments(f, g)
        at = _Stencil(case, _dev(d["at"]), None).interp(u)
        uv = torch.stack(u)
        return dict(rho=(RHO0 + drho).view(shape), u=uv.view(1, 3, *shape[1:]), at=at, mass=drho.sum()[None],
                    momentum=torch.stack([q.sum() for q in j])[None], force=None,
                    umax=uv.norm(dim=0).max()[None], bad=None)

    vel = torch.zeros_like(pos) if pos is not None else None
    F = frc
    for t in range(case["steps"]):
        if pos is not None and (moving or st is None):
            st, g, F = field()
        u = _collide(case, f, g, tau, t, key)
        for i, c in enumerate(C):
            if any(c):
                f[i] = torch.roll(f[i].view(shape), (c[2], c[1], c[0]), (1, 2, 3)).reshape(-1)
        if case["points"] in ("colloids", "chains", "boxes"):
            U = st.interp(u)
            vel = vel + U if case["points"] == "boxes" else U
        if case["points"] == "chains":
            pos = (pos + U) % L
        elif case["points"] == "colloids":
            eta, aL = RHO0 * float(tau[0]) / 3, torch.full_like(pos[:, :1], INV_AL)
            if net is not None:
                o = pos - torch.floor(pos)
                x = torch.cat([2 * o - 1, torch.full_like(o[:, :1], (float(tau[0]) - 1.05) / 0.45)], dim=1)
                aL = net[1] + net[2] * _net(net[0], x)[2][:, None]
            move = U + F / (6 * math.pi * eta) * (INV_A - aL)
            if case["kT"] > 0:
                z = _normals(torch.arange(len(pos), device=DEV), 0xFFFFFFFF, t, 0, key)[:3]
                move = move + torch.sqrt(case["kT"] / (3 * math.pi * eta) * (INV_A - aL)) * torch.stack(z, dim=1)
            pos = (pos + move) % L
    if moving:
        _, g, _ = field()
    drho, _, u = _moments(f, g)
    out = dict(rho=(RHO0 + drho).view(shape),
               u=torch.stack(u).view(3, *shape).transpose(0, 1).contiguous())
    if moving:
        out["pos"] = pos
    if moving or case["points"] == "boxes":
        out["vel"] = vel
    return out
