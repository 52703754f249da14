"""Workloads that the performance of this framework is measured on.

A case is a dict of plain values; `kind` says which program it stands for:

  steps     a time-stepping loop: `steps` fused collide-and-stream updates of a
            periodic box or a lid-driven cavity, on a population array that the
            program owns (Lattice(torch_buffer=True)); the output is that array
  series    the same loop on a small lattice, sampled by step_reduce
  porous    flow through a porous solid to a new state, then its fields
  diagnose  what a monitor calls between stretches of steps: the domain sums,
            the enstrophy and the fields
  snapshot  box filter of a fine lattice into closure features and targets
  train     scoring the closure network on samples, then training it on them

Geometries, sizes and models are those of bench.py, the tests and closure.py:
Taylor-Green vortices of 32^3 to 512^3 nodes, lid-driven cavities, a Gaussian
random-field rock of porosity 0.20, the 7-32-32-1 closure network.  Each initial
field is drawn from the seed (a Taylor-Green vortex of random phase and
amplitude carried by a uniform drift).
"""
import math

import numpy as np
import torch

from paper_2506_09242_amd import inputs, lbm

BLOCK = 4096  # nodes per block of the population array (lbm_population_bytes)
PREC = {"f64": (8, torch.float64), "f32": (4, torch.float32), "f16s": (2, torch.float16)}
TAG = {"bgk": lbm.TAG_BGK, "trt": lbm.TAG_TRT, "smag": lbm.TAG_SMAG, "rr": lbm.TAG_RR, "mlp": lbm.TAG_MLP}
LID = (0.1, 0.02, 0.0)
DRIFT = 0.02


def listed():
    return [
        # the smallest lattice, a convergence study in FP64: launch latency and the reductions count
        dict(name="tgv32_d3q19_bgk_f64_series", kind="series", geom="periodic", nx=32, ny=32, nz=32, q=19, prec="f64",
             model="bgk", steps=20, every=5),
        # an ordinary walled lattice of odd size
        dict(name="cavity101_d3q19_bgk_f32", kind="steps", geom="cavity", nx=101, ny=101, nz=101, q=19, prec="f32",
             model="bgk", steps=20),
        # the lid-driven cavity benchmark
        dict(name="cavity256_d3q19_bgk_f32", kind="steps", geom="cavity", nx=256, ny=256, nz=256, q=19, prec="f32",
             model="bgk", steps=20),
        # the turbulent cavity's robust model in FP64
        dict(name="cavity200_d3q19_rr_f64", kind="steps", geom="cavity", nx=200, ny=200, nz=200, q=19, prec="f64",
             model="rr", steps=10),
        # the headline Taylor-Green vortex: the largest lattice
        dict(name="tgv512_d3q27_smag_f32", kind="steps", geom="periodic", nx=512, ny=512, nz=512, q=27, prec="f32",
             model="smag", steps=10),
        # the same flow in FP16 storage on an ordinary size
        dict(name="tgv256_d3q27_smag_f16s", kind="steps", geom="periodic", nx=256, ny=256, nz=256, q=27, prec="f16s",
             model="smag", steps=20),
        # a ragged periodic box, two-relaxation-time
        dict(name="box250x243x130_d3q19_trt_f32", kind="steps", geom="periodic", nx=250, ny=243, nz=130, q=19,
             prec="f32", model="trt", steps=20),
        # the coarse lattice of the learned closure, its network fused into the collision
        dict(name="tgv128_d3q27_mlp_f32", kind="steps", geom="periodic", nx=128, ny=128, nz=128, q=27, prec="f32",
             model="mlp", steps=20),
        # permeability of a rock: a long stretch of steps, then the fields
        dict(name="porous256_d3q19_trt_f32", kind="porous", geom="porous", nx=256, ny=256, nz=256, q=19, prec="f32",
             model="trt", steps=1000),
        # monitoring of a running vortex
        dict(name="diagnose192_d3q19_bgk_f32", kind="diagnose", geom="periodic", nx=192, ny=192, nz=192, q=19,
             prec="f32", model="bgk"),
        # a training snapshot of the fine run
        dict(name="snapshot256_d3q27_smag_f32", kind="snapshot", geom="periodic", nx=256, ny=256, nz=256, q=27,
             prec="f32", model="smag", factor=4),
        # two epochs of closure training
        dict(name="train65536_batch4096", kind="train", n=65536, batch=4096, epochs=2),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sides(rng, nodes, mult):
    """Three sides of about `nodes` nodes in all, within a factor of two of a cube."""
    a, b = 2.0 ** rng.uniform(-0.4, 0.4), 2.0 ** rng.uniform(-0.4, 0.4)
    n = nodes ** (1.0 / 3.0)
    return [max(16, int(round(s / mult)) * mult) for s in (n * a, n * b, n / (a * b))]


def draw(rng):
    kind = rng.choice(["steps", "steps", "steps", "steps", "series", "porous", "diagnose", "snapshot", "train"])
    if kind == "train":
        return dict(kind=kind, n=_log(rng, 20000, 131072), batch=rng.choice([1000, 2048, 4096, 4096, 8192]),
                    epochs=rng.choice([1, 2]))
    if kind == "series":
        nx, ny, nz = _sides(rng, _log(rng, 24 ** 3, 96 ** 3), rng.choice([1, 8]))
        every = rng.choice([2, 5, 10])
        return dict(kind=kind, geom="periodic", nx=nx, ny=ny, nz=nz, q=rng.choice([19, 27]),
                    prec=rng.choice(["f64", "f32"]), model=rng.choice(["bgk", "smag", "trt"]), steps=20, every=every)
    if kind == "porous":
        nx, ny, nz = _sides(rng, _log(rng, 96 ** 3, 200 ** 3), rng.choice([1, 16, 16]))
        return dict(kind=kind, geom="porous", nx=nx, ny=ny, nz=nz, q=19, prec=rng.choice(["f32", "f64"]),
                    model="trt", steps=rng.choice([300, 400, 500]))
    if kind == "diagnose":
        nx, ny, nz = _sides(rng, _log(rng, 48 ** 3, 192 ** 3), rng.choice([1, 16]))
        return dict(kind=kind, geom="periodic", nx=nx, ny=ny, nz=nz, q=rng.choice([19, 27]),
                    prec=rng.choice(["f64", "f32"]), model="bgk")
    if kind == "snapshot":
        factor = rng.choice([2, 3, 4, 4, 8])
        nx, ny, nz = _sides(rng, _log(rng, 64 ** 3, 240 ** 3), factor)
        return dict(kind=kind, geom="periodic", nx=nx, ny=ny, nz=nz, q=rng.choice([19, 27]),
                    prec=rng.choice(["f32", "f32", "f64"]), model="smag", factor=factor)
    geom = rng.choice(["periodic", "periodic", "cavity"])
    prec = rng.choice(["f32", "f32", "f64", "f16s"])
    q = rng.choice([19, 27])
    model = rng.choice(["bgk", "smag", "trt", "rr"] + (["mlp"] if geom == "periodic" else []))
    if rng.random() < 0.4:  # a power of two along x
        nx = rng.choice([64, 128, 256])
        _, ny, nz = _sides(rng, _log(rng, 64 ** 3, 256 ** 3), 1)
    else:
        nx, ny, nz = _sides(rng, _log(rng, 40 ** 3, 280 ** 3), rng.choice([1, 1, 8]))
    return dict(kind="steps", geom=geom, nx=nx, ny=ny, nz=nz, q=q, prec=prec, model=model,
                steps=rng.choice([6, 10, 20]))


# ------------------------------------------------------------------ inputs
def _dims(case):
    return case["nz"], case["ny"], case["nx"]


def _params(case):
    """Relaxation time and force of the case's flow (the values of bench.py's workloads)."""
    n = case["nx"]
    if case["geom"] == "porous":
        return dict(tau=1.0, force=(1e-5, 0.0, 0.0))
    if case["geom"] == "cavity":
        return dict(tau=3.0 * 0.1 * n / 1000.0 + 0.5, wall_velocity=[LID])
    if case["model"] in ("smag", "mlp"):
        return dict(tau=3.0 * 0.05 * (n / (2 * math.pi)) / 1600.0 + 0.5, smag_cs=0.1)
    return dict(tau=3.0 * 0.04 * n / 100.0 + 0.5)


def _rock(case, seed):
    """Gaussian random field of correlation length 8, thresholded to porosity 0.20."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    f = torch.randn(_dims(case), generator=g, device="cuda")
    for axis in range(3):
        n = f.shape[axis]
        d = torch.arange(n, device="cuda", dtype=torch.float32)
        d = torch.minimum(d, n - d)
        k = torch.exp(-(d / 8.0) ** 2)
        i = torch.arange(n, device="cuda")
        f = torch.moveaxis(torch.tensordot(k[(i[:, None] - i[None, :]) % n], f, dims=([1], [axis])), 0, axis)
    f = f.contiguous()
    cut = torch.sort(f.reshape(-1)).values[int(0.20 * f.numel()) - 1]
    return torch.where(f <= cut, TAG["trt"], lbm.TAG_SOLID).to(torch.uint8).cpu().numpy()


def _tags(case, seed):
    nz, ny, nx = _dims(case)
    if case["geom"] == "porous":
        return _rock(case, seed)
    if case["geom"] == "periodic":
        return inputs.all_fluid(nx, ny, nz, TAG[case["model"]])
    t = np.full((nz, ny, nx), lbm.TAG_SOLID, dtype=np.uint8)
    t[1:-1, 1:-1, 1:-1] = TAG[case["model"]]
    t[nz - 1] = lbm.TAG_WALL0
    return t


def _fields(case, seed):
    """Density and velocity (FP64, host): a Taylor-Green vortex with random phases and
    amplitude in a uniform drift; at rest in the rock."""
    if case["geom"] == "porous":
        return None, None
    r = np.random.RandomState(seed % (2 ** 31))
    u0 = 0.05 * r.uniform(0.8, 1.0)
    ph = r.uniform(0, 2 * math.pi, 3)
    drift = DRIFT * r.uniform(0.5, 1.0, 3)
    z, y, x = (torch.arange(n, dtype=torch.float64) * (2 * math.pi / n) + p for n, p in zip(_dims(case), ph))
    z, y, x = z[:, None, None], y[None, :, None], x[None, None, :]
    u = torch.empty((3,) + _dims(case), dtype=torch.float64)
    torch.mul(u0 * torch.sin(x) * torch.cos(y), torch.cos(z), out=u[0])
    torch.mul(-u0 * torch.cos(x) * torch.sin(y), torch.cos(z), out=u[1])
    u[2] = 0.0
    for a in range(3):
        u[a] += float(drift[a])
    rho = 3.0 * u0 * u0 / 16.0 * (torch.cos(2 * z) + 2.0) * (torch.cos(2 * x) + torch.cos(2 * y))
    rho += 1.0
    return rho.numpy(), u.numpy()


def _network(seed):
    """Closure parameters: He weights, normalisation of the features that a vortex shows."""
    p = inputs.mlp_he_init(seed)
    p[1345:1352] = [0, 0, 0, 0, 0, 0, 1.0]
    p[1352:1359] = [2e-5] * 6 + [1e-3]
    return p


def _samples(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = case["n"]
    x = torch.randn((n, 7), generator=g, device="cuda")
    noise = torch.randn(n, generator=g, device="cuda")
    y = (0.15 * x[:, :6].square().sum(1).sqrt() - 0.2 + 0.1 * noise).clamp(min=0.0)  # a third of the targets are zero
    x[:, :6] *= 2e-5
    x[:, 6] = 1.0 + 1e-3 * x[:, 6]
    perm = torch.stack([torch.randperm(n, generator=g, device="cuda") for _ in range(case["epochs"])])
    return x.contiguous(), y.contiguous(), perm.reshape(-1).contiguous()


def prepare(case, seed):
    if case["kind"] == "train":
        x, y, perm = _samples(case, seed)
        p = _network(seed)
        return dict(case=case, x=x, y=y, perm=perm, host=p, start=torch.as_tensor(p, device="cuda"),
                    params=torch.empty(lbm.MLP_NPARAMS, device="cuda"), nut=torch.empty(case["n"], device="cuda"),
                    log=torch.empty(case["epochs"], device="cuda"))
    lat = lbm.Lattice(_tags(case, seed), q=case["q"], prec=case["prec"], torch_buffer=True, **_params(case))
    lat._buf.zero_()  # the slots of solid nodes and of the last block's padding are never initialised
    if case["model"] == "mlp":
        lat.set_mlp(_network(seed))
    lat.init_equilibrium(*_fields(case, seed))
    state = dict(case=case, lat=lat)
    if case["kind"] == "snapshot":
        nc = (case["nx"] // case["factor"]) * (case["ny"] // case["factor"]) * (case["nz"] // case["factor"])
        state["feat"] = torch.empty((nc, 7), device="cuda")
        state["target"] = torch.empty(nc, device="cuda")
    if case["kind"] == "diagnose":
        lat.step(2)
    return state


def _populations(state):
    case = state["case"]
    return state["lat"]._buf.view(PREC[case["prec"]][1]).view(-1, case["q"], BLOCK)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "train":
        state["params"].copy_(state["start"])
        lbm.lbm_mlp_infer(state["host"], 0.01, state["x"], state["nut"])
        lbm.lbm_mlp_train(state["params"], state["x"], state["y"], state["perm"], case["batch"], case["epochs"], 1e-3,
                          state["log"])
        return dict(nut=state["nut"], params=state["params"], loss=state["log"])
    lat = state["lat"]
    if kind == "steps":
        lat.step(case["steps"])
        return dict(populations=_populations(state))
    if kind == "series":
        series = lat.step_reduce(case["steps"], case["every"])
        out = {k: np.array([m[k] for m in series]) for k in ("n_nonfinite", "mass", "momentum", "velocity_sum",
                                                             "kinetic_energy", "kinetic_energy_rho")}
        return dict(out, populations=_populations(state))
    if kind == "porous":
        lat.step(case["steps"])
        rho, u = lat.read_fields()
        return dict(rho=rho, u=u)
    if kind == "snapshot":
        lat.filter_snapshot(case["factor"], state["feat"], state["target"])
        return dict(features=state["feat"], target=state["target"])
    m = lat.reduce()
    w = lat.enstrophy()
    rho, u = lat.read_fields()
    return dict(mass=m["mass"], momentum=m["momentum"], kinetic_energy=m["kinetic_energy"], enstrophy=w, rho=rho, u=u)


def work(case):
    if case["kind"] == "train":
        # samples, order and targets read once an epoch and once for the score; forward and
        # backward products of a 7-32-32-1 network
        n, e = case["n"], case["epochs"]
        macs = 7 * 32 + 32 * 32 + 32
        return dict(bytes=float(e * n * (7 * 4 + 4 + 8) + n * 8 * 4), flops=float(n * (2 * macs + e * 6 * macs)))
    nodes, s = case["nx"] * case["ny"] * case["nz"], PREC[case["prec"]][0]
    pops = float(nodes * case["q"] * s)
    fluid = nodes if case["geom"] == "periodic" else 0.20 * nodes if case["geom"] == "porous" else \
        (case["nx"] - 2.0) * (case["ny"] - 2.0) * (case["nz"] - 2.0)
    if case["kind"] == "snapshot":
        return dict(bytes=pops + nodes / case["factor"] ** 3 * 32, flops=float(nodes * 40))
    if case["kind"] == "diagnose":
        return dict(bytes=pops + nodes * 32.0, flops=float(nodes * (4 * case["q"] + 130)))
    step = 2.0 * fluid * case["q"] * s  # each population read and written once a step
    flops = fluid * (14.0 * case["q"] + (2600 if case["model"] == "mlp" else 0)) * case["steps"]
    return dict(bytes=step * case["steps"] + (nodes * 32.0 if case["kind"] == "porous" else 0.0), flops=flops)


# --------------------------------------------------- the same in 64 bits, plainly
def _lattice(q):
    half = [(1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 0), (1, -1, 0), (1, 0, 1), (1, 0, -1), (0, 1, 1), (0, 1, -1),
            (1, 1, 1), (1, 1, -1), (1, -1, 1), (1, -1, -1)][: (q - 1) // 2]
    c = [(0, 0, 0)] + half + [(-a, -b, -d) for a, b, d in half]
    w = {19: {0: 1 / 3, 1: 1 / 18, 2: 1 / 36}, 27: {0: 8 / 27, 1: 2 / 27, 2: 1 / 54, 3: 1 / 216}}[q]
    return c, [w[a * a + b * b + d * d] for a, b, d in c]


def _equilibrium(q, rho, u):
    """Second-order equilibrium less w rho0 (rho0 = 1)."""
    c, w = _lattice(q)
    uu = 1.5 * (u * u).sum(0)
    out = torch.empty((q,) + tuple(rho.shape), dtype=torch.float64, device=rho.device)
    for i in range(q):
        cu = sum(c[i][a] * u[a] for a in range(3)) if i else torch.zeros_like(rho)
        out[i] = w[i] * ((rho - 1.0) + rho * (3.0 * cu + 4.5 * cu * cu - uu))
    return out


def _moments(q, h):
    c, _ = _lattice(q)
    rho = 1.0 + h.sum(0)
    j = torch.stack([sum(c[i][a] * h[i] for i in range(q) if c[i][a]) for a in range(3)])
    return rho, j / rho


def _net64(p, x):
    p = torch.as_tensor(p, dtype=torch.float64, device=x.device)
    x = (x - p[1345:1352]) / p[1352:1359]
    a = torch.relu(x @ p[0:224].view(32, 7).T + p[224:256])
    b = torch.relu(a @ p[256:1280].view(32, 32).T + p[1280:1312])
    return torch.nn.functional.softplus(b @ p[1312:1344] + p[1344])


def _collide(case, h, net):
    """Post-collision populations (no body force: the cases with one have no exact value)."""
    q, model, tau = case["q"], case["model"], _params(case)["tau"]
    c, w = _lattice(q)
    rho, u = _moments(q, h)
    e = _equilibrium(q, rho, u)
    d = h - e
    if model == "bgk":
        return h - d / tau
    if model == "trt":
        tm = 0.5 + (3.0 / 16.0) / (tau - 0.5)
        opp = [0] + [i + (q - 1) // 2 if i <= (q - 1) // 2 else i - (q - 1) // 2 for i in range(1, q)]
        do = d[opp]
        return h - (d + do) / (2 * tau) - (d - do) / (2 * tm)
    pi = {(a, b): sum(c[i][a] * c[i][b] * d[i] for i in range(1, q) if c[i][a] * c[i][b]) for a in range(3)
          for b in range(a, 3)}
    pi.update({(b, a): v for (a, b), v in list(pi.items())})
    if model in ("smag", "mlp"):
        qn = torch.sqrt(sum(pi[a, b] ** 2 for a in range(3) for b in range(3)))
        te = 0.5 * (tau + torch.sqrt(tau * tau + 18.0 * math.sqrt(2.0) * 0.01 * qn / rho))
        if model == "mlp":
            nu0 = (tau - 0.5) / 3.0
            x = torch.stack([pi[0, 0], pi[1, 1], pi[2, 2], pi[0, 1], pi[0, 2], pi[1, 2], rho], -1)
            nut = nu0 * _net64(net, x.reshape(-1, 7)).view(rho.shape)
            te = torch.where(nut <= 10 * nu0, 3.0 * (nu0 + nut) + 0.5, te)
        return h - d / te
    # recursive regularized: third-order equilibrium, deviatoric second-order and recursive
    # third-order non-equilibrium
    tr = (pi[0, 0] + pi[1, 1] + pi[2, 2]) / 3.0
    a2 = {k: (1.0 - 1.0 / tau) * (v - tr if k[0] == k[1] else v) for k, v in pi.items()}

    def t3(a, b, g):
        return rho * u[a] * u[b] * u[g] + u[a] * a2[b, g] + u[b] * a2[a, g] + u[g] * a2[a, b]

    sums = [((0, 0, 1), (1, 2, 2)), ((0, 2, 2), (0, 1, 1)), ((1, 1, 2), (0, 0, 2))]
    out = e
    for i in range(q):
        v = torch.zeros_like(rho)
        for a in range(3):
            for b in range(3):
                hab = c[i][a] * c[i][b] - (1.0 / 3.0 if a == b else 0.0)
                if hab:
                    v += 4.5 * hab * a2[a, b]

        def herm(t):
            x, y, z = t
            k = c[i][x] * c[i][y] * c[i][z]
            return k - ((x == y) * c[i][z] + (y == z) * c[i][x] + (x == z) * c[i][y]) / 3.0

        for s, t in sums:
            hp, hm = herm(s) + herm(t), herm(s) - herm(t)
            np_, nm_ = (27.0 / 2.0, 27.0 / 6.0) if q == 19 else (27.0 / 4.0, 27.0 / 4.0)
            if hp:
                v += hp * np_ * (t3(*s) + t3(*t))
            if hm:
                v += hm * nm_ * (t3(*s) - t3(*t))
        if q == 27 and c[i][0] * c[i][1] * c[i][2]:
            v += c[i][0] * c[i][1] * c[i][2] * 27.0 * t3(0, 1, 2)
        out[i] += w[i] * v
    return out


def _stream(case, h, tags):
    q = case["q"]
    c, w = _lattice(q)
    H = (q - 1) // 2
    out = torch.empty_like(h)
    for i in range(q):
        back = dict(shifts=(c[i][2], c[i][1], c[i][0]), dims=(0, 1, 2))  # the value at x - c_i
        out[i] = torch.roll(h[i], **back)
        if case["geom"] != "periodic":
            o = 0 if i == 0 else i + H if i <= H else i - H
            src = torch.roll(tags, **back)
            out[i] = torch.where(src == TAG[case["model"]], out[i], h[o])
            out[i] += (src >= lbm.TAG_WALL0).double() * (6.0 * w[i] * sum(c[i][a] * LID[a] for a in range(3)))
    if case["geom"] != "periodic":
        out[:, tags != TAG[case["model"]]] = 0.0
    return out


def _blocked(h):
    q, n = h.shape[0], h[0].numel()
    pad = torch.zeros((q, -(-n // BLOCK) * BLOCK), dtype=h.dtype, device=h.device)
    pad[:, :n] = h.reshape(q, n)
    return pad.view(q, -1, BLOCK).transpose(0, 1).contiguous()


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        x, y, perm = (t.double() if t.is_floating_point() else t for t in _samples(case, seed))
        p = torch.as_tensor(_network(seed), dtype=torch.float64, device="cuda")
        nut = 0.01 * _net64(p, x)
        n, batch, fixed = case["n"], case["batch"], p[1345:].clone()
        v = p[:1345].clone().requires_grad_(True)
        m1, m2, step, logs = torch.zeros_like(v), torch.zeros_like(v), 0, []
        for e in range(case["epochs"]):
            total, nb = 0.0, -(-n // batch)
            for b in range(nb):
                pick = perm[e * n + b * batch:min(e * n + (b + 1) * batch, (e + 1) * n)]
                loss = (_net64_grad(v, fixed, x[pick]) - y[pick]).square().mean()
                g, = torch.autograd.grad(loss, v)
                step += 1
                with torch.no_grad():
                    m1 = 0.9 * m1 + 0.1 * g
                    m2 = 0.999 * m2 + 0.001 * g * g
                    v -= 1e-3 * (m1 / (1 - 0.9 ** step)) / (torch.sqrt(m2 / (1 - 0.999 ** step)) + 1e-8)
                total += float(loss.detach()) / nb
            logs.append(total)
        return dict(nut=nut, params=torch.cat([v.detach(), fixed]), loss=torch.tensor(logs, dtype=torch.float64))
    nodes = case["nx"] * case["ny"] * case["nz"]
    if kind == "porous" or nodes * case["q"] > 600_000_000:
        return None
    rho, u = (torch.as_tensor(a, device="cuda") for a in _fields(case, seed))
    h = _equilibrium(case["q"], rho, u)
    del rho, u
    tags = torch.as_tensor(_tags(case, seed), device="cuda")
    if case["geom"] != "periodic":
        h[:, tags != TAG[case["model"]]] = 0.0
    net = _network(seed) if case["model"] == "mlp" else None
    if kind == "snapshot":
        return _filter64(case, *_moments(case["q"], h))
    series = []

    def sample():
        r, v = _moments(case["q"], h)
        k = 0.5 * (v * v).sum(0)
        return dict(n_nonfinite=None, mass=float(r.sum()), momentum=(r * v).sum((1, 2, 3)), velocity_sum=v.sum((1, 2, 3)),
                    kinetic_energy=float(k.sum()) / nodes, kinetic_energy_rho=float((r * k).sum()))

    for s in range(case.get("steps", 2)):
        if kind == "series" and s % case["every"] == 0:
            series.append(sample())
        h = _stream(case, _collide(case, h, net), tags)
    if kind == "diagnose":
        r, v = _moments(case["q"], h)
        m = sample()

        def diff(f, axis):
            return sum(k * (torch.roll(f, -s, axis) - torch.roll(f, s, axis))
                       for s, k in ((1, 0.8), (2, -0.2), (3, 4.0 / 105.0), (4, -1.0 / 280.0)))

        curl = (diff(v[2], 1) - diff(v[1], 0), diff(v[0], 0) - diff(v[2], 2), diff(v[1], 2) - diff(v[0], 1))
        return dict(mass=m["mass"], momentum=m["momentum"], kinetic_energy=m["kinetic_energy"],
                    enstrophy=0.5 * float(sum((x * x).sum() for x in curl)) / nodes, rho=r, u=v)
    if kind == "series":
        if case["steps"] % case["every"] == 0:
            series.append(sample())
        out = {k: None if k == "n_nonfinite" else torch.stack([torch.as_tensor(m[k], dtype=torch.float64).cpu() for m in series])
               for k in series[0]}
        return dict(out, populations=_blocked(h))
    return dict(populations=_blocked(h))


def _net64_grad(v, fixed, x):
    x = (x - fixed[:7]) / fixed[7:14]
    a = torch.relu(x @ v[0:224].view(32, 7).T + v[224:256])
    b = torch.relu(a @ v[256:1280].view(32, 32).T + v[1280:1312])
    return torch.nn.functional.softplus(b @ v[1312:1344] + v[1344])


def _filter64(case, rho, u):
    f = case["factor"]
    nz, ny, nx = (n // f for n in _dims(case))

    def box(a):
        return a.view(nz, f, ny, f, nx, f).mean((1, 3, 5))

    r = box(rho)
    U = torch.stack([box(rho * u[a]) / r for a in range(3)])
    T = {(a, b): box(rho * u[a] * u[b]) / r - U[a] * U[b] for a in range(3) for b in range(3)}
    G = [[0.5 * (torch.roll(U[b], -1, 2 - a) - torch.roll(U[b], 1, 2 - a)) for b in range(3)] for a in range(3)]
    S = {(a, b): 0.5 * (G[a][b] + G[b][a]) for a in range(3) for b in range(3)}
    tr = (T[0, 0] + T[1, 1] + T[2, 2]) / 3.0
    num = sum((T[k] - (tr if k[0] == k[1] else 0.0)) * S[k] for k in S)
    ss = sum(S[k] ** 2 for k in S)
    nut = (-num / (2.0 * ss + 1e-30)).clamp(min=0.0)
    nu_c = (_params(case)["tau"] - 0.5) / 3.0 / f
    k = -(2.0 / 3.0) * r * (3.0 * (nu_c + nut) + 0.5)
    feat = torch.stack([k * S[a] for a in ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))] + [r], -1)
    return dict(features=feat.reshape(-1, 7), target=(nut / nu_c).reshape(-1))
