"""The measured work of this framework: flows advanced and read out, and the learned closure's pipeline.

A case is what a program has the library do in one go through its public entry points:

* ``flow``: advance a prepared simulation by ``steps`` steps (one lb_step call) and read it out:
  "fields" (rho and u), "populations" (the whole stored state, as a checkpoint takes it) or
  "monitor" (the FP64 totals and the enstrophy beside the fields, as the dipole benchmark and the
  workload runner sample a run).  Any lattice, order, storage, box, walls and check interval.
* ``coarse_run``: start a coarse D2Q9 run with the learned closure from filtered fields, advance
  it and read the fields out.
* ``coarse_data``: one snapshot of the closure's training data: fine fields, coarse-graining,
  the fine steps of one coarse step, target, coarse state, features and labels.
* ``train``: optimiser steps of the closure network (gradient of a batch, Adam update).
* ``score``: normalisation statistics of a data set and the network's predictions on it.

Fields returned are in the element type a program asks for: FP32 for FP32 states, FP64 for FP64
states.  ``exact`` computes the same results with plain FP64 torch operations.
"""
import math

import numpy as np
import torch

import paper_1505_06900_amd as lbrr
from paper_1505_06900_amd import closure as lc

CS = 1.0 / math.sqrt(3.0)
DIM = {"D2Q9": 2, "D3Q19": 3, "D3Q27": 3}
Q = {"D2Q9": 9, "D3Q19": 19, "D3Q27": 27}
STORED_BYTES = {"fp64": 8, "fp32": 4, "fp16": 2, "mom_fp64": 8, "mom_fp32": 4}


def _flow(name, lattice, shape, storage, steps, read, order=4, tau=0.51, mach=0.1, walls="", check=0):
    nz, ny, nx = shape
    case = dict(kind="flow", lattice=lattice, nz=nz, ny=ny, nx=nx, storage=storage, steps=steps, read=read,
                order=order, tau=tau, mach=mach, walls=walls, check=check)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest grid in use: a 64^2 vortex sampled every few steps; launches and read-out latency
        _flow("vortex_64_fp64", "D2Q9", (1, 64, 64), "fp64", 10, "monitor", tau=0.596, mach=0.087),
        # the dipole-wall benchmark: FP64, walls on both axes, odd rows, energy and enstrophy sampled
        _flow("dipole_501_walls_fp64", "D2Q9", (1, 501, 501), "fp64", 100, "monitor", tau=0.5015, mach=0.05,
              walls="xy"),
        # a long 2D run with the stability check on: 2048^2 shear layer size
        _flow("shear_2048_fp32", "D2Q9", (1, 2048, 2048), "fp32", 100, "fields", tau=0.570945, mach=0.2, check=50),
        # the headline: 256^3 Taylor-Green box, FP32 populations
        _flow("tgv_256_d3q27_fp32", "D3Q27", (256, 256, 256), "fp32", 20, "fields", tau=0.504411),
        # the same box with the state held as moments
        _flow("tgv_256_d3q27_mom32", "D3Q27", (256, 256, 256), "mom_fp32", 20, "fields", tau=0.504411),
        # the largest box: 512^3 random field, FP16 populations, state written out whole
        _flow("field_512_d3q19_fp16", "D3Q19", (512, 512, 512), "fp16", 10, "populations", tau=0.51),
        # reference-precision 3D run on a box of odd sides, full order, sampled
        _flow("odd_fp64_o6", "D3Q27", (75, 131, 150), "fp64", 8, "monitor", order=6, tau=0.52),
        # a 3D channel: walls on one axis, rows that fill no whole tile
        _flow("channel_walls_fp32", "D3Q19", (65, 130, 301), "fp32", 20, "fields", order=3, tau=0.56, walls="z"),
        # the learned closure in use: a coarse run of 256^2
        dict(kind="coarse_run", name="closure_run_256", n=256, ny=256, order=4, steps=100),
        # one snapshot of the closure's training data from a 1024^2 run
        dict(kind="coarse_data", name="closure_data_1024", n=1024, ny=1024, factor=4),
        # closure training at the batch the training uses
        dict(kind="train", name="closure_train_4096", rows=1 << 20, batch=4096, steps=10),
        # statistics of a data set and predictions on it (20 snapshots of 256^2 nodes)
        dict(kind="score", name="closure_score_1m3", rows=20 * 65536),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: mostly flows, every lattice, storage, order and read-out among them."""
    kind = rng.choice(["flow2", "flow2", "flow3", "flow3", "flow3", "coarse_run", "coarse_data", "train", "score"])
    if kind == "flow2":
        nx, ny = _log_int(rng, 48, 2300), _log_int(rng, 48, 2300)
        storage = rng.choice(["fp64", "fp32", "fp16", "mom_fp64", "mom_fp32"])
        walls = rng.choice(["", "", "x", "y", "xy"])
        read = rng.choice(["fields", "monitor"]) if storage.endswith("fp64") else "fields"
        return _flow("", "D2Q9", (1, ny, nx), storage, _log_int(rng, 1, 100), "populations" if storage == "fp16" else read,
                     order=rng.choice([2, 3, 4, 4]), tau=rng.choice([0.5015, 0.51, 0.57, 0.8]),
                     mach=rng.choice([0.05, 0.1]), walls=walls, check=rng.choice([0, 0, 7, 25]))
    if kind == "flow3":
        lattice = rng.choice(["D3Q19", "D3Q27", "D3Q27"])
        storage = rng.choice(["fp64", "fp32", "fp32", "fp16", "mom_fp64", "mom_fp32"])
        nz, ny, nx = (_log_int(rng, 24, 330) for _ in range(3))
        update = 2 * Q[lattice] * STORED_BYTES[storage]  # bytes per node and step, at most those of the largest listed case
        steps = min(_log_int(rng, 1, 20), max(1, int(8e10 / (nz * ny * nx * update))))
        walls = rng.choice(["", "", "", "z", "yz", "x"])
        read = rng.choice(["fields", "monitor"]) if storage.endswith("fp64") else "fields"
        return _flow("", lattice, (nz, ny, nx), storage, steps, "populations" if storage == "fp16" else read,
                     order=rng.choice([2, 3, 4, 4] if lattice == "D3Q19" else [2, 3, 4, 4, 5, 6]),
                     tau=rng.choice([0.51, 0.52, 0.6, 0.8]), mach=rng.choice([0.05, 0.1]), walls=walls,
                     check=rng.choice([0, 0, 5]))
    if kind == "coarse_run":
        return dict(kind="coarse_run", n=_log_int(rng, 40, 1100), ny=_log_int(rng, 40, 1100), order=rng.choice([2, 3, 4]),
                    steps=_log_int(rng, 5, 100))
    if kind == "coarse_data":
        f = rng.choice([2, 3, 4, 4, 8])
        return dict(kind="coarse_data", n=f * _log_int(rng, 24, 1200 // f), ny=f * _log_int(rng, 24, 1200 // f), factor=f)
    if kind == "train":
        return dict(kind="train", rows=_log_int(rng, 5000, 1 << 20), batch=_log_int(rng, 64, 8192), steps=_log_int(rng, 1, 10))
    return dict(kind="score", rows=_log_int(rng, 1000, 20 * 65536))


# ---- inputs ------------------------------------------------------------------


def _modes(rng, n, kmax, count=3):
    """A smooth periodic profile along an axis of n nodes: a few low sine modes."""
    x = 2.0 * math.pi * torch.arange(n, device="cuda", dtype=torch.float64) / n
    out = torch.zeros(n, device="cuda", dtype=torch.float64)
    for _ in range(count):
        k = int(rng.integers(1, kmax + 1))
        out += float(rng.uniform(0.3, 1.0)) * torch.sin(k * x + float(rng.uniform(0, 2 * math.pi)))
    return out / count


def _initial(case, seed):
    """Smooth fields of a flow: a Taylor-Green vortex with random phases plus a divergence-free
    sum of profiles (u_x of y and z, u_y of z and x, u_z of x and y), 0 on walls; FP64."""
    rng = np.random.default_rng(seed)
    nz, ny, nx = case["nz"], case["ny"], case["nx"]
    d = DIM[case["lattice"]]
    u0 = case["mach"] * CS
    ax = [2.0 * math.pi * torch.arange(n, device="cuda", dtype=torch.float64) / n + float(rng.uniform(0, 2 * math.pi))
          for n in (nx, ny, nz)]
    X, Y, Z = ax[0].view(1, 1, nx), ax[1].view(1, ny, 1), ax[2].view(nz, 1, 1)
    cz = torch.cos(Z) if d == 3 else torch.ones_like(Z)
    u = torch.empty((d, nz, ny, nx), device="cuda", dtype=torch.float64)
    u[0] = 0.6 * torch.sin(X) * torch.cos(Y) * cz
    u[1] = -0.6 * torch.cos(X) * torch.sin(Y) * cz
    prof = lambda n, axis: _modes(rng, n, max(1, min(8, n // 12))).view([-1 if k == axis else 1 for k in range(3)])
    u[0] += 0.4 * prof(ny, 1)
    u[1] += 0.4 * prof(nx, 2)
    if d == 3:
        u[0] += 0.4 * prof(nz, 0)
        u[1] += 0.4 * prof(nz, 0)
        u[2] = 0.4 * prof(nx, 2) + 0.4 * prof(ny, 1)
    u *= u0
    rho = 1.0 + (3.0 * u0 * u0 / 16.0) * (torch.cos(2 * X) + torch.cos(2 * Y)) * (cz + 2.0) + torch.zeros_like(u[0])
    for axis, name in ((3, "x"), (2, "y"), (1, "z")):
        if name in case["walls"]:
            n = u.shape[axis]
            damp = torch.sin(math.pi * torch.arange(n, device="cuda", dtype=torch.float64) / (n - 1))
            damp[0] = damp[-1] = 0.0
            u *= damp.view([n if k == axis else 1 for k in range(4)])
    return rho, u


def _vorticity_fields(ny, nx, mach, seed):
    """Decaying 2D turbulence start: u from a random streamfunction of modes 4 <= |k| <= 12."""
    rng = np.random.default_rng(seed)
    x = 2.0 * math.pi * torch.arange(nx, device="cuda", dtype=torch.float64) / nx
    y = 2.0 * math.pi * torch.arange(ny, device="cuda", dtype=torch.float64) / ny
    u = torch.zeros((2, 1, ny, nx), device="cuda", dtype=torch.float64)
    for _ in range(24):
        r, th, ph = rng.uniform(4, 12), rng.uniform(0, math.pi), rng.uniform(0, 2 * math.pi)
        kx, ky = round(r * math.cos(th)), round(r * math.sin(th))
        s = torch.cos((ky * y).view(-1, 1) + (kx * x).view(1, -1) + ph) / math.hypot(kx, ky)
        u[0, 0] += ky * s
        u[1, 0] -= kx * s
    u *= mach * CS / torch.sqrt((u * u).sum(0).mean())
    return torch.ones((1, ny, nx), device="cuda", dtype=torch.float64), u


def _network(rng):
    """Network parameters and normalisation of the closure (FP32, on the GPU) and its raw feature scale."""
    p = lc.init_params(int(rng.integers(1 << 30)))
    p = p + (0.02 * rng.standard_normal(p.shape)).astype(np.float32)
    norm = np.concatenate([0.001 * rng.standard_normal(36), 0.02 * (1 + rng.uniform(size=36)),
                           1e-6 * rng.standard_normal(3), 1e-5 * (1 + rng.uniform(size=3))]).astype(np.float32)
    return torch.from_numpy(p.astype(np.float32)).cuda(), torch.from_numpy(norm).cuda()


def _data_set(rows, seed):
    """Raw features (rows x 36) and targets (rows x 3) with the scales of a coarse flow, FP32."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rng = np.random.default_rng(seed)
    scale = torch.from_numpy((0.02 * (1 + rng.uniform(size=36))).astype(np.float32)).cuda()
    shift = torch.from_numpy((0.005 * rng.standard_normal(36)).astype(np.float32)).cuda()
    z = torch.randn((rows, 36), generator=g, device="cuda")
    x = z * scale + shift
    t = 1e-5 * torch.stack([torch.tanh(z[:, 0] + 0.5 * z[:, 9]), z[:, 1] * z[:, 2], torch.sin(z[:, 4]) + 0.3 * z[:, 35]], 1)
    return x.contiguous(), t.contiguous()


TAU_FINE, TAU_COARSE = 0.535472, 0.508868  # the closure's fine and coarse relaxation times


def prepare(case, seed):
    kind = case["kind"]
    if kind == "flow":
        rho, u = _initial(case, seed)
        sim = lbrr.Simulation(case["lattice"], (case["nz"], case["ny"], case["nx"]), case["tau"], case["order"],
                              storage=case["storage"])
        if case["walls"]:
            sim.set_walls(*(a in case["walls"] for a in "xyz"))
        if case["check"]:
            sim.set_check_interval(case["check"])
        sim.init_fields(rho, u)
        return {"case": case, "sim": sim}
    if kind == "coarse_run":
        rho, u = _vorticity_fields(case["ny"], case["n"], 0.1, seed)
        params, norm = _network(np.random.default_rng(seed))
        sim = lbrr.Simulation("D2Q9", (1, case["ny"], case["n"]), TAU_COARSE, case["order"], storage="fp32")
        sim.set_closure(params, norm)
        pi1 = torch.zeros((3,) + rho.shape, device="cuda", dtype=torch.float64)
        return {"case": case, "sim": sim, "rho": rho, "u": u, "pi1": pi1, "params": params, "norm": norm}
    if kind == "coarse_data":
        rho, u = _vorticity_fields(case["ny"], case["n"], 0.1, seed)
        f = case["factor"]
        fine = lbrr.Simulation("D2Q9", (1, case["ny"], case["n"]), TAU_FINE, 4, storage="fp32")
        fine.init_fields(rho, u)
        fine.step(DATA_WARM)
        coarse = lbrr.Simulation("D2Q9", (1, case["ny"] // f, case["n"] // f), TAU_COARSE, 4, storage="fp64")
        return {"case": case, "fine": fine, "coarse": coarse}
    if kind == "train":
        x, t = _data_set(case["rows"], seed)
        rng = np.random.default_rng(seed + 1)
        params, _ = _network(rng)
        norm = _plain_norm(x, t)
        idx = torch.from_numpy(rng.integers(0, case["rows"], size=(case["steps"], case["batch"]), dtype=np.int32)).cuda()
        return {"case": case, "x": x, "t": t, "norm": norm, "idx": idx, "params": params, "m": torch.zeros_like(params),
                "v": torch.zeros_like(params), "g": torch.empty_like(params), "done": 0,
                "loss": torch.empty(1, device="cuda", dtype=torch.float32)}
    x, t = _data_set(case["rows"], seed)
    params, _ = _network(np.random.default_rng(seed + 1))
    return {"case": case, "x": x, "t": t, "params": params}


DATA_WARM = 8  # fine steps before the first snapshot


def _plain_norm(x, t):
    """Normalisation vector a program kept from an earlier statistics pass."""
    return torch.cat([x.double().mean(0), x.double().std(0, unbiased=False), t.double().mean(0),
                      t.double().std(0, unbiased=False)]).float().contiguous()


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "flow":
        sim = state["sim"]
        sim.step(case["steps"])
        if case["read"] == "populations" and not case["storage"].startswith("mom"):
            return {"populations": sim.get_populations()}
        out = {}
        if case["read"] == "monitor":
            out["totals"] = np.array(sim.reduce())
            out["enstrophy"] = sim.enstrophy()
        out["rho"], out["u"] = sim.moments(torch.float64 if case["storage"].endswith("fp64") else torch.float32)
        return out
    if kind == "coarse_run":
        sim = state["sim"]
        sim.init_fields(state["rho"], state["u"], state["pi1"])
        sim.step(case["steps"])
        rho, u = sim.moments(torch.float32)
        return {"rho": rho, "u": u}
    if kind == "coarse_data":
        fine, coarse, f = state["fine"], state["coarse"], case["factor"]
        alpha, beta = lc.state_factors(TAU_FINE, TAU_COARSE, "flux")
        rc, uc, pc = lc.coarsen(*lc.fine_fields(fine), f, alpha, beta)
        fine.step(f)
        _, _, target = lc.coarsen(*lc.fine_fields(fine), f, 0.0, lc.flux_label_factor(TAU_COARSE))
        coarse.init_fields(rc, uc, pc)
        features, labels = coarse.closure_features(a_target=target, plain_weight=0.0)
        return {"features": features, "labels": labels}
    if kind == "train":
        p = lambda t: t.data_ptr()
        s = torch.cuda.current_stream().cuda_stream
        st = state
        for k in range(case["steps"]):
            lbrr.check(lbrr.lb_mlp_gradient(p(st["params"]), p(st["norm"]), p(st["x"]), p(st["t"]), case["rows"],
                                            p(st["idx"][k]), case["batch"], p(st["g"]), p(st["loss"]), s))
            st["done"] += 1
            lbrr.check(lbrr.lb_mlp_adam(p(st["params"]), p(st["m"]), p(st["v"]), p(st["g"]), st["done"], 1e-3, 0.9, 0.999,
                                        1e-8, s))
        return {"params": st["params"], "loss": st["loss"]}
    norm = lc.norm_stats(state["x"], state["t"])
    return {"norm": norm, "y": lc.predict(state["params"], norm, state["x"])}


# ---- what a pass cannot do without --------------------------------------------

# floating-point operations of one node update (moments, coefficients, reconstruction), about
UPDATE_FLOPS = {"D2Q9": 120, "D3Q19": 400, "D3Q27": 340}
MLP_FLOPS = 2 * (36 * 64 + 64 * 64 + 64 * 3)


def _state_bytes(case):
    d = DIM[case["lattice"]]
    values = 1 + d + d * (d + 1) // 2 if case["storage"].startswith("mom") else Q[case["lattice"]]
    return case["nz"] * case["ny"] * case["nx"] * values * STORED_BYTES[case["storage"]]


def work(case):
    """Bytes: the inputs read once and the outputs (the advanced state among them) written once."""
    kind = case["kind"]
    if kind == "flow":
        nodes, d = case["nz"] * case["ny"] * case["nx"], DIM[case["lattice"]]
        out = _state_bytes(case) if case["read"] == "populations" else nodes * (1 + d) * (
            8 if case["storage"].endswith("fp64") else 4)
        return {"bytes": 2 * _state_bytes(case) + out, "flops": nodes * case["steps"] * UPDATE_FLOPS[case["lattice"]]}
    if kind == "coarse_run":
        nodes = case["n"] * case["ny"]
        return {"bytes": nodes * (6 * 8 + 9 * 4 + 3 * 4),
                "flops": nodes * case["steps"] * (UPDATE_FLOPS["D2Q9"] + MLP_FLOPS + 128 * 10)}
    if kind == "coarse_data":
        nodes, f = case["n"] * case["ny"], case["factor"]
        return {"bytes": nodes * 2 * 9 * 4 + nodes // (f * f) * 39 * 4, "flops": nodes * (f * UPDATE_FLOPS["D2Q9"] + 60)}
    if kind == "train":
        return {"bytes": case["steps"] * (case["batch"] * 40 * 4 + 6723 * 4 * 6),
                "flops": case["steps"] * case["batch"] * 3 * MLP_FLOPS}
    return {"bytes": case["rows"] * (36 + 3 + 3) * 4, "flops": case["rows"] * (MLP_FLOPS + 128 * 10 + 39 * 4)}


# ---- the same results in 64 bits, plain torch -----------------------------------


def _velocities(lattice):
    cz = (0,) if lattice == "D2Q9" else (-1, 0, 1)
    c = [(x, y, z) for z in cz for y in (-1, 0, 1) for x in (-1, 0, 1)]
    if lattice == "D3Q19":
        c = [v for v in c if v[0] ** 2 + v[1] ** 2 + v[2] ** 2 <= 2]
        return c, [{0: 1 / 3, 1: 1 / 18, 2: 1 / 36}[v[0] ** 2 + v[1] ** 2 + v[2] ** 2] for v in c]
    w1 = {-1: 1 / 6, 0: 2 / 3, 1: 1 / 6}
    return c, [w1[v[0]] * w1[v[1]] * (w1[v[2]] if lattice != "D2Q9" else 1.0) for v in c]


class _Plain:
    """The regularised scheme in plain FP64 torch: Hermite polynomials of the velocity set, their
    projection matrices, streaming by rolls, and the recursion's pair sums; in slabs of planes."""

    def __init__(self, lattice, order, tau, shape, walls):
        self.c, w = _velocities(lattice)
        self.w = w
        self.D, self.tau, self.shape = DIM[lattice], tau, shape
        self.walls = [a in walls for a in "xyz"]
        h = (lambda v: 1.0, lambda v: float(v), lambda v: v * v - 1.0 / 3.0)
        pw = lambda n: [(a, b, e) for a in range(3) for b in range(3) for e in range(3 if self.D == 3 else 1)
                        if a + b + e <= n and (lattice != "D3Q19" or 0 in (a, b, e))]

        def projection(n):  # populations whose moments on the kept polynomials are the coefficients
            ks = pw(n)
            H = np.array([[h[a](v[0]) * h[b](v[1]) * h[e](v[2]) for (a, b, e) in ks] for v in self.c])
            gram = H.T @ (np.array(w)[:, None] * H)
            return ks, torch.from_numpy(np.array(w)[:, None] * (H @ np.linalg.inv(gram))).cuda()

        self.k0, self.P0 = projection(order)
        self.k1, self.P1 = projection(min(order, 3) if lattice == "D3Q19" else order)

    def post(self, rho, u, A):
        """f0(rho, u) + (1 - 1/tau) f1(u, A); A maps sorted index pairs to a1^(2) (None: zero)."""
        n = rho.numel()
        flat = lambda v: v.reshape(n)
        up = [[torch.ones(n, device="cuda", dtype=torch.float64), flat(u[a]), flat(u[a]) ** 2] if a < self.D else None
              for a in range(3)]

        def power(k):
            out = None
            for a in range(self.D):
                if k[a]:
                    out = up[a][k[a]] if out is None else out * up[a][k[a]]
            return up[0][0] if out is None else out

        C = torch.stack([flat(rho) * power(k) for k in self.k0])
        f = torch.mm(self.P0, C)
        del C
        if A is not None:
            rows = []
            for k in self.k1:
                s = torch.zeros(n, device="cuda", dtype=torch.float64)
                for a in range(self.D):
                    for b in range(a, self.D):
                        r = list(k)
                        r[a] -= 1
                        r[b] -= 1
                        if min(r) < 0:
                            continue
                        mult = k[a] * (k[a] - 1) / 2 if a == b else k[a] * k[b]
                        s += mult * flat(A[a, b]) * power(r)
                rows.append(s)
            f += (1.0 - 1.0 / self.tau) * torch.mm(self.P1, torch.stack(rows))
        return f.view((len(self.c),) + tuple(rho.shape))

    def moments(self, f):
        rho = f.sum(0)
        j = [sum(v[a] * f[i] for i, v in enumerate(self.c) if v[a]) for a in range(self.D)]
        return rho, [ja / rho for ja in j]

    def stress(self, f, rho, u):
        out = {}
        for a in range(self.D):
            for b in range(a, self.D):
                s = sum(v[a] * v[b] * f[i] for i, v in enumerate(self.c) if v[a] * v[b])
                out[a, b] = s - rho * u[a] * u[b] - (rho / 3.0 if a == b else 0.0)
        return out

    def pulled(self, g, z0, z1):
        nz = self.shape[0]
        f = torch.empty((len(self.c), z1 - z0) + tuple(self.shape[1:]), device="cuda", dtype=torch.float64)
        for i, (cx, cy, cz) in enumerate(self.c):
            zs = (torch.arange(z0, z1, device="cuda") - cz) % nz
            f[i] = torch.roll(g[i][zs], (cy, cx), (1, 2))
        return f

    def at_walls(self, f, z0, z1):
        """Wall nodes of a streamed slab: (mask, rho, a1^(2)) of the completed sets at u = 0."""
        nz, ny, nx = self.shape
        pos = (torch.arange(nx, device="cuda").view(1, 1, -1), torch.arange(ny, device="cuda").view(1, -1, 1),
               torch.arange(z0, z1, device="cuda").view(-1, 1, 1))
        full = torch.zeros((z1 - z0, ny, nx), device="cuda", dtype=torch.bool)

        def outside(v):
            m = full
            for walled, p, cc, n in zip(self.walls, pos, v, (nx, ny, nz)):
                if walled and cc:
                    m = m | (p == (0 if cc > 0 else n - 1))
            return m

        opp = [self.c.index((-v[0], -v[1], -v[2])) for v in self.c]
        unk = [outside(v) for v in self.c]
        s, wb = torch.zeros_like(f[0]), torch.zeros_like(f[0])
        for i in range(len(self.c)):
            bounced, buried = unk[i] & ~unk[opp[i]], unk[i] & unk[opp[i]]
            s += torch.where(~unk[i], f[i], torch.where(bounced, f[opp[i]], 0.0))
            wb += self.w[i] * buried
        rho = s / (1.0 - wb)
        A = {(a, b): torch.zeros_like(rho) for a in range(self.D) for b in range(a, self.D)}
        wall = full.clone()
        for i, v in enumerate(self.c):
            wall |= unk[i]
            bounced = unk[i] & ~unk[opp[i]]
            neq = torch.where(~unk[i], f[i] - self.w[i] * rho, torch.where(bounced, f[opp[i]] - self.w[i] * rho, 0.0))
            for (a, b) in A:
                if v[a] * v[b]:
                    A[a, b] += v[a] * v[b] * neq
        return wall, rho, A

    def step(self, g, correct=None):
        nz = self.shape[0]
        slab = max(1, (1 << 22) // (self.shape[1] * self.shape[2]))
        out = torch.empty_like(g)
        for z0 in range(0, nz, slab):
            z1 = min(nz, z0 + slab)
            f = self.pulled(g, z0, z1)
            rho, u = self.moments(f)
            A = self.stress(f, rho, u)
            if correct is not None:
                correct(g, f, A)
            if any(self.walls):
                wall, rw, Aw = self.at_walls(f, z0, z1)
                rho = torch.where(wall, rw, rho)
                u = [torch.where(wall, 0.0, ua) for ua in u]
                A = {k: torch.where(wall, Aw[k], A[k]) for k in A}
            out[:, z0:z1] = self.post(rho, u, A)
        return out

    def start(self, rho, u, pi1=None):
        nz = self.shape[0]
        slab = max(1, (1 << 22) // (self.shape[1] * self.shape[2]))
        g = torch.empty((len(self.c),) + tuple(self.shape), device="cuda", dtype=torch.float64)
        for z0 in range(0, nz, slab):
            z1 = min(nz, z0 + slab)
            g[:, z0:z1] = self.post(rho[z0:z1], [u[a, z0:z1] for a in range(self.D)],
                                    None if pi1 is None else {k: v[z0:z1] for k, v in pi1.items()})
        return g


def _derivative(a, dim, walled):
    d = 0.5 * (torch.roll(a, -1, dim) - torch.roll(a, 1, dim))
    if walled:
        n = a.shape[dim]
        e = lambda k: a.narrow(dim, k, 1)
        d.narrow(dim, 0, 1).copy_(0.5 * (-3.0 * e(0) + 4.0 * e(1) - e(2)))
        d.narrow(dim, n - 1, 1).copy_(0.5 * (3.0 * e(n - 1) - 4.0 * e(n - 2) + e(n - 3)))
    return d


def _enstrophy(u, walls):
    dim = {"x": 2, "y": 1, "z": 0}
    dd = lambda a, axis: _derivative(a, dim[axis], axis in walls)
    if len(u) == 2:
        w2 = (dd(u[1], "x") - dd(u[0], "y")) ** 2
    else:
        w2 = ((dd(u[2], "y") - dd(u[1], "z")) ** 2 + (dd(u[0], "z") - dd(u[2], "x")) ** 2
              + (dd(u[1], "x") - dd(u[0], "y")) ** 2)
    vol = 1.0
    for axis in "xyz"[: len(u)]:
        n = w2.shape[dim[axis]]
        vol *= n - 1 if axis in walls else n
        if axis in walls:
            w2.narrow(dim[axis], 0, 1).mul_(0.5)
            w2.narrow(dim[axis], n - 1, 1).mul_(0.5)
    return float(0.5 * w2.sum() / vol)


def _mlp64(params, norm, x):
    """Normalised outputs and activations of the network in FP64."""
    P, o, parts = params.double(), 0, []
    for rows, cols in ((64, 36), (64, 64), (3, 64)):
        parts.append((P[o:o + rows * cols].view(rows, cols), P[o + rows * cols:o + rows * cols + rows]))
        o += rows * cols + rows
    n = norm.double()
    xn = (x.double() - n[:36]) / n[36:72]
    z1 = torch.mm(xn, parts[0][0].t().contiguous()) + parts[0][1]
    h1 = torch.nn.functional.gelu(z1)
    z2 = torch.mm(h1, parts[1][0].t().contiguous()) + parts[1][1]
    h2 = torch.nn.functional.gelu(z2)
    y = torch.mm(h2, parts[2][0].t().contiguous()) + parts[2][1]
    return y, (xn, z1, h1, z2, h2, parts)


def _gelu_slope(z):
    return 0.5 * (1.0 + torch.erf(z / math.sqrt(2.0))) + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)


def _box(a, f):
    ny, nx = a.shape[-2:]
    return a.reshape(a.shape[:-2] + (ny // f, f, nx // f, f)).mean((-3, -1))


def _coarse64(rho, u, A, f, alpha, beta):
    rc = _box(rho, f)
    uc = [_box(rho * ua, f) / rc for ua in u]
    return rc, torch.stack(uc), {(a, b): alpha * _box(A[a, b], f) + beta * (_box(rho * u[a] * u[b], f) - rc * uc[a] * uc[b])
                                 for (a, b) in A}


def _features64(lat, g, f):
    """The 36 features (one row per node) of pulled populations f from the stored populations g."""
    w = torch.tensor(lat.w, device="cuda", dtype=torch.float64).view(9, 1, 1, 1)
    rho, u = lat.moments(g)
    cols = [v for v in (f - w)]
    for dy in (-1, 0, 1):
        for dx in (-1, 0, 1):
            cols += [torch.roll(v, (-dy, -dx), (1, 2)) for v in (rho - 1.0, u[0], u[1])]
    return torch.stack([c.reshape(-1) for c in cols], 1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "flow":
        rho, u = _initial(case, seed)
        shape = (case["nz"], case["ny"], case["nx"])
        lat = _Plain(case["lattice"], case["order"], case["tau"], shape, case["walls"])
        if shape[0] * shape[1] * shape[2] * case["steps"] > 2_000_000_000:
            return None
        g = lat.start(rho, u)
        del rho, u
        for _ in range(case["steps"]):
            g = lat.step(g)
        if case["read"] == "populations" and not case["storage"].startswith("mom"):
            for i, w in enumerate(lat.w):
                g[i] -= w
            return {"populations": g}
        rho, u = lat.moments(g)
        out = {"rho": rho, "u": torch.stack(u)}
        if case["read"] == "monitor":
            j = [float((rho * ua).sum()) for ua in u] + [0.0] * (3 - lat.D)
            out["totals"] = np.array([float(rho.sum())] + j + [float(0.5 * (rho * sum(ua * ua for ua in u)).sum())])
            out["enstrophy"] = _enstrophy(u, case["walls"])
        return out
    if kind == "coarse_run":
        rho, u = _vorticity_fields(case["ny"], case["n"], 0.1, seed)
        params, norm = _network(np.random.default_rng(seed))
        lat = _Plain("D2Q9", case["order"], TAU_COARSE, (1, case["ny"], case["n"]), "")
        n = norm.double()

        def correct(g, f, A):
            y = _mlp64(params, norm, _features64(lat, g, f))[0] * n[75:78] + n[72:75]
            for k, pair in enumerate(((0, 0), (0, 1), (1, 1))):
                A[pair] += y[:, k].view(A[pair].shape)

        g = lat.start(rho, u)
        for _ in range(case["steps"]):
            g = lat.step(g, correct)
        rho, u = lat.moments(g)
        return {"rho": rho, "u": torch.stack(u)}
    if kind == "coarse_data":
        ny, nx, f = case["ny"], case["n"], case["factor"]
        rho, u = _vorticity_fields(ny, nx, 0.1, seed)
        lat = _Plain("D2Q9", 4, TAU_FINE, (1, ny, nx), "")
        g = lat.start(rho, u)
        for _ in range(DATA_WARM):
            g = lat.step(g)
        om = 1.0 - 1.0 / TAU_FINE
        read = lambda: (lambda r, v: (r, v, {k: a / om for k, a in lat.stress(g, r, v).items()}))(*lat.moments(g))
        half = lambda tau: 1.0 - 0.5 / tau
        omc = 1.0 - 1.0 / TAU_COARSE
        rc, uc, pc = _coarse64(*read(), f, half(TAU_FINE) / half(TAU_COARSE), 0.0)
        for _ in range(f):
            g = lat.step(g)
        _, _, target = _coarse64(*read(), f, 0.0, (1.0 - omc) / omc)
        cl = _Plain("D2Q9", 4, TAU_COARSE, (1, ny // f, nx // f), "")
        gc = cl.start(rc, uc, pc)
        return {"features": _features64(cl, gc, cl.pulled(gc, 0, 1)),
                "labels": torch.stack([target[k].reshape(-1) for k in ((0, 0), (0, 1), (1, 1))], 1)}
    if kind == "train":
        x, t = _data_set(case["rows"], seed)
        rng = np.random.default_rng(seed + 1)
        params, _ = _network(rng)
        norm = _plain_norm(x, t)
        idx = torch.from_numpy(rng.integers(0, case["rows"], size=(case["steps"], case["batch"]), dtype=np.int32)).cuda()
        p = params.double()
        m, v, n = torch.zeros_like(p), torch.zeros_like(p), norm.double()
        for k in range(case["steps"]):
            rows = idx[k].long()
            tn = (t[rows].double() - n[72:75]) / n[75:78]
            y, (xn, z1, h1, z2, h2, parts) = _mlp64(p, norm, x[rows])
            loss = ((y - tn) ** 2).mean()
            dy = 2.0 * (y - tn) / y.numel()
            dz2 = torch.mm(dy, parts[2][0]) * _gelu_slope(z2)
            dz1 = torch.mm(dz2, parts[1][0]) * _gelu_slope(z1)
            mt = lambda a, b: torch.mm(a.t().contiguous(), b).reshape(-1)
            g = torch.cat([mt(dz1, xn), dz1.sum(0), mt(dz2, h1), dz2.sum(0), mt(dy, h2), dy.sum(0)])
            m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
            p = p - 1e-3 * (m / (1 - 0.9 ** (k + 1))) / (torch.sqrt(v / (1 - 0.999 ** (k + 1))) + 1e-8)
        return {"params": p, "loss": loss.reshape(1)}
    x, t = _data_set(case["rows"], seed)
    params, _ = _network(np.random.default_rng(seed + 1))
    norm = torch.cat([x.double().mean(0), x.double().std(0, unbiased=False), t.double().mean(0),
                      t.double().std(0, unbiased=False)])
    y = _mlp64(params, norm, x)[0] * norm[75:78] + norm[72:75]
    return {"norm": norm, "y": y}
