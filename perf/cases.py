"""The work a user of this framework has it do, as cases that can be timed.

Each case goes through the package's public entry points (``Simulation``,
``autograd.simulate_totals``, ``graph.range_sums``) on a seeded synthetic pore
volume: uniform noise smoothed by a Gaussian of sigma = 2 voxels and thresholded
at a porosity, the recipe of ``inputs.synthetic_volume`` carried out on the
GPU (every pore is kept, isolated ones too).  Kinds of a case:

  step       ``Simulation.step``: explicit time steps, mass totals logged
  subcycled  ``Simulation.step_subcycled``: unequal transformation and
             diffusion steps, Algorithm 2
  network    voxel-method data for the pore-network fit: steps on a
             brick-ordered volume, then the mass of every brick
  implicit   ``Simulation.implicit_step``, diagonal or multigrid preconditioner
  gradient   a loss on the CO2 curve and its gradient: forward and adjoint
"""
import math

import numpy as np
import torch

from paper_2406_04177_amd import autograd, diffusion_experiment, inputs, pngm
from paper_2406_04177_amd.graph import Graph, range_sums
from paper_2406_04177_amd.sim import Simulation

DEV = "cuda"
DTYPE = {"f32": torch.float32, "f64": torch.float64, "f32c": torch.float32}
# Algorithm 1 costs about this many operations per voxel, diffusion of one pool 13, the reverse step 110
T_FLOPS, D_FLOPS, REV_FLOPS = 32, 13, 110


def listed():
    base = {"vols": 1, "porosity": 0.17, "brick": 0, "init": "workload"}
    return [
        # the parity-size run of the smallest workload: launches and latency count
        dict(base, name="step_48_f64", kind="step", nz=48, ny=48, nx=48, precision="f64", init="spots", steps=100,
             log_every=50),
        # the medium workload: fits the last-level cache
        dict(base, name="step_256_f32", kind="step", nz=256, ny=256, nx=256, precision="f32", steps=100, log_every=100),
        # the full-size workload in a short call, as between two outputs of a run
        dict(base, name="step_512_f32", kind="step", nz=512, ny=512, nx=512, precision="f32", steps=20, log_every=20),
        # the same volume with the fields that hold 1e-5 over long runs
        dict(base, name="step_512_f32c", kind="step", nz=512, ny=512, nx=512, precision="f32c", steps=10, log_every=10),
        # a cut-out of no round size at the reference precision, every pool occupied (a restarted run), frequent totals
        dict(base, name="step_ragged_f64", kind="step", nz=331, ny=257, nx=403, precision="f64", init="dense", steps=33,
             log_every=11),
        # the paper's test 3: diffusion steps 4.3 times shorter than the transformation's; the sequential algorithm
        dict(base, name="subcycled_ragged_f32", kind="subcycled", nz=301, ny=290, nx=277, precision="f32", init="dense",
             steps=8, ratio=4.3),
        # training data of the pore-network fit: one record of the full-size volume in bricks of 16
        dict(base, name="network_512_f64", kind="network", nz=512, ny=512, nx=512, precision="f64", brick=16,
             init="scenario", steps=10),
        # one implicit step at 20 times the explicit bound, the paper's preconditioner
        dict(base, name="implicit_512_f32", kind="implicit", nz=512, ny=512, nx=512, precision="f32", factor=20.0,
             multigrid=False),
        # one 30 s step of the z-layer experiment, multigrid preconditioner
        dict(base, name="layers_512_f64_mg", kind="implicit", nz=512, ny=512, nx=512, precision="f64", init="layers",
             factor=0.0, multigrid=True),
        # an epoch of the parameter fit, shortened: a batch of volumes with region factors, every derivative
        dict(base, name="gradient_16x128_f32", kind="gradient", vols=16, nz=128, ny=128, nx=128, precision="f32",
             regions=True, steps=40, every=20, static=True),
        # the gradient of the full-size volume: uniform conductances, static pools' D left out
        dict(base, name="gradient_512_f32", kind="gradient", nz=512, ny=512, nx=512, precision="f32", regions=False,
             steps=12, every=12, static=False),
        # a small fit in double precision: launches and host work count
        dict(base, name="gradient_4x40_f64", kind="gradient", vols=4, nz=40, ny=44, nx=38, precision="f64",
             regions=True, steps=24, every=12, static=True),
    ]


def _edge(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Sizes spread over their logarithm, odd ones among them; every kind, precision and option of the listed cases."""
    kind = rng.choice(["step", "step", "step", "subcycled", "network", "implicit", "implicit", "gradient", "gradient"])
    e = _edge(rng, 40, 420)
    dims = [max(24, min(512, int(round(e * rng.uniform(0.8, 1.2))))) for _ in range(3)]
    c = {"kind": kind, "vols": 1, "nz": dims[0], "ny": dims[1], "nx": dims[2], "brick": 0,
         "porosity": round(rng.uniform(0.12, 0.25), 3), "precision": rng.choice(["f32", "f64"]), "init": "workload"}
    if kind == "step":
        c["precision"] = rng.choice(["f32", "f32", "f64", "f64", "f32c"])
        c["init"] = rng.choice(["workload", "dense"])
        c["steps"] = rng.randint(5, 40)
        c["log_every"] = rng.choice([0, c["steps"], max(1, c["steps"] // 3)])
    elif kind == "subcycled":
        c.update(init="dense", steps=rng.randint(3, 8), ratio=round(rng.uniform(1.5, 5.0), 2))
    elif kind == "network":
        c.update(precision="f64", brick=rng.choice([8, 16]), init="scenario", steps=rng.randint(5, 12))
    elif kind == "implicit":
        c["multigrid"] = rng.random() < 0.5
        c["factor"] = 0.0 if rng.random() < 0.3 else round(rng.uniform(2.0, 40.0), 1)
        c["init"] = "layers" if c["factor"] == 0.0 else "workload"
    else:
        c["vols"] = rng.choice([1, 1, 4, 8]) if e < 150 else 1
        c["regions"] = c["vols"] > 1 or rng.random() < 0.5
        c["static"] = rng.random() < 0.5
        c["steps"] = rng.randint(6, 16)
        c["every"] = rng.randint(4, 16)
    return c


# ------------------------------------------------------------------ inputs
def _mask(shape, porosity, seed):
    """Pore mask on the GPU: the round(porosity * voxels) smallest values of smoothed noise."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    x = torch.rand(shape, generator=gen, device=DEV, dtype=torch.float32)
    k = np.exp(-0.5 * (np.arange(-8, 9) / 2.0) ** 2)
    k /= k.sum()
    for axis in range(3):
        n = x.shape[axis]
        m = min(8, n)
        p = torch.cat([x.narrow(axis, 0, m).flip(axis), x, x.narrow(axis, n - m, m).flip(axis)], axis)
        x = torch.zeros_like(x)
        for j, w in enumerate(k):
            x.add_(p.narrow(axis, j, n), alpha=float(w))
    flat = x.reshape(-1)
    k = max(1, int(round(porosity * flat.numel())))
    t = flat.sort().values[k - 1]
    pore = flat < t
    ties = torch.nonzero(flat == t).reshape(-1)
    pore[ties[: k - int(pore.sum())]] = True    # exactly k pores
    return pore.to(torch.uint8).reshape(shape)


def _masks(case, seed):
    shape = (case["nz"], case["ny"], case["nx"])
    return [_mask(shape, case["porosity"], 1000 * int(seed) + b) for b in range(case["vols"])]


def _order(mask, brick):
    """Linear indices of the pore voxels in the order of the compacted list: raster, or brick by brick."""
    lin = torch.nonzero(mask.reshape(-1)).reshape(-1)
    if not brick:
        return lin
    nz, ny, nx = mask.shape
    x, y, z = lin % nx, (lin // nx) % ny, lin // (nx * ny)
    nbx, nby = -(-nx // brick), -(-ny // brick)
    blk = (z // brick * nby + y // brick) * nbx + x // brick
    return lin[torch.argsort(blk * brick ** 3 + ((z % brick) * brick + y % brick) * brick + x % brick)]


def _fields(case, masks, seed):
    """[5, n] FP64 initial masses, one volume after the other in the order of the compacted list."""
    parts = []
    for b, mask in enumerate(masks):
        lin = _order(mask, case["brick"])
        n = lin.numel()
        gen = torch.Generator(device=DEV).manual_seed(7000003 + 1000 * int(seed) + b)

        def rnd(size):
            return torch.rand(size, generator=gen, device=DEV, dtype=torch.float64)

        x = torch.zeros((5, n), dtype=torch.float64, device=DEV)
        some = torch.randint(n, (100,), generator=gen, device=DEV)
        if case["init"] == "dense":
            x = rnd((5, n)) * torch.tensor([0.5, 1.0, 0.3, 0.2, 0.1], dtype=torch.float64, device=DEV)[:, None]
        elif case["init"] == "spots":
            x[1, some[:50]] = 1.0
            x[0, some] = 0.5
        elif case["init"] == "scenario":
            u = rnd(n)
            x[1] = torch.where(u < 0.01, u, 0.0)
            x[1] /= x[1].sum()
        elif case["init"] == "layers":
            low = lin < 2 * mask.shape[1] * mask.shape[2]
            x[1] = torch.where(low, diffusion_experiment.M0 / low.sum().clamp(min=1), 0.0)
        else:
            u = rnd(n)
            x[1] = torch.where(u < 0.005, u * 200.0, 0.0)
            x[0, some] = 0.5
        parts.append(x)
    return torch.cat(parts, 1)


def _params(case):
    if case["kind"] == "network":
        return pngm.pngm_params()
    if case["init"] == "layers":
        return diffusion_experiment.params()
    return inputs.ModelParams(sequential=case["kind"] == "subcycled")


def _dt(case, p):
    if case["kind"] == "network":
        return 0.1
    if case["kind"] == "implicit":
        return 30.0 if case["init"] == "layers" else inputs.explicit_dt(p, case["factor"])
    return inputs.explicit_dt(p, 0.8 if case["kind"] == "gradient" else 0.9)


def _target(case, p, dt, x0, counts):
    """[steps + 1, volumes] CO2 curve a tenth above what the first biomass respires."""
    mb = torch.stack([v.sum() for v in x0[0].split(counts)])
    k = torch.arange(case["steps"] + 1, dtype=torch.float64, device=DEV)
    return 1.1 * p.rho * dt * k[:, None] * mb[None, :]


def prepare(case, seed):
    masks = _masks(case, seed)
    x0 = _fields(case, masks, seed)
    counts = [int(m.sum()) for m in masks]
    g = Graph.from_masks([m.cpu().numpy() for m in masks], brick=case["brick"])
    p = _params(case)
    kind = case["kind"]
    opts = {"implicit": kind == "implicit"}
    if kind == "implicit":
        opts["multigrid"] = case["multigrid"]
    if kind == "gradient":
        opts["adjoint"] = True
        opts["regions"] = [1.0] * 8 if case["regions"] else None
    sim = Simulation(g, p, precision=case["precision"], **opts)
    s = {"case": case, "sim": sim, "dt": _dt(case, p), "p": p}
    if kind == "gradient":
        s["x0"] = x0.to(DTYPE[case["precision"]])
        s["theta"] = autograd.theta_of(p)
        s["target"] = _target(case, p, s["dt"], x0, counts)
        if not case["static"]:
            sim.set_adjoint_options(skip_static_d=True)
        return s
    if kind == "implicit":
        s["x0"] = x0.to(DTYPE[case["precision"]])
        if case["multigrid"]:
            sim.set_preconditioner("mg")
        return s
    sim.set_fields(x0)
    if kind == "network":
        bricks = -(-case["nx"] // case["brick"]), -(-case["ny"] // case["brick"]), -(-case["nz"] // case["brick"])
        lin = _order(masks[0], case["brick"])
        x, y, z = lin % case["nx"], (lin // case["nx"]) % case["ny"], lin // (case["nx"] * case["ny"])
        b = case["brick"]
        blk = (z // b * bricks[1] + y // b) * bricks[0] + x // b
        cnt = torch.bincount(blk, minlength=bricks[0] * bricks[1] * bricks[2])
        cnt = cnt[cnt > 0]
        s["offsets"] = torch.cat([cnt.new_zeros(1), cnt.cumsum(0)])
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    case, sim = s["case"], s["sim"]
    kind = case["kind"]
    if kind == "step":
        log = sim.step(case["steps"], s["dt"], log_every=case["log_every"])
        return {"fields": sim.fields, "log": log}
    if kind == "subcycled":
        sim.step_subcycled(case["steps"], case["ratio"] * s["dt"], s["dt"])
        return {"fields": sim.fields}
    if kind == "network":
        sim.step(case["steps"], s["dt"])
        return {"fields": sim.fields, "masses": range_sums(sim.fields[1], s["offsets"])}
    if kind == "implicit":
        sim.set_fields(s["x0"])
        sim.implicit_step(s["dt"])
        return {"fields": sim.fields}
    theta = s["theta"].clone().requires_grad_(True)
    x0 = s["x0"].detach().requires_grad_(True)
    tot = autograd.simulate_totals(sim, theta, x0, case["steps"], s["dt"], case["every"])
    loss = autograd.co2_mse(tot, s["target"])
    loss.backward()
    return {"totals": tot.detach(), "loss": loss.detach(), "theta": theta.grad, "x0": x0.grad}


def work(case):
    n = case["vols"] * case["porosity"] * case["nz"] * case["ny"] * case["nx"]
    e = {"f32": 4, "f64": 8, "f32c": 6}[case["precision"]]
    state, graph = 5 * e * n, 4 * n
    kind = case["kind"]
    flops = case.get("steps", 1) * n * (T_FLOPS + D_FLOPS)
    if kind == "subcycled":
        flops = case["steps"] * n * (T_FLOPS + math.ceil(case["ratio"]) * D_FLOPS)
    if kind == "gradient":
        flops = case["steps"] * n * (T_FLOPS + D_FLOPS + REV_FLOPS)
    return {"bytes": 2 * state + graph, "flops": flops}


# ------------------------------------------------------------------ 64 bits
def _least(a, b):
    """a clamped to b; at equality the derivative is a's, as the clamps' strict > has it."""
    return torch.where(a > b, b, a)


class _Exact:
    """The method in plain torch, FP64: neighbours by index, Scheme 1, Algorithms 1 and 2."""

    def __init__(self, case, masks, p):
        self.p = p
        nbr, off = [], 0
        for mask in masks:
            lin = _order(mask, case["brick"])
            nz, ny, nx = mask.shape
            idx = torch.full((nz + 2, ny + 2, nx + 2), -1, dtype=torch.int64, device=DEV)
            x, y, z = lin % nx + 1, (lin // nx) % ny + 1, lin // (nx * ny) + 1
            own = torch.arange(lin.numel(), device=DEV) + off
            idx[z, y, x] = own
            js = []
            for dz, dy, dx in ((0, 0, -1), (0, 0, 1), (0, -1, 0), (0, 1, 0), (-1, 0, 0), (1, 0, 0)):
                j = idx[z + dz, y + dy, x + dx]
                js.append(torch.where(j < 0, own, j))
            nbr.append(torch.stack(js))
            off += lin.numel()
            del idx
        self.nbr = torch.cat(nbr, 1)
        self.counts = [int(m.sum()) for m in masks]
        if case.get("regions"):
            octs = []
            for mask in masks:
                lin = _order(mask, case["brick"])
                nz, ny, nx = mask.shape
                octs.append(4 * (lin // (nx * ny) >= nz // 2) + 2 * ((lin // nx) % ny >= ny // 2) + 1 * (lin % nx >= nx // 2))
            self.oct = torch.cat(octs)
        else:
            self.oct = None

    def lap(self, u, c=None):
        s = torch.zeros_like(u)
        for k in range(6):
            d = u.index_select(0, self.nbr[k]) - u
            if c is not None:
                d = d * (0.5 * (c[self.oct] + c[self.oct.index_select(0, self.nbr[k])]))
            s = s + d
        return s

    def diffuse(self, x, dt, D=None, c=None, all_pools=False):
        """Scheme 1; with all_pools every pool takes its own D (also where that is 0, for its derivative)."""
        D = self.p.D if D is None else D
        rows = []
        for s in range(5):
            if s == 1 or all_pools:
                rows.append(x[s] + (D[s] * dt / self.p.h ** 2) * self.lap(x[s], c))
            else:
                rows.append(x[s])
        return torch.stack(rows)

    def transform(self, x, dt, v=None):
        p = self.p
        vd, kd, rho, mu, beta, vs, vp = v if v is not None else (p.v_dom, p.k_dom, p.rho, p.mu, p.beta, p.v_som, p.v_p4)
        m1, m2, m3, m4, m5 = x
        if p.sequential:
            up = torch.where((m1 > 0) & (m2 > 0), _least(vd * m2 / (kd + m2) * m1 * dt, m2), torch.zeros_like(m2))
            m1, m2 = m1 + up, m2 - up
            dead = _least(mu * m1 * dt, m1)
            m1, m2, m3 = m1 - dead, m2 + beta * dead, m3 + (1 - beta) * dead
            resp = _least(rho * m1 * dt, m1)
            m1, m5 = m1 - resp, m5 + resp
            ts = _least(vs * m3 * dt, m3)
            m3, m2 = m3 - ts, m2 + ts
            tp = _least(vp * m4 * dt, m4)
            return torch.stack([m1, m2 + tp, m3, m4 - tp, m5])
        up = _least(vd * m2 / (kd + m2) * m1 * dt, m2)
        resp, mort = rho * m1 * dt, mu * m1 * dt
        over = resp + mort > m1
        allm = over & (mort > m1)
        resp = torch.where(allm, torch.zeros_like(m1), torch.where(over, m1 - mort, resp))
        mort = torch.where(allm, m1, mort)
        tp = _least(vp * m4 * dt, m4)
        ts = _least(vs * m3 * dt, m3)
        return torch.stack([m1 + (up - mort - resp), m2 + (beta * mort - up + tp + ts), m3 + ((1 - beta) * mort - ts),
                            m4 - tp, m5 + resp])

    def totals(self, x):
        t = torch.stack([torch.stack([v.sum() for v in x[s].split(self.counts)]) for s in range(5)], 1)
        return t

    def solve(self, b, a):
        """(I - a lap) y = b by conjugate gradients to rounding."""
        deg = sum((self.nbr[k] != torch.arange(b.numel(), device=DEV)).to(torch.float64) for k in range(6))
        minv = 1.0 / (1.0 + a * deg)
        y = b.clone()
        r = b - (y - a * self.lap(y))
        z = minv * r
        q = z.clone()
        rz = float(r @ z)
        stop = 1e-15 * float(b.norm())
        for _ in range(2000):
            if float(r.norm()) <= stop:
                break
            w = q - a * self.lap(q)
            al = rz / float(q @ w)
            y += al * q
            r -= al * w
            z = minv * r
            new = float(r @ z)
            q = z + (new / rz) * q
            rz = new
        return y


@torch.no_grad()
def exact(case, seed):
    masks = _masks(case, seed)
    x0 = _fields(case, masks, seed)
    p = _params(case)
    dt = _dt(case, p)
    E = _Exact(case, masks, p)
    kind = case["kind"]
    x = x0
    if kind in ("implicit", "gradient", "step", "subcycled") and case["precision"] == "f32":
        x = x0.float().double()     # what the fields hold
    if kind == "step" or kind == "network":
        every = case.get("log_every", 0)
        log = []
        for k in range(1, case["steps"] + 1):
            x = E.diffuse(E.transform(x, dt), dt)
            if every and k % every == 0:
                t = E.totals(x)
                log.append(torch.cat([t, t.sum(1, keepdim=True)], 1))
        if kind == "step":
            return {"fields": x, "log": torch.stack(log) if log else None}
        bricks = [-(-case[d] // case["brick"]) for d in ("nx", "ny", "nz")]
        lin, b = _order(masks[0], case["brick"]), case["brick"]
        vx, vy, vz = lin % case["nx"], (lin // case["nx"]) % case["ny"], lin // (case["nx"] * case["ny"])
        blk = (vz // b * bricks[1] + vy // b) * bricks[0] + vx // b
        total = bricks[0] * bricks[1] * bricks[2]
        cnt = torch.bincount(blk, minlength=total)
        return {"fields": x, "masses": torch.bincount(blk, weights=x[1], minlength=total)[cnt > 0]}
    if kind == "subcycled":
        dt_t, end, kt, kd = case["ratio"] * dt, case["steps"] * (case["ratio"] * dt), 0, 0
        while kt < case["steps"] or kd * dt < end:
            if kt < case["steps"] and (not kd * dt < end or kt * dt_t <= kd * dt):
                x = E.transform(x, dt_t)
                kt += 1
            else:
                x = E.diffuse(x, dt if (kd + 1) * dt <= end else end - kd * dt)
                kd += 1
        return {"fields": x}
    if kind == "implicit":
        x = E.transform(x, dt)
        x[1] = E.solve(x[1], p.D[1] * dt / p.h ** 2)
        return {"fields": x}
    return _exact_gradient(case, E, x, p, dt)


def _exact_gradient(case, E, x0, p, dt):
    theta = autograd.theta_of(p).to(DEV)

    def step(x, th):
        c = th[12:20] if E.oct is not None else None
        return E.diffuse(E.transform(x, dt, th[5:12]), dt, th[0:5], c, all_pools=case["static"])

    xs = [x0]
    for _ in range(case["steps"]):
        xs.append(step(xs[-1], theta))
    tot = torch.stack([E.totals(x) for x in xs])
    target = _target(case, p, dt, x0, E.counts)
    diff = tot[:, :, 4] - target
    loss = (diff ** 2).mean()
    seg = torch.repeat_interleave(torch.arange(len(E.counts), device=DEV), torch.tensor(E.counts, device=DEV))
    seed = 2.0 * diff / diff.numel()
    lam = torch.zeros_like(x0)
    lam[4] += seed[-1][seg]
    grad = torch.zeros_like(theta)
    for k in range(case["steps"] - 1, -1, -1):
        with torch.enable_grad():
            x = xs[k].detach().requires_grad_(True)
            th = theta.detach().requires_grad_(True)
            gx, gt = torch.autograd.grad(step(x, th), (x, th), lam)
        lam = gx
        lam[4] += seed[k][seg]
        grad += gt
        xs[k + 1] = None
    if not case["static"]:
        grad[[0, 2, 3, 4]] = math.nan       # left out on request
    return {"totals": tot, "loss": loss, "theta": grad.cpu(), "x0": lam}
