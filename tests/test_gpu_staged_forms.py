"""The kernels that stage tiles in LDS (reverse sweep and conjugate gradients)
against the direct ones (the table) over the forms they accept: distinct region
factors with pores on both sides of every mid-plane, halos of one wave up to a
whole block, batches, every field type, and the tile's edges where the staged
kernels start (2^21 voxels; 2^20 for the conjugate gradients).

Reverse sweep: the initial state's adjoint is bit-identical (the same
operations per voxel); a parameter derivative is a sum of the same FP64 terms
in another order, n terms of which cancel by up to four orders: 1e-8 of its
value.  Conjugate gradients: iterates differ by a few FP64 roundings per
iteration, amplified by at most the condition number (<= 41): 1e-12 of max |y|
after 7 iterations, plus the rounding to the field type (one spacing of FP32,
one of the compensated fields' 2^-39).  Tolerances set before the first run."""
import numpy as np
import pytest
import torch

from paper_2406_04177_amd import _lib, inputs

pytestmark = pytest.mark.gpu

REGIONS = [0.7, 1.0, 0.8, 0.9, 1.1, 0.75, 0.95, 0.85]
N2 = 1 << 21


def volume(n, nx, ny):
    """A random volume of exactly n pores (porosity 0.9: long runs and gaps)."""
    nz = -(-int(n / 0.9) // (nx * ny)) + 1
    order = np.random.default_rng(n).permutation(nz * ny * nx)
    mask = np.zeros(nz * ny * nx, np.uint8)
    mask[order[:n]] = 1
    return mask.reshape(nz, ny, nx)


# nx of 0.9 porosity: x and y distances up to 64, 128, 256
ROWS = {"halo64": (50, 60), "halo128": (120, 110), "halo256": (250, 50)}


def graph(n, row, volumes=1, regions=False):
    from paper_2406_04177_amd.graph import Graph
    nx, ny = ROWS[row]
    nz = volume(n // volumes, nx, ny).shape[0]
    masks = [volume(n // volumes + 17 * b, nx, ny)[:nz - 1] if volumes > 1 else volume(n, nx, ny)
             for b in range(volumes)]
    g = Graph.from_masks(masks, regions=regions)
    near = max(int((j - torch.arange(g.n, device="cuda", dtype=torch.int32)).max()) for j in (g.nbr[1], g.nbr[3]))
    lo, hi = {"halo64": (0, 64), "halo128": (65, 128), "halo256": (193, 256)}[row]
    assert lo < near <= hi, near
    return g


@pytest.mark.parametrize("tape_dom", [False, True], ids=["states", "tape_dom"])
@pytest.mark.parametrize("regions,skip", [(False, True), (True, False)], ids=["unit-dom_d", "regions-all_d"])
@pytest.mark.parametrize("n,row,volumes", [(N2, "halo128", 1), (N2 + 1, "halo64", 1), (N2 + 1023, "halo256", 1),
                                           (N2 + 4 * 30000 + 333, "halo128", 4)],
                         ids=["full", "one-halo64", "short-halo256", "batch"])
def test_reverse_sweep(n, row, volumes, regions, skip, tape_dom):
    from paper_2406_04177_amd.sim import Simulation
    g = graph(n, row, volumes, regions)
    assert g.n >= N2
    p = inputs.ModelParams(v_dom=0.02, rho=0.005, mu=0.004, v_som=0.01, v_p4=0.02)
    dt = inputs.explicit_dt(p, 0.8)
    gen = torch.Generator(device="cuda").manual_seed(3)
    x0 = torch.rand((5, g.n), generator=gen, device="cuda", dtype=torch.float32)
    k = 3
    seeds = torch.rand((k, volumes, 5), generator=gen, device="cuda", dtype=torch.float64)
    out = []
    for kernel in (_lib.VG_KERNEL_TABLE, _lib.VG_KERNEL_RELATIVE):
        sim = Simulation(g, p, precision="f32", implicit=False, adjoint=True, regions=REGIONS if regions else None)
        sim.set_kernel(kernel)
        sim.set_adjoint_options(skip_static_d=skip, tape_dom=tape_dom)
        sim.set_fields(x0)
        states = torch.empty((k, sim.tape_rows, g.n), dtype=torch.float32, device="cuda")
        sim.record(k, dt, states)
        lam = torch.empty((5, g.n), dtype=torch.float32, device="cuda")
        grad = torch.zeros(20, dtype=torch.float64, device="cuda")
        sim.seed_lambda(seeds[0], lam, zero=True)
        sim.adjoint(k, dt, states, seeds, lam, grad)
        out.append((lam, grad))
    (l0, g0), (l1, g1) = out
    assert torch.equal(l0, l1)
    assert torch.equal(torch.isnan(g0), torch.isnan(g1)) and bool(torch.isnan(g0).any()) == skip
    keep = ~torch.isnan(g0)
    if regions:
        assert bool((g0[12:20] != 0).all())
    assert float(((g0 - g1).abs() / g0.abs().clamp_min(1e-300))[keep].max()) <= 1e-8


@pytest.mark.parametrize("precision", ["f32", "f64", "f32c"])
@pytest.mark.parametrize("n,row,volumes", [((1 << 20) + 333, "halo64", 1), ((1 << 20) + 1023, "halo256", 1),
                                           ((1 << 20) + 4 * 20000 + 77, "halo128", 4)],
                         ids=["halo64", "halo256", "batch"])
def test_conjugate_gradients(n, row, volumes, precision):
    from paper_2406_04177_amd.sim import Simulation
    g = graph(n, row, volumes)
    assert g.n >= 1 << 20
    p = inputs.ModelParams()
    dt = 20 * inputs.explicit_dt(p, 1.0)
    x0 = torch.rand((5, g.n), generator=torch.Generator(device="cuda").manual_seed(5), device="cuda",
                    dtype=torch.float64)
    sim = Simulation(g, p, precision=precision, implicit=True)
    out = []
    for kernel in (_lib.VG_KERNEL_TABLE, _lib.VG_KERNEL_RELATIVE):
        sim.set_kernel(kernel)
        sim.set_fields(x0)
        its, _, rc = sim.implicit_step(dt, rtol=1e-30, max_iter=7, check=False)
        assert rc == _lib.VG_ENOCONV and its[1] == 7
        y7 = sim.state()[1]
        sim.set_fields(x0)
        its, rel, rc = sim.implicit_step(dt, rtol=1e-10)
        assert rc == 0 and rel[1] <= 1e-10
        out.append((y7, its[1]))
    (a, ia), (b, ib) = out
    assert abs(ia - ib) <= 1
    rounding = {"f32": 2.0 ** -23, "f64": 0.0, "f32c": 2.0 ** -38}[precision]
    assert float((a - b).abs().max()) <= (1e-12 + rounding) * float(a.abs().max())
