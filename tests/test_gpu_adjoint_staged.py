"""The adjoint sweep's staged kernel (FP32 volumes of at least 2^20 voxels with
relative codes) against the direct one (the table, VG_KERNEL_TABLE) on the same
recorded states: the initial state's adjoint is bit-identical (the same
operations per voxel), and the parameter derivatives differ only by the order
of FP64 sums of equal terms: 1e-12 of each sum's terms, taken as 1e-9 of its
value for sums whose terms cancel by up to three orders (tolerances set before
the first run).  The sizes put the last tile at a full one, one voxel, one
short of full and a ragged remainder; a batch crosses tiles with volumes."""
import numpy as np
import pytest
import torch

from paper_2406_04177_amd import _lib, inputs

pytestmark = pytest.mark.gpu

NMIN, TILE = 1 << 20, 1024


def volume(n, nx=120, ny=110):
    nz = -(-int(n / 0.9) // (nx * ny)) + 1
    order = np.random.default_rng(n).permutation(nz * ny * nx)
    mask = np.zeros(nz * ny * nx, np.uint8)
    mask[order[:n]] = 1
    return mask.reshape(nz, ny, nx)


@pytest.mark.parametrize("tape_dom", [False, True], ids=["states", "tape_dom"])
@pytest.mark.parametrize("regions,skip", [(False, True), (False, False), (True, False)],
                         ids=["unit-dom_d", "unit-all_d", "regions-all_d"])
@pytest.mark.parametrize("n", [NMIN, NMIN + 1, NMIN + TILE - 1, NMIN + 300, 0], ids=["full", "one", "short", "ragged",
                                                                                      "batch"])
def test_staged_equals_direct(n, regions, skip, tape_dom):
    from paper_2406_04177_amd.graph import Graph
    from paper_2406_04177_amd.sim import Simulation
    masks = [volume(n)] if n else [volume(350000 + 17 * b, 60, 80)[:98] for b in range(4)]
    g = Graph.from_masks(masks, regions=regions)
    assert g.n >= NMIN
    p = inputs.ModelParams(v_dom=0.02, rho=0.005, mu=0.004, v_som=0.01, v_p4=0.02)
    dt = inputs.explicit_dt(p, 0.8)
    gen = torch.Generator(device="cuda").manual_seed(3)
    x0 = torch.rand((5, g.n), generator=gen, device="cuda", dtype=torch.float32)
    k = 3
    seeds = torch.rand((k, len(masks), 5), generator=gen, device="cuda", dtype=torch.float64)
    out = []
    for kernel in (_lib.VG_KERNEL_TABLE, _lib.VG_KERNEL_RELATIVE):
        sim = Simulation(g, p, precision="f32", implicit=False, adjoint=True, regions=[1.0] * 8 if regions else None)
        sim.set_kernel(kernel)
        sim.set_adjoint_options(skip_static_d=skip, tape_dom=tape_dom)
        sim.set_fields(x0)
        states = torch.empty((k, sim.tape_rows, g.n), dtype=torch.float32, device="cuda")
        sim.record(k, dt, states)
        lam = torch.empty((5, g.n), dtype=torch.float32, device="cuda")
        grad = torch.zeros(20, dtype=torch.float64, device="cuda")
        sim.seed_lambda(seeds[0], lam, zero=True)
        sim.adjoint(k, dt, states, seeds, lam, grad)
        out.append((lam, torch.nan_to_num(grad, nan=7.0)))
    (l0, g0), (l1, g1) = out
    assert torch.equal(l0, l1)
    assert float(((g0 - g1).abs() / g0.abs().clamp_min(1e-300)).max()) <= 1e-9
