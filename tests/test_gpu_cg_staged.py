"""The conjugate-gradient kernels that stage a tile in LDS (large volumes with
relative codes and near x / y neighbours) against the direct ones (the table,
VG_KERNEL_TABLE) on the same volume: same iteration count within one, and
iterates stopped after k iterations equal up to rounding.  The sizes put the
last tile at a full tile, one voxel, one voxel short and a ragged remainder.

Tolerance, set before the first run: the two forms evaluate the same sums in
FP64 with other orders of the partial sums only, so an iterate differs by a
few roundings per iteration, amplified by at most the condition number
(<= 1 + 12 a = 41 here): 1e-12 of max |y| after 7 iterations."""
import numpy as np
import pytest
import torch

from paper_2406_04177_amd import _lib, inputs

pytestmark = pytest.mark.gpu

TILE = 1024
NMIN = 1 << 20          # voxels from which the staged kernels run


def volume(n, nx=120, ny=110):
    """A random volume of exactly n pores (porosity 0.9: long runs and gaps)."""
    nz = -(-int(n / 0.9) // (nx * ny)) + 1
    order = np.random.default_rng(n).permutation(nz * ny * nx)
    mask = np.zeros(nz * ny * nx, np.uint8)
    mask[order[:n]] = 1
    return mask.reshape(nz, ny, nx)


@pytest.mark.parametrize("regions", [None, [0.7, 1.0, 0.8, 0.9, 1.1, 0.75, 0.95, 0.85]], ids=["unit", "regions"])
@pytest.mark.parametrize("n", [NMIN, NMIN + 1, NMIN + TILE - 1, NMIN + 333], ids=["full", "one", "short", "ragged"])
@pytest.mark.parametrize("precond", ["jacobi", "mg"])
def test_staged_equals_direct(n, regions, precond):
    from paper_2406_04177_amd.graph import Graph
    from paper_2406_04177_amd.sim import Simulation
    g = Graph.from_masks(volume(n), regions=regions is not None)
    assert g.n == n
    p = inputs.ModelParams()
    dt = 20 * inputs.explicit_dt(p, 1.0)
    gen = torch.Generator(device="cuda").manual_seed(5)
    x0 = torch.rand((5, n), generator=gen, device="cuda", dtype=torch.float64)
    out = {}
    sim = Simulation(g, p, precision="f64", implicit=True, regions=regions, multigrid=True)
    sim.set_preconditioner(precond)
    for kernel in (_lib.VG_KERNEL_TABLE, _lib.VG_KERNEL_RELATIVE):
        sim.set_kernel(kernel)
        sim.set_fields(x0)
        its, _, rc = sim.implicit_step(dt, rtol=1e-30, max_iter=7, check=False)
        assert rc == _lib.VG_ENOCONV and its[1] == 7
        y7 = sim.fields[1].clone()
        sim.set_fields(x0)
        its, rel, rc = sim.implicit_step(dt, rtol=1e-10)
        assert rc == 0 and rel[1] <= 1e-10
        out[kernel] = (y7, its[1])
    (a, ia), (b, ib) = out[_lib.VG_KERNEL_TABLE], out[_lib.VG_KERNEL_RELATIVE]
    assert abs(ia - ib) <= 1
    assert float((a - b).abs().max()) <= 1e-12 * float(a.abs().max())
