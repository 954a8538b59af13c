"""Implicit steps of FP32 volumes of 2^29 voxels and more, whose FP64 vectors
outgrow 32-bit byte offsets: the packed neighbour sources with 64-bit indices
against the table on the same volume.  The two differ by the order of FP64
partial sums only, so after a few iterations the FP32 results differ by at most
one float spacing (2^-23 of a value)."""
import numpy as np
import pytest
import torch

from paper_2406_04177_amd import _lib, inputs

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]


def test_wide_packed_sources_equal_the_table():
    from paper_2406_04177_amd.graph import Graph
    from paper_2406_04177_amd.sim import Simulation
    shape = (1000, 700, 800)          # distances of 1, 10 and 20 bits: both packings fit
    g = Graph.from_masks(np.ones(shape, np.uint8))
    assert g.n >= 1 << 29
    p = inputs.ModelParams()
    dt = 20 * inputs.explicit_dt(p, 1.0)
    sim = Simulation(g, p, precision="f32", implicit=True, multigrid=True, band=False)
    gen = torch.Generator(device="cuda")
    for precond in ("jacobi", "mg"):
        sim.set_preconditioner(precond)
        out = {}
        for kernel in (_lib.VG_KERNEL_TABLE, _lib.VG_KERNEL_RELATIVE, _lib.VG_KERNEL_OFFSET):
            sim.set_kernel(kernel)
            assert sim.kernel_in_use() == kernel
            sim.fields.uniform_(generator=gen.manual_seed(5))
            print(precond, "kernel", kernel, flush=True)
            its, rel, rc = sim.implicit_step(dt, rtol=1e-30, max_iter=3, check=False)
            assert rc == _lib.VG_ENOCONV and its[1] == 3
            out[kernel] = (sim.fields[1].clone(), rel[1])
        ref, res = out.pop(_lib.VG_KERNEL_TABLE)
        for y, r in out.values():
            assert abs(r - res) <= 1e-12 * res
            assert bool(((y - ref).abs() <= 2.0 ** -23 * torch.maximum(y.abs(), ref.abs())).all())
        del out, ref, y
    # the preconditioner alone (its own launch path)
    r = torch.rand(g.n, generator=gen.manual_seed(6), device="cuda", dtype=torch.float64)
    z = []
    for kernel in (_lib.VG_KERNEL_TABLE, _lib.VG_KERNEL_RELATIVE):
        sim.set_kernel(kernel)
        z.append(sim.precondition(20.0 / 6.0, r))
    assert float((z[0] - z[1]).abs().max()) <= 1e-12 * float(z[0].abs().max())
