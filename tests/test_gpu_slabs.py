"""Passes of compensated fields run slab by slab (fields larger than the
last-level cache, packed neighbours) against whole passes (the table,
VG_KERNEL_TABLE, never takes slabs): fields and totals bit for bit, as every
voxel sees the same operations in the same order.  Both step orders, logged
steps at the start, inside and at the end of a group, more passes than a
group, region weights, Algorithm 2 and every pool diffusing."""
import pytest
import torch

from paper_2406_04177_amd import _lib, inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mask():
    return inputs.synthetic_volume((352, 341, 517), porosity=0.2, seed=1)     # 12.4 M pores


CASES = {
    "plain": ({}, None, 0),
    "diffusion-first": ({}, None, 1),
    "regions": ({}, [0.7, 1.0, 0.8, 0.9, 1.1, 0.75, 0.95, 0.85], 0),
    "algorithm-2": ({"sequential": True}, None, 0),
    "every-pool": ({"D": (1e-10, 1e-9, 0.0, 2e-10, 0.0)}, None, 0),
}


@pytest.mark.parametrize("case", CASES)
def test_slabs_equal_whole_passes(mask, case):
    from paper_2406_04177_amd.graph import Graph
    from paper_2406_04177_amd.sim import Simulation
    kw, regions, order = CASES[case]
    g = Graph.from_masks(mask, regions=regions is not None)
    p = inputs.ModelParams(v_dom=0.05, k_dom=0.5, rho=0.01, mu=0.02, v_som=0.01, v_p4=0.02, **kw)
    dt = inputs.explicit_dt(p, 0.8)
    gen = torch.Generator(device="cuda").manual_seed(2)
    x0 = torch.rand((5, g.n), generator=gen, device="cuda", dtype=torch.float64)
    out = []
    for kernel in (_lib.VG_KERNEL_AUTO, _lib.VG_KERNEL_TABLE):
        sim = Simulation(g, p, precision="f32c", implicit=False, regions=regions, step_order=order)
        sim.set_kernel(kernel)
        if kernel == _lib.VG_KERNEL_AUTO:
            assert sim.kernel_in_use() == _lib.VG_KERNEL_RELATIVE
        got = []
        for steps, log_every in ((1, 0), (2, 1), (5, 0), (21, 4), (17, 17)):
            sim.set_fields(x0)
            log = sim.step(steps, dt, log_every=log_every)
            got.append((sim.state(), log))
        out.append(got)
        del sim
    for (fa, la), (fb, lb) in zip(*out):
        assert torch.equal(fa, fb)
        assert (la is None and lb is None) or torch.equal(la, lb)
