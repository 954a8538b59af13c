"""The band kernel's march at its edges: planes whose ranges need one, two and
all three slots of its threads, bands cut off by the volume, one-row bands,
chunks of one and of all planes, and every parity of pass pairs before a
single pass takes the state back (bit for bit equal to the single-pass kernel,
as both do the same operations in the same order)."""
import numpy as np
import pytest
import torch

from paper_2406_04177_amd import _lib, inputs

pytestmark = pytest.mark.gpu


def mask_of(shape, por, seed):
    """Smoothed noise (unsmoothed noise of these sizes has neighbour distances
    that spread too far for the relative codes), full at porosity 1."""
    mask = np.ones(shape, np.uint8) if por >= 1 else inputs.synthetic_volume(shape, porosity=por, seed=seed)
    return mask


# (nz, ny, nx), porosity: rows of 1 to 325 pores, and 600 (one-row bands)
SHAPES = [((11, 33, 1), 0.7), ((7, 67, 50), 0.6), ((1, 40, 410), 0.6), ((13, 21, 410), 0.62), ((5, 9, 1000), 0.7),
          ((4, 5, 600), 1.0), ((70, 3, 64), 0.5)]


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("shape,por", SHAPES, ids=["x".join(map(str, s)) for s, _ in SHAPES])
def test_pairs_equal_single_passes(shape, por, precision):
    from paper_2406_04177_amd.graph import Graph
    from paper_2406_04177_amd.sim import Simulation
    mask = mask_of(shape, por, 3)
    g = Graph.from_masks(mask)
    p = inputs.ModelParams(v_dom=0.05, k_dom=0.5, rho=0.01, mu=0.02, v_som=0.01, v_p4=0.02)
    dt = inputs.explicit_dt(p, 0.9)
    x0 = torch.rand((5, g.n), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda",
                    dtype=torch.float64)
    sims = []
    for kernel in (_lib.VG_KERNEL_BAND, _lib.VG_KERNEL_RELATIVE):
        sim = Simulation(g, p, precision=precision, implicit=False)
        sim.set_kernel(kernel)
        sim.set_launch_options("off")
        assert sim.kernel_in_use() == kernel
        sims.append(sim)
    for steps, log_every in ((2, 0), (3, 0), (4, 0), (5, 0), (6, 0), (7, 0), (14, 4), (15, 5), (17, 6)):
        logs = []
        for sim in sims:
            sim.set_fields(x0)
            logs.append(sim.step(steps, dt, log_every=log_every))
        assert torch.equal(sims[0].fields, sims[1].fields), (steps, log_every)
        if log_every:
            assert torch.equal(logs[0], logs[1]), (steps, log_every)
