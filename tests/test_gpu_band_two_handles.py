"""The band kernel's LDS limit belongs to the kernel, not to a handle: an FP32
volume whose blocks need more than half a CU's LDS still runs after a second
handle of smaller blocks was made (one-row bands of 3 x 610 and of 3 x 560
pores: 81 and 74 KiB), bit for bit as on single passes."""
import numpy as np
import pytest
import torch

from paper_2406_04177_amd import _lib, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_a_second_handle_lowers_nothing(precision):
    from paper_2406_04177_amd.graph import Graph
    from paper_2406_04177_amd.sim import Simulation
    p = inputs.ModelParams(v_dom=0.05, k_dom=0.5, rho=0.01, mu=0.02, v_som=0.01, v_p4=0.02)
    dt = inputs.explicit_dt(p, 0.9)

    def sim(nx, kernel):
        s = Simulation(Graph.from_masks(np.ones((5, 9, nx), np.uint8)), p, precision=precision, implicit=False)
        s.set_kernel(kernel)
        s.set_launch_options("off")
        assert s.kernel_in_use() == kernel
        return s

    wide = 610 if precision == "f32" else 480
    big, ref = sim(wide, _lib.VG_KERNEL_BAND), sim(wide, _lib.VG_KERNEL_RELATIVE)
    small = sim(wide - 50, _lib.VG_KERNEL_BAND)
    x0 = torch.rand((5, big.graph.n), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda",
                    dtype=torch.float64)
    for s in (big, ref):
        s.set_fields(x0)
    small.step(5, dt)
    big.step(9, dt)
    ref.step(9, dt)
    assert torch.equal(big.fields, ref.fields)
