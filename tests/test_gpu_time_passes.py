"""Plan.time_passes tells the fused plane pass from the four passes (GPU): what is
not launched, the plane's y passes and the residual's own launch, has a time of 0."""

import pytest
import torch

from paper_2506_15411_amd.solver import Plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,fused", [((32, 32, 16), True), ((32, 36, 16), False),
                                         ((128, 128, 32), True), ((128, 128, 12), False)])
def test_y_entries(shape, fused, device):
    p = Plan(shape, 1.064e-6 / 8, pml=(2, 2, 2), device=device)
    eps = torch.ones(shape[::-1], device=device)
    eps[4:8, 8:16, 8:16] = 1.5
    p.set_permittivity(eps)
    t = p.time_passes(iters=3)
    assert (t["ky_forward"] == 0.0 and t["ky_inverse"] == 0.0) == fused
    assert t["residual"] == 0.0   # reduced inside the next z pass
    assert t["kz_green"] > 0.0 and t["kx_update"] > 0.0
    p.close()
