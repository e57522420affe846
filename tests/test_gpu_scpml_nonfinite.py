"""Fields that leave the range of FP32 in a stretched-layer solve are reported as
divergence, never as a converged result (GPU)."""

import numpy as np
import pytest
import torch

from paper_2506_15411_amd import libcbs as L
from paper_2506_15411_amd import scenes
from paper_2506_15411_amd.solver import Plan

pytestmark = pytest.mark.gpu
LAM = 1.064e-6
SHAPE, PML = (24, 20, 32), (3, 3, 4)


def plan(device):
    p = Plan(SHAPE, LAM / 8, LAM, 1.0, PML, device=device, sigma_max=0.0)
    eps = scenes.random_passive_eps(SHAPE, PML, 3, loss=0.0)
    p.set_permittivity(torch.from_numpy(np.ascontiguousarray(eps)).to(device))
    return p


def test_non_finite_source_is_refused(device):
    """A NaN in the source makes the right-hand side's norm NaN, which must not
    pass for a source of zero (a solve that has nothing to do)."""
    p = plan(device)
    S = torch.from_numpy(scenes.random_field(SHAPE, 5)).to(device)
    E, st = p.solve_scpml(field=S, tol=0.0, max_iter=4, restart=4)
    assert st.iterations == 4
    S[1, 7, 6, 5] = complex(float("nan"), 0.0)
    with pytest.raises(L.CbsError) as ei:
        p.solve_scpml(field=S, tol=1e-3, max_iter=4, restart=4)
    assert ei.value.code == L.CBS_E_DIVERGED and "non-finite" in str(ei.value)
    # the plan stays usable
    S[1, 7, 6, 5] = 0.0
    S[1, 7, 6, 5] = torch.from_numpy(scenes.random_field(SHAPE, 5))[1, 7, 6, 5].to(device)
    E2, _ = p.solve_scpml(field=S, tol=0.0, max_iter=4, restart=4)
    assert torch.equal(E, E2)
    p.close()
