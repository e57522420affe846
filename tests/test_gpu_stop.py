"""Where a solve stops does not depend on how the host cuts it into quanta (GPU): the
stop flag goes up inside a z pass whose other work-groups may or may not see it, and
whatever is in flight behind leaves the field as the last counted iteration left it."""

import numpy as np
import pytest
import torch

from paper_2506_15411_amd import scenes
from paper_2506_15411_amd.solver import Plan

pytestmark = pytest.mark.gpu
LAM = 1.064e-6


# the fused plane pass, the four passes with the flag behind their loads (z
# work-groups of 2 to 15 waves), and a grid whose passes look at it first
@pytest.mark.parametrize("shape", [(32, 32, 32), (128, 128, 36), (64, 48, 40), (96, 64, 121),
                                   (20, 36, 315), (189, 189, 189)])
@pytest.mark.parametrize("warm", [False, True])
def test_stop_is_the_same_for_every_quantum(shape, warm, device):
    pml = tuple(min(8, n // 6) for n in shape)
    eps = scenes.random_passive_eps(shape, pml, 7, loss=0.0)
    p = Plan(shape, LAM / 6, LAM, 1.0, pml, device=device)
    p.set_permittivity(torch.from_numpy(np.ascontiguousarray(eps)).to(device))
    E0, _ = p.solve(tol=0.0, max_iter=5)
    start = E0 if warm else torch.zeros_like(E0)
    p.solve(start.clone(), tol=0.0, max_iter=24, history=True, warm=warm)
    eta = np.asarray(p.history())
    # stop at the first iteration at or below the residual of iteration 15
    tol = float(eta[14])
    stop = 1 + int(np.argmax(eta <= tol))
    ref, st = p.solve(start.clone(), tol=0.0, max_iter=stop, warm=warm)
    assert st.residual == eta[stop - 1]
    for every in (1, 2, 7, 16, 200):
        E, st = p.solve(start.clone(), tol=tol, max_iter=500, check_every=every, warm=warm)
        assert (st.iterations, st.converged, st.residual) == (stop, True, eta[stop - 1]), every
        assert torch.equal(E, ref), every
    p.close()
