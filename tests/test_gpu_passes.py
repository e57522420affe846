"""The passes of a CBS iteration at the edges of their work splits, against the
FP64 oracle at equal iteration counts (GPU).

Tolerance: an iteration's transforms carry about 1e-7 log2 N of FP32 round-off
relative to the field, and K iterations add at most K of them; with K = 6 and
log2 N <= 20 that is 1.2e-5."""

import numpy as np
import pytest
import torch

from oracle import cbs as oc
from paper_2506_15411_amd import scenes
from paper_2506_15411_amd.solver import Plan

pytestmark = pytest.mark.gpu
LAM = 1.064e-6
K = 6
TOL = 1.2e-5


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


def check(shape, pml, dev, loss=0.03):
    eps = scenes.random_passive_eps(shape, pml, 11, loss=loss)
    g = oc.Grid(*shape, LAM / 8, LAM, 1.0, pml)
    p = Plan(shape, LAM / 8, LAM, 1.0, pml, device=dev)
    p.set_permittivity(torch.from_numpy(np.ascontiguousarray(eps)).to(dev))
    E, st = p.solve(tol=0.0, max_iter=K, check_every=4)
    Eo, res = oc.solve_forward(g, eps, tol=0.0, max_iter=K)
    assert st.iterations == K
    assert rel(E.cpu().numpy(), Eo) < TOL
    assert abs(st.residual - res.history[-1]) < TOL * max(1.0, res.history[-1]) * 10
    p.close()


# x-pass work-groups hold 4 to 8 rows: row counts that leave one row, one row
# less than a full group, and exactly full groups
@pytest.mark.parametrize("nx", [96, 121, 189, 192, 261, 275, 315, 621])
@pytest.mark.parametrize("ny", [8, 9, 15])
def test_rows_per_group(nx, ny, device):
    check((nx, ny, 5), (2, 1, 1), device)
