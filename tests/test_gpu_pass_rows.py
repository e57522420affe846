"""x-pass work-groups at the edges of their row groups, against the FP64 oracle at
equal iteration counts (GPU).

A work-group takes R rows (k1_rows_for in csrc/kernels.hpp; 4 to 8 by length): grids
whose ny leaves groups exactly full, one row, and one row short of a full group, for
each length's own R.  Tolerance: an iteration's transforms carry about 1e-7 log2 N of
FP32 round-off and K iterations add at most K of them: with K = 6 and log2 N <= 20,
1.2e-5."""

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

# rows per group by length, and for each R supported lengths that leave groups full,
# one row and one row short
ROWS = {27: 7, 64: 8, 96: 5, 100: 6, 121: 5, 128: 8, 189: 6, 192: 8, 256: 8, 261: 4, 275: 5,
        315: 8, 621: 4}
NY = {4: (12, 13, 11), 5: (15, 16, 14), 6: (12, 13, 11), 7: (14, 15, 13), 8: (16, 25, 15)}


def test_every_kind_of_remainder():
    for r, (full, one, short) in NY.items():
        assert full % r == 0 and one % r == 1 and short % r == r - 1


@pytest.mark.parametrize("nx,ny", [(nx, ny) for nx, r in ROWS.items() for ny in NY[r]])
def test_rows_left_over(nx, ny, device):
    shape, pml = (nx, ny, 5), (2, 1, 1)
    eps = scenes.random_passive_eps(shape, pml, 11, loss=0.03)
    g = oc.Grid(*shape, LAM / 8, LAM, 1.0, pml)
    p = Plan(shape, LAM / 8, LAM, 1.0, pml, device=device)
    p.set_permittivity(torch.from_numpy(np.ascontiguousarray(eps)).to(device))
    E, st = p.solve(tol=0.0, max_iter=K, check_every=4)
    Eo, res = oc.solve_forward(g, eps, tol=0.0, max_iter=K)
    got = E.cpu().numpy()
    assert st.iterations == K
    assert float(np.linalg.norm((got - Eo).ravel()) / np.linalg.norm(Eo.ravel())) < TOL
    assert abs(st.residual - res.history[-1]) < TOL * max(1.0, res.history[-1]) * 10
    p.close()
