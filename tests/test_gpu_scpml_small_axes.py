"""The stretched layer's operator on the shortest axes and on lengths that are one
register transform (second factor 1), with a layer of one voxel and more: the edge
form there has an axis's first and last voxel alone, and lengths below five take the
whole transforms.  Against the FP64 oracle (GPU); tolerance as for every other length
(FP32 round-off of three to five transforms on white noise, 2e-6 for n <= 621)."""

import numpy as np
import pytest
import torch

from oracle import cbs as oc
from oracle import scpml
from paper_2506_15411_amd.solver import Plan

pytestmark = pytest.mark.gpu
LAM = 1.064e-6


@pytest.mark.parametrize("n,p", [(3, 1), (4, 1), (5, 1), (5, 2), (6, 1), (6, 2), (7, 1), (8, 1),
                                 (11, 1), (11, 5), (13, 1), (13, 2), (29, 1), (29, 2), (29, 14)])
def test_one_codelet_lengths(n, p, device):
    for shape in ((n, 9, 5), (9, n, 2), (5, 3, n)):
        axis = shape.index(n) if shape.count(n) == 1 else 2
        pml = tuple(p if a == axis else 0 for a in range(3))
        g = oc.Grid(*shape, LAM / 8, LAM, 1.0, pml, sigma_max=0.0)
        rng = np.random.default_rng(n + p)
        v = (rng.standard_normal((3,) + g.vshape)
             + 1j * rng.standard_normal((3,) + g.vshape)).astype(np.complex64)
        q = Plan(shape, LAM / 8, LAM, 1.0, pml, device=device, sigma_max=0.0)
        out = q.scpml_operator(torch.from_numpy(v).to(device), 0.75, 2).cpu().numpy()
        ref = scpml.delta_apply(g, v.astype(np.complex128), 0.75, 2)
        err = float(np.linalg.norm(out - ref) / np.linalg.norm(ref))
        assert err < 2e-6, (shape, pml, err)
        q.close()
