"""The stretched layer's operator on every axis length and at the edges of its
line tiles, against the FP64 oracle (GPU).

Tolerance: a transform of n points carries about 1e-7 log2 n of FP32 round-off;
on white noise the symbols -p^2 and i p weigh it like the result itself, so the
relative error stays below 1e-7 log2 n (three to five transforms): 2e-6 for
n <= 621."""

import numpy as np
import pytest
import torch

from oracle import cbs as oc
from oracle import scpml
from paper_2506_15411_amd.solver import Plan

pytestmark = pytest.mark.gpu
LAM = 1.064e-6

LENGTHS = [7, 8, 9, 10, 12, 13, 14, 15, 16, 18, 20, 24, 25, 27, 29, 32, 36, 40, 48, 64, 96, 100,
           121, 128, 189, 192, 256, 261, 275, 315, 621]


@pytest.mark.parametrize("n", LENGTHS)
def test_every_length_on_every_axis(n, device):
    # the other axes leave tiles of 1, 4, 8 and more lines
    shapes = [(n, 3, 5), (9, n, 2)] + ([(5, 3, n)] if n != 621 else [])
    for shape in shapes:
        for frac, order in ((8, 1), (3, 2)):
            # at least one voxel: without a layer the operator is exactly zero
            pml = tuple(max(1, m // frac) if m == n else (1 if m == 9 else 0) for m in shape)
            g = oc.Grid(*shape, LAM / 8, LAM, 1.0, pml, sigma_max=0.0)
            rng = np.random.default_rng(n)
            v = (rng.standard_normal((3,) + g.vshape)
                 + 1j * rng.standard_normal((3,) + g.vshape)).astype(np.complex64)
            p = Plan(shape, LAM / 8, LAM, 1.0, pml, device=device, sigma_max=0.0)
            out = p.scpml_operator(torch.from_numpy(v).to(device), 0.75, order).cpu().numpy()
            ref = scpml.delta_apply(g, v.astype(np.complex128), 0.75, order)
            err = float(np.linalg.norm(out - ref) / np.linalg.norm(ref))
            assert err < 2e-6, (shape, pml, order, err)
            p.close()


# layers one voxel below, at and one above the length (N2 = 8, 9, 10, 11, 23) up to
# which the transforms form the layer's elements alone
@pytest.mark.parametrize("n,p", [(64, 7), (64, 8), (64, 9), (189, 8), (189, 9), (189, 10),
                                 (100, 9), (100, 10), (100, 11), (275, 1), (275, 10), (275, 11),
                                 (275, 12), (621, 22), (621, 23), (621, 24)])
def test_layers_around_the_edge_form(n, p, device):
    for shape in [(n, 3, 5), (9, n, 2)] + ([(5, 3, n)] if n != 621 else []):
        pml = tuple(p if m == n else 0 for m in shape)
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
