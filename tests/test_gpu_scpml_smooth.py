"""The stretched layer's operator on a spherical wave sampled at lambda/16, against
the FP64 oracle (GPU).

On a smooth field the symbol -p^2 (up to pi^2, rms 4.4) multiplies round-off that is
white in p, while the field itself has p = 2 pi/16, p^2 = 0.154: an error of e in the
first transform becomes 29 e in the result.  Tolerance: that transform is rounded to
FP32 once, between its two levels (2^-25 = 3e-8 rms): 8.7e-7, and 1e-7 log2 n / 4 or
so for the transforms behind the symbol: 1.1e-6.  In FP32 throughout, with some
log2 n roundings, the error is 1.9e-6 on the first grid."""

import numpy as np
import pytest
import torch

from oracle import cbs as oc
from oracle import scpml
from paper_2506_15411_amd.solver import Plan

pytestmark = pytest.mark.gpu
LAM = 1.064e-6


@pytest.mark.parametrize("shape,pml", [((64, 64, 64), (8, 8, 8)), ((128, 36, 40), (8, 6, 6)),
                                       ((27, 100, 48), (4, 8, 16)), ((24, 32, 192), (4, 4, 36)),
                                       ((29, 16, 121), (4, 2, 18))])
def test_spherical_wave(shape, pml, device):
    g = oc.Grid(*shape, LAM / 16, LAM, 1.0, pml, sigma_max=0.0)
    nx, ny, nz = shape
    z, y, x = np.meshgrid(np.arange(nz) - nz / 2, np.arange(ny) - ny / 2, np.arange(nx) - nx / 2,
                          indexing="ij")
    r = np.sqrt(x * x + y * y + z * z + 4.0)
    f = np.exp(2j * np.pi / 16 * r) / r
    v = np.stack([f, 0.5 * f, 1j * f]).astype(np.complex64)
    p = Plan(shape, LAM / 16, LAM, 1.0, pml, device=device, sigma_max=0.0)
    out = p.scpml_operator(torch.from_numpy(v).to(device), 0.75, 1).cpu().numpy()
    ref = scpml.delta_apply(g, v.astype(np.complex128), 0.75, 1)
    err = float(np.linalg.norm(out - ref) / np.linalg.norm(ref))
    print(f"{shape}: {err:.2e}")
    assert err < 1.1e-6, err
    p.close()
