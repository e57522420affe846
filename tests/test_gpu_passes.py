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


# the fused plane pass: every square length it covers, at plane counts on both
# sides of its rule, with every kind of source and batched
@pytest.mark.parametrize("n,nz", [(9, 5), (10, 8), (12, 7), (14, 9), (15, 5), (16, 8), (18, 6),
                                  (20, 7), (24, 9), (25, 5), (27, 8), (32, 9), (36, 5), (40, 6),
                                  (48, 5), (64, 5), (96, 16), (96, 18), (100, 16), (100, 18),
                                  (121, 25), (121, 27), (128, 27), (128, 32)])
def test_fused_plane(n, nz, device):
    check((n, n, nz), (2, 1, 1), device)


@pytest.mark.parametrize("n,nz", [(16, 9), (25, 8), (64, 6), (100, 18)])
def test_fused_plane_sources(n, nz, device):
    pml = (2, 2, 1)
    shape = (n, n, nz)
    eps = scenes.random_passive_eps(shape, pml, 5, loss=0.02)
    g = oc.Grid(*shape, LAM / 8, LAM, 1.0, pml)
    p = Plan(shape, LAM / 8, LAM, 1.0, pml, device=device)
    p.set_permittivity(torch.from_numpy(np.ascontiguousarray(eps)).to(device))
    pol, d = (0.96, 0.0, -0.28), (0.28, 0.0)
    waves = [((1.0, 0.0, 0.0), None), (pol, d)]
    refs = [oc.cbs(g, eps, oc.plane_wave_source(g, eps, w, dd or (0.0, 0.0)), tol=0.0,
                   max_iter=K).E_s for w, dd in waves]
    for (w, dd), ref in zip(waves, refs):
        E, _ = p.solve(tol=0.0, max_iter=K, pol=w, direction=dd, scattered=True)
        assert rel(E.cpu().numpy(), ref) < TOL
    Eb, st = p.solve_batch(waves, tol=0.0, max_iter=K, scattered=True)
    for b, ref in enumerate(refs):
        assert rel(Eb[b].cpu().numpy(), ref) < TOL
    S = scenes.random_field(shape, 9)
    for conj in (False, True):
        Ea, _ = p.adjoint(field=torch.from_numpy(S).to(device), conj=conj, tol=0.0, max_iter=K)
        ref = oc.cbs(g, eps, (np.conj(S) if conj else S).astype(np.complex128), tol=0.0,
                     max_iter=K).E_s
        assert rel(Ea.cpu().numpy(), ref) < TOL
    r0 = (n // 2, n // 3, nz // 2)
    Ep, _ = p.solve(point=(r0, (1.0, 0.5j, 0.0)), tol=0.0, max_iter=K)
    ref = oc.cbs(g, eps, oc.point_source(g, r0, np.array([1.0, 0.5j, 0.0])), tol=0.0, max_iter=K).E_s
    assert rel(Ep.cpu().numpy(), ref) < TOL
    p.close()


# a field source's zero rows are found by the prologue and not read afterwards:
# sources at a point, in a plane, in a strip of rows and everywhere, one after the
# other on one plan, so a row left over from the source before would show
@pytest.mark.parametrize("shape", [(36, 20, 9), (121, 29, 7), (192, 9, 6), (27, 16, 5)])
def test_field_source_with_zero_rows(shape, device):
    nx, ny, nz = shape
    pml = (2, 1, 1)
    eps = scenes.random_passive_eps(shape, pml, 3, loss=0.02)
    g = oc.Grid(*shape, LAM / 8, LAM, 1.0, pml)
    p = Plan(shape, LAM / 8, LAM, 1.0, pml, device=device)
    p.set_permittivity(torch.from_numpy(np.ascontiguousarray(eps)).to(device))
    full = scenes.random_field(shape, 4)
    parts = []
    for sel in ((1, nz // 2, ny // 3, nx - 1), (0, nz - 2, slice(None), slice(None)),
                (slice(None), slice(None), slice(2, 4), slice(None)),
                (slice(None),) * 4, (2, 0, 0, 0)):
        S = np.zeros_like(full)
        S[sel] = full[sel]
        parts.append(S)
    for S in parts:
        for conj in (False, True):
            E, _ = p.adjoint(field=torch.from_numpy(S).to(device), conj=conj, tol=0.0, max_iter=K)
            ref = oc.cbs(g, eps, (np.conj(S) if conj else S).astype(np.complex128), tol=0.0,
                         max_iter=K).E_s
            assert rel(E.cpu().numpy(), ref) < TOL
    p.close()
