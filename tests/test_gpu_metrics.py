"""cbs_lens_metrics on planes of every kind of length, against numpy in FP64 on
the same complex64 field (GPU).

The library computes in FP64 from the same inputs: focus exact, the others to
1e-10 (direct sums of up to 621 terms)."""

import math

import numpy as np
import pytest
import torch

from paper_2506_15411_amd.solver import Plan

pytestmark = pytest.mark.gpu
LAM = 1.064e-6


def reference(E, pitch, lo, hi, aperture):
    I = (np.abs(E.astype(np.complex128)) ** 2).sum(0)
    box = I[lo[2]:hi[2], lo[1]:hi[1], lo[0]:hi[0]]
    z, y, x = np.unravel_index(np.argmax(box), box.shape)
    f = (x + lo[0], y + lo[1], z + lo[2])

    def width(v, i0):
        half, l, r = 0.5 * v[i0], i0, i0
        while l > 0 and v[l - 1] >= half:
            l -= 1
        while r < len(v) - 1 and v[r + 1] >= half:
            r += 1
        if l == 0 or r == len(v) - 1:
            return math.nan
        return (r + (v[r] - half) / (v[r] - v[r + 1]) - (l - 1)
                - (half - v[l - 1]) / (v[l] - v[l - 1])) * pitch

    fw = (width(I[f[2], f[1]], f[0]), width(I[f[2], :, f[0]], f[1]), width(I[:, f[1], f[0]], f[2]))
    ny, nx = I.shape[1:]
    A = np.fft.fft2(E[:2, f[2]].astype(np.complex128))
    k = 2 * math.pi / LAM
    kx = 2 * math.pi * np.fft.fftfreq(nx, pitch)[None, :]
    ky = 2 * math.pi * np.fft.fftfreq(ny, pitch)[:, None]
    kz2 = k * k - kx * kx - ky * ky
    on = kz2 > 0
    kz = np.sqrt(np.where(on, kz2, 1.0))
    ex, ey = A * on
    ez = -(kx * ex + ky * ey) / kz
    ex, ey, hx, hy = np.fft.ifft2([ex, ey, (ky * ez - kz * ey) / k, (kz * ex - kx * ez) / k])
    sz = (ex * np.conj(hy) - ey * np.conj(hx)).real
    rad = 0.75 * (fw[0] + fw[1]) / pitch
    yy, xx = np.mgrid[0:ny, 0:nx]
    flux = sz[(xx - f[0]) ** 2 + (yy - f[1]) ** 2 <= rad * rad].sum() * pitch * pitch
    return f, float(I[f[2], f[1], f[0]]), fw, flux, flux / (math.pi * 0.25 * aperture ** 2)


@pytest.mark.parametrize("shape", [(9, 10, 12), (16, 15, 29), (64, 64, 20), (65 - 1, 121, 9),
                                   (121, 100, 8), (275, 189, 10), (621, 64, 8), (36, 621, 8)])
def test_figures_match_numpy(shape, device):
    nx, ny, nz = shape
    pitch = LAM / 6
    rng = np.random.default_rng(nx + ny)
    x, y, z = (np.arange(n) for n in shape)
    g = (np.exp(-((x - 0.52 * nx) / (0.13 * nx)) ** 2)[None, None, :]
         * np.exp(-((y - 0.45 * ny) / (0.14 * ny)) ** 2)[None, :, None]
         * np.exp(-((z - 0.5 * nz) / (0.2 * nz)) ** 2 + 1j * z)[:, None, None])
    E = 0.003 * (rng.standard_normal((3, nz, ny, nx)) + 1j * rng.standard_normal((3, nz, ny, nx)))
    E[0] += g
    E[1] += 0.3j * g
    E = E.astype(np.complex64)
    p = Plan(shape, pitch, LAM, device=device)
    lo, hi = (1, 1, 1), (nx - 1, ny - 1, nz - 1)
    r = p.lens_metrics(torch.from_numpy(E).to(device), lo, hi, aperture_m=nx * pitch)
    f, peak, fw, flux, eta = reference(E, pitch, lo, hi, nx * pitch)
    assert tuple(r["focus"]) == f
    assert r["peak"] == pytest.approx(peak, rel=1e-10)
    assert r["fwhm"] == pytest.approx(fw, rel=1e-10, nan_ok=True)
    assert r["disc_flux"] == pytest.approx(flux, rel=1e-10, nan_ok=True)
    assert r["eta_f"] == pytest.approx(eta, rel=1e-10, nan_ok=True)
    p.close()


def test_a_field_without_finite_values(device):
    p = Plan((12, 10, 9), LAM / 6, LAM, device=device)
    E = torch.full(p.fshape, float("nan"), dtype=torch.complex64, device=device)
    r = p.lens_metrics(E, (0, 0, 0), (12, 10, 9), aperture_m=1e-6)
    assert tuple(r["focus"]) == (0, 0, 0) and r["peak"] == -1.0 and math.isnan(r["eta_f"])
    p.close()
