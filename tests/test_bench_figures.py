"""The figures bench.py derives from the times of the passes (CPU only)."""

import pytest

import bench


def test_four_passes():
    t = {"ky_forward": 0.8, "kz_green": 1.1, "ky_inverse": 0.9, "kx_update": 2.2, "residual": 0.0}
    f = bench.iteration_figures(t, 10**8, lambda kernel: kernel)
    assert f["iteration_ms"] == 5.0
    assert f["hbm_frac_iteration"] == pytest.approx(248e8 / 5e-3 / 8e12, abs=1e-4)
    r = f["roofline"]
    assert (r["kernel"], r["traffic"], r["alg_bytes_per_launch"]) == ("kx_update", "kx_update", 104 * 10**8)
    assert r["achieved"] == pytest.approx(104e8 / 2.2e-3 / 1e9, abs=0.1)
    assert set(f["passes_ms"]) == set(t)


def test_fused_plane_pass():
    """Two launches an iteration: 48 + 104 bytes a voxel, and no y passes."""
    t = {"ky_forward": 0.0, "kz_green": 0.006, "ky_inverse": 0.0, "kx_update": 0.014, "residual": 0.0}
    n = 64 ** 3
    f = bench.iteration_figures(t, n, lambda kernel: None)
    assert f["hbm_frac_iteration"] == pytest.approx(152 * n / 20e-6 / 8e12, abs=1e-4)
    assert f["passes_ms"] == {"kz_green": 0.006, "plane": 0.014, "residual": 0.0}
    assert f["roofline"]["kernel"] == "plane"
    assert f["roofline"]["alg_bytes_per_launch"] == 104 * n


def test_hash_covers_the_splits(tmp_path, monkeypatch):
    """Counters taken on other splits of the lengths are not those of these kernels."""
    before = bench.kernel_hash()
    assert any(p.endswith("sizes_large.hip") for p in bench.PASS_SOURCES)
    for p in bench.PASS_SOURCES:
        (tmp_path / p).parent.mkdir(parents=True, exist_ok=True)
        (tmp_path / p).write_text(open(f"{bench.ROOT}/{p}", encoding="utf-8").read())
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.kernel_hash() == before
    large = tmp_path / "paper_2506_15411_amd/csrc/sizes_large.hip"
    large.write_text(large.read_text().replace("CBS_SIZE_XYZ(189, 21, 9, 27, 7)",
                                               "CBS_SIZE_XYZ(189, 27, 7, 27, 7)"))
    assert bench.kernel_hash() != before
