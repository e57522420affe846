"""What the fused plane pass takes of a CU, from the compiler's resource report (CPU
only; compiles four lengths): the bound on its waves per SIMD is a rule on the plane's
LDS and registers, and no form is pressed into it at the price of spills that cost more
than the occupancy brings."""

import os
import re
import shutil
import subprocess

import pytest

from paper_2506_15411_amd import build as B

# (n1, n2): the longest split with the bound, the one below, and the two lengths above,
# which hold two rounds of tasks (96) and one plane a CU (100)
SPLITS = [(8, 6), (8, 8), (12, 8), (10, 10)]


@pytest.fixture(scope="module")
def report(tmp_path_factory):
    try:
        cc = B.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not found")
    filt = shutil.which("c++filt")
    if filt is None:
        pytest.skip("c++filt not found")
    d = tmp_path_factory.mktemp("plane")
    inst = "\n".join(f"template void launch_kxy<{a}, {b}>(const CbsArgs&, int, hipStream_t);"
                     for a, b in SPLITS)
    (d / "x.hip").write_text(f'#include "kernels.hpp"\nnamespace cbs {{\n{inst}\n}}\n')
    r = subprocess.run([cc, *B.HIPCC_FLAGS, "-I", B.CSRC, "-Rpass-analysis=kernel-resource-usage",
                        "--cuda-device-only", "-c", str(d / "x.hip"), "-o", str(d / "x.o")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    out, name = {}, None
    for line in subprocess.run([filt], input=r.stderr, capture_output=True, text=True).stdout.splitlines():
        m = re.search(r"Function Name: void cbs::kxy_pass<(\d+), (\d+), (\d+), (\d+)>", line)
        if m:
            name = tuple(int(v) for v in m.groups())
            out[name] = {}
        m = re.search(r"remark: .*?(VGPRs|ScratchSize \[bytes/lane\]|Occupancy \[waves/SIMD\]): (\d+)", line)
        if m and name:
            out[name].setdefault(m.group(1).split()[0], int(m.group(2)))
    assert len(out) == 7 * len(SPLITS)
    return out


def test_no_form_spills_more_than_a_few_registers(report):
    for (n1, n2, mode, form), u in report.items():
        limit = 16 if (n1, n2, mode) == (8, 8, 1) and form != 2 else 0
        assert u["ScratchSize"] <= limit, (n1, n2, mode, form, u)


def test_six_waves_where_planes_share_a_cu(report):
    # plane waves and points, normal and oblique
    for form in (0, 1):
        assert report[(8, 8, 1, form)]["Occupancy"] >= 6
        assert report[(8, 6, 1, form)]["Occupancy"] >= 6
