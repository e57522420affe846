"""Workspace sizes of the stretched layer, to the last field (host arithmetic)."""

import pytest

from paper_2506_15411_amd import libcbs as L


@pytest.mark.parametrize("shape", [(24, 20, 32), (64, 64, 64), (275, 275, 315), (8, 7, 6)])
@pytest.mark.parametrize("restart", [1, 8, 40, 64])
def test_stretched_layer_fields(shape, restart):
    """restart + 1 basis fields, the right-hand side, the derivative source and the
    three scalar fields T_b v_b: (restart + 4) vector fields of 24 bytes a voxel.
    Beside them an axis's factors and twiddles (24 bytes a voxel of the axis), 65 x
    512 partial sums, 3 x 65 + 65 sums and each region's padding to 256 bytes."""
    n = shape[0] * shape[1] * shape[2]
    fields = (restart + 4) * 24 * n
    small = 24 * sum(shape) + 16 * (65 * 512 + 3 * 65 + 65)
    b = L.cbs_scpml_workspace_bytes(*shape, restart)
    assert fields + small <= b <= fields + small + 256 * 13
