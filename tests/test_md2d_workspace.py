"""A multi-die 2D problem's workspace on the transforms' grids does not depend on the precision, whatever its number of
nodes: its solves take the float32 transforms in both, and no context of it takes a step of its own, which
alone would need split contractions from 2^20 instances on.  (Sizes are asked on the host, no GPU.)"""
import ctypes

import pytest

from paper_2403_09070_amd import place3d
from test_abi import L, _md_problem  # noqa: F401


@pytest.mark.parametrize("nodes", [(1 << 20) - 3, (1 << 20) + 3, 4 << 20])
def test_precisions_take_the_same_workspace(L, nodes):  # noqa: F811
    sizes = []
    for precision in (place3d.FP32, place3d.BF16X3):
        p, n = _md_problem(), ctypes.c_size_t()
        p.n_nodes, p.nx, p.ny, p.precision = nodes, 1024, 1024, precision
        p.n_layer[0], p.n_layer[1], p.n_layer[2] = nodes - 20, 10, 10
        assert L.place3d_md2d_workspace_size(ctypes.byref(p), ctypes.byref(n)) == 0
        sizes.append(n.value)
    assert sizes[0] == sizes[1]
