"""The dense float32 contractions of the solve give the same bits whichever output tile they take.

A contraction sums over k in ascending order in every tile, so that a map solved for one output at a
time (few tiles: the narrow ones) equals the same outputs asked for together (three times the tiles:
the wide ones).  Ragged on every side of both tiles, with and without folding.  The narrow tiles'
values against the oracle are the parity tests' (grids from 24 x 20 to 280 x 264)."""
import numpy as np
import pytest
import torch

from gpu_common import gpu_problem, log, need_gpu
from paper_2403_09070_amd import place3d, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(999, 1001, 4), (1002, 998, 4)])
def test_outputs_together_equal_outputs_alone(grid):
    need_gpu()
    nx, ny, nz = grid
    log(f"[gemm] {grid}")
    case = synth.make_case(config=synth.small_config(n_cells=64, n_nets=40, die=1500.0, nx=nx, ny=ny, nz=nz), seed=3)
    prob = gpu_problem(case, precision=place3d.FP32)
    rho = torch.from_numpy(np.random.default_rng(nx).random((nz, ny, nx), dtype=np.float32)).cuda()
    keys = ("phi", "ex", "ey", "ez")
    together = prob.field(rho, want=keys)
    for k in keys:
        assert torch.equal(prob.field(rho, want=(k,))[k], together[k]), (grid, k)
