"""Which dense contractions the BF16X3 precision takes: float32 from 4097 to 786432 bins and on ragged grids (the
field is then the FP32 problem's, bit for bit), split bf16 elsewhere (within the parity tests' 1e-4 of
it, E against |E|)."""
import numpy as np
import pytest
import torch

from gpu_common import gpu_problem, log, need_gpu
from paper_2403_09070_amd import place3d, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,split", [((32, 32, 4), True), ((33, 47, 4), False), ((200, 66, 2), False), ((512, 256, 6), False),
                                        ((398, 354, 6), False), ((999, 403, 2), False), ((576, 256, 6), True),
                                        ((448, 440, 4), True), ((700, 562, 2), True)])
def test_field_of_the_precision_form(grid, split):
    need_gpu()
    nx, ny, nz = grid
    log(f"[split rule] {grid}")
    case = synth.make_case(config=synth.small_config(n_cells=64, n_nets=40, die=2.0 * max(grid), nx=nx, ny=ny, nz=nz),
                           seed=4)
    rho = torch.from_numpy(np.random.default_rng(ny).random((nz, ny, nx), dtype=np.float32)).cuda()
    keys = ("ex", "ey", "ez")
    a, b = [gpu_problem(case, precision=p).field(rho, want=keys) for p in (place3d.FP32, place3d.BF16X3)]
    assert all(torch.equal(a[k], b[k]) for k in keys) == (not split)
    norm = torch.sqrt(sum((a[k].double() ** 2).sum() for k in keys))
    assert all((a[k].double() - b[k].double()).norm() <= 1e-4 * norm for k in keys)
