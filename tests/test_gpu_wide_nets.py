"""Nets of more pins than a wavefront's lanes hold (256), which it reads from memory in each of its passes: the
values on the edges of its rounds (128 pins), and its time.

Values against the oracle with the parity tests' bars.  Time: one wavefront takes such a net, a round of
64 pins after the other, each a chain of three loads, 0.4 us where nothing overlaps it (924 us for the
2345 rounds of 30000 pins read five times): a gradient may cost as much as those five readings with
their loads one after the other, 1 ms for 30000 pins."""
import numpy as np
import pytest
import torch

import test_gpu_parity as parity
from gpu_common import gpu_problem, log, need_gpu, with_nets
from paper_2403_09070_amd import place3d, synth

pytestmark = pytest.mark.gpu


def wide_case(degrees, n_cells, seed=8):
    case = synth.make_case(config=synth.small_config(n_cells=n_cells, n_nets=10, die=150.0, nx=32, ny=32, nz=4,
                                                     macros=("uniform", 3, 0.01, 0.03), degree=("geo", 0.6, 8)), seed=seed)
    rng = np.random.default_rng(seed)
    return with_nets(case, [rng.choice(case.n_inst, size=d, replace=False) for d in degrees], seed)


@pytest.mark.parametrize("precision", [place3d.FP32, place3d.BF16X3])
@pytest.mark.parametrize("one_die", [False, True])
def test_wide_nets_match_the_oracle(precision, one_die):
    need_gpu()
    case = wide_case([256, 257, 319, 320, 321, 383, 384, 385, 511, 512, 513, 700, 1000, 2, 3, 60], 1200)
    if one_die:
        case.xyz0[2] = np.minimum(case.xyz0[2], 0.25 * case.nz * 0.5 * (case.die_x / case.nx + case.die_y / case.ny))
    log(f"[wide] precision {precision} one die {one_die}")
    parity.test_wirelength(("wide", case, gpu_problem(case, precision=precision)))


def test_a_wide_net_takes_no_more_than_five_readings():
    need_gpu()
    log("[wide] one net of 30000 pins")
    case = wide_case([30000], 60000)
    prob = gpu_problem(case, precision=place3d.FP32)
    x = prob.xyz(case.xyz0)
    times = []
    for _ in range(12):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        prob.wl_grad(x)
        b.record()
        b.synchronize()
        times.append(1e3 * a.elapsed_time(b))
    log(f"[wide] {np.median(times):.0f} us")
    assert np.median(times) <= 1000
