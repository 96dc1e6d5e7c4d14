"""The overflow that a step reports, on both sides of the numbers of instances from which a launch of its own adds up
the partial sums (512 workgroups' of the combine, 131072 instances; multi-die 2048 and 524288 nodes), against the
oracle's map at the same positions.  More instances on the bottom die than on top, and another number on
each layer, so that no two overflows are alike.  Bar: the parity tests' 1e-6 absolute."""
import numpy as np
import pytest
import torch

from gpu_common import gpu_problem, log, need_gpu, oracle_problem
from oracle import density as oden
from oracle import multidie as md
from oracle import optimizer as opt
from paper_2403_09070_amd import place3d, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_inst", [700, 512 * 256, 512 * 256 + 1])
def test_step_overflow(n_inst):
    need_gpu()
    log(f"[overflow] step of {n_inst} instances")
    case = synth.make_case(config=synth.small_config(n_cells=n_inst - 3, n_nets=300, die=1.1 * n_inst ** 0.5, nx=64, ny=64, nz=2),
                           seed=9)
    assert case.n_inst == n_inst
    rng = np.random.default_rng(1)
    dz = case.nz * 0.5 * (case.die_x / case.nx + case.die_y / case.ny)
    xyz = case.xyz0.copy()
    xyz[2] = np.where(rng.random(n_inst) < 0.7, 0.3 * dz, 0.65 * dz)
    prob, pb = gpu_problem(case, precision=place3d.FP32), oracle_problem(case)
    st = prob.new_state()
    x = prob.xyz(xyz)
    for t in (st.u, st.v):
        t.copy_(x)
    st.v_prev.copy_(x + 0.01)
    st.scalars[place3d.S["a"]] = 1.0
    st.scalars[place3d.S["lam"]] = 1.0
    prob.step(st)
    s = st.read()
    want = opt.overflow(pb, oden.density_map(case.size, case.kind, xyz, pb.geo), xyz.astype(np.float64))
    log(f"[overflow] {s['ovfl_bot']:.7f} {s['ovfl_top']:.7f}, oracle {want[0]:.7f} {want[1]:.7f}")
    assert min(want) > 1e-3 and abs(want[0] - want[1]) > 1e-3
    assert abs(s["ovfl_bot"] - want[0]) <= 1e-6 and abs(s["ovfl_top"] - want[1]) <= 1e-6


@pytest.mark.parametrize("n", [900, 2048 * 256, 2048 * 256 + 1])
def test_multi_die_step_overflow(n):
    need_gpu()
    log(f"[overflow] multi-die step of {n} nodes")
    rng = np.random.default_rng(n)
    die = 0.5 * n ** 0.5
    layer = rng.choice(3, n, p=[0.5, 0.3, 0.2]).astype(np.uint8)
    xy = (die * (0.1 + 0.8 * rng.random((2, n)))).astype(np.float32)
    lay = md.Layered(w=np.full(n, 1.0), h=np.full(n, 1.0), kind=np.zeros(n, np.uint8), layer=layer,
                     net_start=np.arange(0, 601, 2, dtype=np.int32), pin2node=rng.permutation(n)[:600].astype(np.int32),
                     pin_off=np.zeros((2, 600)), grid=md.Grid2D(die, die, 64, 64), gamma=10.0, ramp=1.05, target=1.0,
                     n_inst=n, n_hbt=0)
    prob = place3d.MultiDie2D.from_layered(lay, fixed_xy=xy)
    st = prob.new_state()
    x = torch.from_numpy(xy).cuda()
    for t in (st.u, st.v):
        t.copy_(x)
    st.v_prev.copy_(x + 0.01)
    st.scalars[place3d.MS["a"]] = 1.0
    st.scalars[place3d.MS["lam_bot"]:place3d.MS["lam_bot"] + 3] = 1.0
    prob.step(st)
    s, want = st.read(), md.overflow_2d(lay, xy.astype(np.float64))
    log(f"[overflow] {[s[k] for k in ('ovfl_bot', 'ovfl_top', 'ovfl_hbt')]}, oracle {want}")
    assert min(want) > 1e-3 and min(abs(want[0] - want[1]), abs(want[1] - want[2])) > 1e-3
    for k, w in zip(("ovfl_bot", "ovfl_top", "ovfl_hbt"), want):
        assert abs(s[k] - w) <= 1e-6, (k, s[k], w)
