"""Crowded density tiles in the forms that share the split of a heavy tile: more than 256 tiles (narrow workgroups),
fillers (two sums a bin), more than 2^20 entries in a tile (chunks beyond the smallest size, so that
their number stays bounded), and the layers of a multi-die problem, one of them crowded, in one launch.

Against the oracle with the parity tests' bars: maps rel L2 <= 1e-6, overflow 1e-6 absolute (at most 16
float32 terms a thread, then float64).  A second call gives the same bits: the chunk counters are zero again."""
import dataclasses

import numpy as np
import pytest
import torch

from gpu_common import gpu_problem, log, need_gpu, oracle_problem, rel_l2
from oracle import density as oden
from oracle import multidie as md
from oracle import optimizer as opt
from oracle.geometry import geometry_of
from paper_2403_09070_amd import place3d, synth

pytestmark = pytest.mark.gpu

FILLER = 4


def crowded_case(cells, nx, ny, nz, fillers):
    """Cells of a third of a bin in the middle of one tile (every seventeenth anywhere), six large instances; with
    fillers, every third cell without a pin is one."""
    case = synth.make_case(config=synth.small_config(n_cells=cells, n_nets=40, die=2.0 * max(nx, ny), nx=nx, ny=ny, nz=nz,
                                                     macros=("uniform", 6, 0.002, 0.01)), seed=31)
    rng = np.random.default_rng(cells)
    xyz, size, kind = case.xyz0.copy(), case.size.copy(), case.kind.copy()
    wb, hb = case.die_x / nx, case.die_y / ny
    cell = np.nonzero(kind == 0)[0]
    size[:, cell] = np.float32(min(wb, hb) / 3)
    far = np.arange(cell.size) % 17 == 0
    xyz[0, cell[~far]] = rng.uniform(8, 24, (~far).sum()) * wb
    xyz[1, cell[~far]] = rng.uniform(8, 24, (~far).sum()) * hb
    if fillers:
        free = np.setdiff1d(cell, case.pin2node)
        kind[free[::3]] = FILLER
    return dataclasses.replace(case, xyz0=xyz.astype(np.float32), size=size, kind=kind)


@pytest.mark.parametrize("cells,nx,ny,nz,fillers", [(20000, 640, 416, 2, False), (75000, 640, 416, 2, False),
                                                    (20000, 48, 80, 4, True), (120000, 48, 80, 4, True),
                                                    (120000, 640, 416, 4, True), (1200000, 48, 80, 2, False)])
def test_crowded_tiles(cells, nx, ny, nz, fillers):
    need_gpu()
    log(f"[split shapes] {cells} cells on {nx} x {ny} x {nz}, fillers {fillers}")
    case = crowded_case(cells, nx, ny, nz, fillers)
    prob = gpu_problem(case, precision=place3d.FP32)
    got = prob.density(case.xyz0).cpu().numpy()
    again = prob.density(case.xyz0).cpu().numpy()
    ref = oden.density_map(case.size, case.kind, case.xyz0, geometry_of(case))
    log(f"[split shapes] density {rel_l2(got, ref):.2e}")
    assert rel_l2(got, ref) <= 1e-6 and np.array_equal(got, again)
    st = prob.new_state()
    x = prob.xyz(case.xyz0)
    for t in (st.u, st.v):
        t.copy_(x)
    st.v_prev.copy_(x + 0.01)
    st.scalars[place3d.S["a"]] = 1.0
    st.scalars[place3d.S["lam"]] = 1.0
    prob.step(st)
    s = st.read()
    want = opt.overflow(oracle_problem(case), ref, case.xyz0.astype(np.float64))
    log(f"[split shapes] overflow {s['ovfl_bot']:.7f} {s['ovfl_top']:.7f}, oracle {want[0]:.7f} {want[1]:.7f}")
    assert min(want) > 0
    assert abs(s["ovfl_bot"] - want[0]) <= 1e-6 and abs(s["ovfl_top"] - want[1]) <= 1e-6


@pytest.mark.parametrize("crowd", [0, 2])
def test_layers_of_uneven_crowds(crowd):
    need_gpu()
    log(f"[split shapes] layer {crowd} crowded")
    rng = np.random.default_rng(crowd)
    count = [700, 90, 12]
    count[crowd] = 90000
    layer = rng.permutation(np.repeat(np.arange(3), count)).astype(np.uint8)
    n, die = layer.size, 300.0
    xy = rng.uniform(3, die - 3, (2, n))
    heavy = layer == crowd
    xy[:, heavy] = rng.uniform(40, 110, (2, int(heavy.sum())))
    xy = xy.astype(np.float32)
    nets = rng.permutation(n)[:600]
    lay = md.Layered(w=np.full(n, 1.0), h=np.full(n, 1.0), kind=np.zeros(n, np.uint8), layer=layer,
                     net_start=np.arange(0, 601, 2, dtype=np.int32), pin2node=nets.astype(np.int32),
                     pin_off=np.zeros((2, 600)), grid=md.Grid2D(die, die, 64, 64), gamma=10.0, ramp=1.05, target=1.0,
                     n_inst=n, n_hbt=0)
    prob = place3d.MultiDie2D.from_layered(lay, fixed_xy=xy)
    for _ in range(2):
        rho = prob.eval(xy)[2].cpu().numpy()
        for L in range(3):
            on = layer == L
            ref = md.density_2d(lay.w[on], lay.h[on], xy[:, on].astype(np.float64), lay.grid)
            log(f"[split shapes] layer {L} {rel_l2(rho[L], ref):.2e}")
            assert rel_l2(rho[L], ref) <= 1e-6
    st = prob.new_state()
    x = torch.from_numpy(xy).cuda()
    for t in (st.u, st.v):
        t.copy_(x)
    st.v_prev.copy_(x + 0.01)
    st.scalars[place3d.MS["a"]] = 1.0
    st.scalars[place3d.MS["lam_bot"]:place3d.MS["lam_bot"] + 3] = 1.0
    prob.step(st)
    s, want = st.read(), md.overflow_2d(lay, xy.astype(np.float64))
    for k, w in zip(("ovfl_bot", "ovfl_top", "ovfl_hbt"), want):
        assert abs(s[k] - w) <= 1e-6, (k, s[k], w)
