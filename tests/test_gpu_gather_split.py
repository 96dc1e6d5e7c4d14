"""The field gather of tiles that its launch keeps whole though the chunk plan splits them: between 320 and 767
tiles up to twice the mean tile's entries, where the mean tile's chunks would not all be in one round, from 768
tiles on up to 1536 entries.

Values against the oracle with the split tiles' bar (rel L2 <= 1e-5).  Time: 676 tiles are one round on the
chip, as 256 are, for 2.6 times the work: 1.6 times as long when every tile is whole, 1.9 with all of
them split into two chunks."""
import numpy as np
import pytest
import torch

from gpu_common import gpu_problem, log, need_gpu, rel_l2
from oracle import density_grad as odg
from oracle.geometry import geometry_of
from paper_2403_09070_amd import place3d, synth

pytestmark = pytest.mark.gpu


def crowded(nx, ny, counts, rest, seed=3):
    """Small cells, counts[k] of them in the middle of tile k of the first row of 32 x 32 bin tiles, `rest` a tile
    all over, and six large instances."""
    n = sum(counts) + rest * (-(-nx // 32) * -(-ny // 32))
    case = synth.make_case(config=synth.small_config(n_cells=n, n_nets=10, die=2.0 * max(nx, ny), nx=nx, ny=ny, nz=2,
                                                     macros=("uniform", 6, 0.001, 0.003)), seed=seed)
    rng = np.random.default_rng(seed)
    wb, hb = case.die_x / nx, case.die_y / ny
    cell = np.nonzero(case.kind == 0)[0]
    case.size[:, cell] = np.float32(min(wb, hb) / 3)
    tile = np.repeat(np.arange(len(counts)), counts)
    case.xyz0[0, cell[:tile.size]] = (32 * tile + rng.uniform(8, 24, tile.size)) * wb
    case.xyz0[1, cell[:tile.size]] = rng.uniform(8, 24, tile.size) * hb
    return case


@pytest.mark.parametrize("nx,ny", [(512, 608), (512, 640), (760, 1000), (736, 1024), (768, 1024), (800, 1000)])   # 304 .. 800 tiles
@pytest.mark.parametrize("rest", [2, 1100])       # a mean tile of one chunk and of two
def test_whole_and_split_tiles(nx, ny, rest):
    need_gpu()
    tiles = -(-nx // 32) * -(-ny // 32)
    log(f"[gather split] {nx} x {ny}, {tiles} tiles, {rest} cells a tile")
    counts = [1024, 1025, 1535, 1536, 1537, 3000, 5000, 9000]
    case = crowded(nx, ny, counts, rest)
    prob = gpu_problem(case, precision=place3d.FP32)
    rng = np.random.default_rng(1)
    maps = [rng.normal(size=(case.nz, ny, nx)).astype(np.float32) for _ in range(3)]
    g = prob.field_force(case.xyz0, *(torch.from_numpy(m).cuda() for m in maps), lam=1.0).cpu().numpy()
    ref = odg.field_gather(case.size, case.kind, case.xyz0, *(m.astype(np.float64) for m in maps), geometry_of(case))
    err = rel_l2(g, ref)
    log(f"[gather split] {tiles} tiles: {err:.2e}")
    assert err <= 1e-5


def test_a_grid_of_one_round_keeps_its_tiles_whole():
    need_gpu()
    times = []
    for side in (512, 832):
        log(f"[gather split] uniform map on {side} x {side}")
        n, die = 1000 * (side // 32) ** 2, 1600.0 * side / 512
        rng = np.random.default_rng(1)
        xyz = (rng.random((3, n)) * np.array([[die], [die], [2 * die / side]]) + np.array([[0], [0], [die / side]])).astype(np.float32)
        size = np.ones((4, n), np.float32)
        prob = place3d.Problem(size=size, kind=np.zeros(n, np.uint8), net_start=np.zeros(1, np.int32),
                               pin2node=np.zeros(0, np.int32), pin_off=np.zeros((4, 0), np.float32), fixed_xyz=xyz,
                               die_x=die, die_y=die, nx=side, ny=side, nz=4, gamma=1.0, alpha=0.0)
        x, e = prob.xyz(xyz), [torch.rand(4, side, side, device="cuda") for _ in range(3)]
        ms = []
        for _ in range(12):
            prob.profile(True, ["dgrad"])
            for _ in range(4):
                prob.field_force(x, *e, lam=1.0)
            ms.append(prob.profile_read()["dgrad"][0])
            prob.profile(False)
        times.append(float(np.median(ms)))
    log(f"[gather split] 676 tiles {times[1] / times[0]:.2f} of 256")
    assert times[1] <= 1.75 * times[0]
