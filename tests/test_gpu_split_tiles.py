"""Density tiles on the edges of their splits: all cells in one tile, with the tile whole, split in
two, in as many chunks as one workgroup adds up, and in one more, and large instances shared by the
chunks.

Against the oracle with the bars of the small-case parity tests: density map rel L2 <= 1e-6 (float32
overlaps, sums in integers), field gather and exact adjoint rel L2 <= 1e-5.  Repeated calls must give
the same map bit for bit (the chunk counters are left at zero).
"""
import dataclasses

import numpy as np
import pytest
import torch

from gpu_common import gpu_problem, log, need_gpu, rel_l2
from oracle import density as oden
from oracle import density_grad as odg
from oracle.geometry import geometry_of
from paper_2403_09070_amd import place3d, synth

pytestmark = pytest.mark.gpu

DENSITY, CHUNK, GATHER, GROUP = 8192, 4096, 1024, 16   # entries a tile, a chunk may hold; chunks one workgroup adds up
COUNTS = [GATHER, GATHER + 1, DENSITY, DENSITY + 1, GROUP * CHUNK, GROUP * CHUNK + 1, 68 * CHUNK + 7]


def one_tile_case(cells):
    """`cells` cells of a third of a bin at random in the middle half of tile (0, 0) of a 48 x 80 grid,
    six large instances with their centres in the same tile."""
    case = synth.make_case(config=synth.small_config(n_cells=cells, n_nets=40, die=240.0, nx=48, ny=80, nz=4,
                                                     macros=("uniform", 6, 0.01, 0.04)), seed=31)
    rng = np.random.default_rng(cells)
    xyz, size = case.xyz0.copy(), case.size.copy()
    wb, hb = case.die_x / case.nx, case.die_y / case.ny
    n = case.n_inst
    xyz[0] = rng.uniform(8, 24, n) * wb
    xyz[1] = rng.uniform(8, 24, n) * hb
    cell = case.kind == 0
    size[:, cell] = np.float32(min(wb, hb) / 3)
    case = dataclasses.replace(case, xyz0=xyz.astype(np.float32), size=size)
    # no cell edge within 1e-3 of a bin face: the adjoint is one-sided there
    geo = geometry_of(case)
    while True:
        box, _ = oden.footprints(case.size, case.kind, case.xyz0, geo)
        edge = np.stack([box[k] / d for k, d in zip(range(6), (geo.wb, geo.wb, geo.hb, geo.hb, geo.db, geo.db))])
        near = cell & (np.abs(edge - np.round(edge)).min(axis=0) < 1e-3)
        if not near.any():
            return case
        case.xyz0[0, near] = rng.uniform(8, 24, near.sum()) * wb
        case.xyz0[1, near] = rng.uniform(8, 24, near.sum()) * hb
        case.xyz0[2, near] = rng.uniform(0.3, 0.7, near.sum()) * geo.dz


@pytest.mark.parametrize("cells", COUNTS)
def test_split_edges(cells):
    need_gpu()
    log(f"[split] {cells} cells in one tile")
    case = one_tile_case(cells)
    assert int((case.kind == 0).sum()) == cells
    geo = geometry_of(case)
    prob = gpu_problem(case, precision=place3d.FP32)
    ref = oden.density_map(case.size, case.kind, case.xyz0, geo)
    got = prob.density(case.xyz0).cpu().numpy()
    again = prob.density(case.xyz0).cpu().numpy()
    rng = np.random.default_rng(1)
    maps = [rng.normal(size=(case.nz, case.ny, case.nx)).astype(np.float32) for _ in range(3)]
    g = prob.field_force(case.xyz0, *(torch.from_numpy(m).cuda() for m in maps), lam=1.0).cpu().numpy()
    gref = odg.field_gather(case.size, case.kind, case.xyz0, *(m.astype(np.float64) for m in maps), geo)
    a = prob.density_vjp(case.xyz0, torch.from_numpy(maps[0]).cuda()).cpu().numpy()
    aref = odg.density_vjp(case.size, case.kind, case.xyz0, maps[0].astype(np.float64), geo)
    log(f"[split] {cells}: density {rel_l2(got, ref):.3e} gather {rel_l2(g, gref):.3e} adjoint {rel_l2(a, aref):.3e}")
    assert rel_l2(got, ref) <= 1e-6
    assert np.array_equal(got, again)
    assert rel_l2(g, gref) <= 1e-5 and rel_l2(a, aref) <= 1e-5
