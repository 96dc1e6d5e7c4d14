"""The split-bf16 contractions of the solve against the oracle on grids of several tiles that they alone take: the
chain with halves that are no multiple of its tiles, k blocks or lanes, and the general contraction.

Tolerance: an operand keeps 16 significant bits, so that each of the four contractions rounds its data and
its basis by at most 2^-18 and drops a product of two remainders of at most 2^-9; twelve errors of up to
2^-18, evenly spread and independent, are 7.6e-6 of a norm, and three times that is the bar.  The map's
largest variations are its lowest frequencies, so that neither the potential nor a component of the
field (taken against |E|) is a small remainder."""
import numpy as np
import pytest

from gpu_common import log, need_gpu, rel_l2
from oracle import poisson as opois
from oracle.geometry import Geometry
from test_gpu_fft import problem

pytestmark = pytest.mark.gpu
TOL = 2.3e-5


@pytest.mark.parametrize("nx,ny,nz", [(700, 562, 2), (662, 406, 4), (1022, 386, 4), (576, 256, 6)])
def test_split_solve_matches_the_oracle(nx, ny, nz):
    need_gpu()
    import torch
    log(f"[split chain] {nx}x{ny}x{nz}")
    x, y = np.pi * (np.arange(nx) + 0.5) / nx, np.pi * (np.arange(ny) + 0.5) / ny
    rng = np.random.default_rng(nx)
    rho = 0.1 * rng.random((nz, ny, nx))
    for z in range(nz):
        for i, j in ((1, 0), (0, 1), (1, 1), (2, 1), (1, 3)):
            rho[z] += (rng.random() - 0.5) / (i + j) * np.cos(j * y)[:, None] * np.cos(i * x)
    rho = rho.astype(np.float32)
    dev = torch.from_numpy(rho).cuda()
    out = problem(nx, ny, nz, 1).field(dev)
    assert not torch.equal(out["ex"], problem(nx, ny, nz, 0).field(dev, want=("ex",))["ex"]), "not the split form"
    ref = opois.solve(rho.astype(np.float64), Geometry(2.0 * nx, 3.0 * ny, nx, ny, nz))
    norm = np.sqrt(sum(np.linalg.norm(ref[k]) ** 2 for k in ("ex", "ey", "ez")))
    errs = {k: np.linalg.norm(out[k].cpu().numpy() - ref[k]) / norm for k in ("ex", "ey", "ez")}
    errs["phi"] = rel_l2(out["phi"].cpu().numpy(), ref["phi"])
    log(f"[split chain] {nx}x{ny}x{nz} " + " ".join(f"{k} {e:.2e}" for k, e in errs.items()))
    assert max(errs.values()) <= TOL
