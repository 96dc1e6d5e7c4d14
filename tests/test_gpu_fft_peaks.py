"""The fast transforms on maps whose peaks stand far above the rest, as a crowded start's or a macro's do: one
bin, and a lattice of 64, over an even density.

A peak's rounding is the same wherever it stands, so that the error against the oracle at one place is
held to that at three others.  An error's norm is that of many bins for the field, of a few low
frequencies for the potential: two draws from two such components differ by more than 8 in one of 65
cases, the largest of three draws from a fourth far less."""
import numpy as np
import pytest

from gpu_common import log, need_gpu
from oracle import poisson as opois
from oracle.geometry import Geometry
from test_gpu_fft import problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz", [(64, 64, 2), (128, 512, 4), (1024, 1024, 2), (2048, 128, 4), (256, 2048, 2)])
@pytest.mark.parametrize("peaks", ["one", "lattice"])
def test_the_error_does_not_depend_on_where_peaks_stand(nx, ny, nz, peaks):
    need_gpu()
    import torch
    log(f"[fft] {nx}x{ny}x{nz} peaks: {peaks}")
    prob, geo = problem(nx, ny, nz), Geometry(2.0 * nx, 3.0 * ny, nx, ny, nz)
    lane = np.arange(64) if peaks == "lattice" else np.array([20])
    y, x = lane * (ny // 64) + ny // 128, (lane * 37 & 63) * (nx // 64) + nx // 128

    def errors(dy, dx):
        rho = 0.7 + 0.3 * np.random.default_rng(1).random((nz, ny, nx))
        rho[0, (y + dy) % ny, (x + dx) % nx] = 1e4 / len(lane) ** 0.5
        rho = rho.astype(np.float32)
        ref = opois.solve(rho.astype(np.float64), geo)
        out = prob.field(torch.from_numpy(rho).cuda())
        return {k: np.linalg.norm(out[k].cpu().numpy() - ref[k]) for k in ref}

    at, others = errors(0, 0), [errors(*d) for d in ((1, 1), (1, 3), (3, 1))]
    for k, e in at.items():
        most = max(o[k] for o in others)
        log(f"[fft] {nx}x{ny}x{nz} {peaks} {k} {e / most:.2f} of the error elsewhere")
        assert e <= 8 * most, k
