"""The fast transforms of the spectral solve against the FP64 oracle: every transform length, both
layer counts, every subset of outputs, and output maps that are not 16-byte aligned.

Tolerance: a float32 FFT of N points errs by at most about eps log2 N relative to its norm (eps =
6e-8); a map goes through four of them (two axes forward, two inverse) of at most 2048 points, so
4 * 11 * 6e-8 = 2.6e-6, and the tables and scalings add a few eps: 3e-6.  The map changes from layer to
layer as much as along the layers, so that no component of the field is a small remainder."""
import ctypes

import numpy as np
import pytest

from gpu_common import log, need_gpu, rel_l2
from oracle import poisson as opois
from oracle.geometry import Geometry

pytestmark = pytest.mark.gpu
TOL = 3e-6


def problem(nx, ny, nz, precision=0):
    from paper_2403_09070_amd import place3d
    size = np.ones((4, 1), np.float32)
    return place3d.Problem(size=size, kind=np.zeros(1, np.uint8), net_start=np.zeros(1, np.int32),
                           pin2node=np.zeros(0, np.int32), pin_off=np.zeros((4, 0), np.float32),
                           fixed_xyz=np.ones((3, 1), np.float32), die_x=2.0 * nx, die_y=3.0 * ny, nx=nx, ny=ny, nz=nz,
                           gamma=1.0, alpha=0.0, precision=precision)


def some_map(nx, ny, nz):
    rng = np.random.default_rng(nx + 3 * ny + 5 * nz)
    return (rng.random((nz, ny, nx)) ** 2 + np.arange(nz)[:, None, None]).astype(np.float32)


@pytest.mark.parametrize("nx,ny,nz", [(64, 64, 2), (64, 128, 4), (128, 64, 2), (256, 64, 4), (64, 256, 2), (512, 64, 4),
                                      (128, 512, 4), (1024, 64, 2), (64, 1024, 4), (2048, 64, 4), (64, 2048, 2),
                                      (64, 2048, 4), (1024, 256, 4)])
@pytest.mark.parametrize("precision", [0, 1])
def test_every_length_matches_the_oracle(nx, ny, nz, precision):
    need_gpu()
    import torch
    log(f"[fft] {nx}x{ny}x{nz} precision {precision}")
    rho = some_map(nx, ny, nz)
    prob = problem(nx, ny, nz, precision)
    ref = opois.solve(rho.astype(np.float64), Geometry(2.0 * nx, 3.0 * ny, nx, ny, nz))
    dev = torch.from_numpy(rho).cuda()
    out = prob.field(dev)
    for k in ref:
        err = rel_l2(out[k].cpu().numpy(), ref[k])
        log(f"[fft] {nx}x{ny}x{nz} {k} {err:.2e}")
        assert err <= TOL, k
    for want in (("phi",), ("ex",), ("ey",), ("ez",), ("ex", "ey", "ez")):
        part = prob.field(dev, want=want)
        assert all(torch.equal(part[k], out[k]) for k in want), want


@pytest.mark.parametrize("nx,ny,nz", [(512, 2048, 4), (1024, 2048, 4)])
def test_sixteen_rows_a_workgroup_match_the_oracle(nx, ny, nz):
    """Maps of 8192 rows and more, where the x pass takes sixteen rows a workgroup at every side."""
    test_every_length_matches_the_oracle(nx, ny, nz, 0)


@pytest.mark.parametrize("nx,ny,nz", [(64, 64, 4), (1024, 128, 2)])
def test_unaligned_maps_give_the_same_values(nx, ny, nz):
    """The map and the outputs at 4-byte aligned addresses (a slice of a larger array)."""
    need_gpu()
    import torch
    from paper_2403_09070_amd import place3d
    prob = problem(nx, ny, nz)
    rho = torch.from_numpy(some_map(nx, ny, nz)).cuda()
    ref = prob.field(rho)
    n = rho.numel()
    odd = [torch.zeros(n + 8, device="cuda")[1:1 + n] for _ in range(5)]
    odd[0].copy_(rho.reshape(-1))
    ptr = [ctypes.c_void_p(t.data_ptr()) for t in odd]
    rc = place3d.lib().place3d_field(prob._ctx, *ptr, None, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    for t, k in zip(odd[1:], ("phi", "ex", "ey", "ez")):
        assert torch.equal(t.reshape(rho.shape), ref[k]), k
