"""The sizes at which passes change how they share their launches: the scatter that adds up the tiles'
counts itself against the scan pass (32768 counts, 4096 tiles), the wide density workgroups (256 tiles)
and the move that sums the step's norms
itself against a reduction (512 partials, 131072 instances; multi-die 2048 and 524288 nodes).

Density maps against the oracle with the parity tests' bar (rel L2 <= 1e-6).  A step's size against
its definition, |v_k - v_{k-1}| / |g_k - g_{k-1}| in float64 from the state before and after: 1.6M
additions of non-negative terms on either side, each within 1.1e-16, leave at most 2 * 1.7e-10 of the
squares, so 1e-9 of their ratio."""
import numpy as np
import pytest
import torch

from gpu_common import gpu_problem, log, need_gpu, rel_l2
from oracle import density as oden
from oracle.geometry import geometry_of
from paper_2403_09070_amd import place3d, synth

pytestmark = pytest.mark.gpu


def sized_case(n_inst, nx, ny, die):
    return synth.make_case(config=synth.small_config(n_cells=n_inst - 3, n_nets=300, die=die, nx=nx, ny=ny, nz=2), seed=9)


@pytest.mark.parametrize("n_inst,nx,ny", [(32 * 2048, 1024, 1024), (32 * 2048 + 1, 1024, 1024),     # 32 and 33 x 1024
                                          (2048, 2048, 2048), (2048, 2049, 2048), (5000, 40, 1000),
                                          (9000, 512, 512), (9000, 513, 512)])
def test_counts_added_by_either_pass(n_inst, nx, ny):
    need_gpu()
    log(f"[launches] {n_inst} instances on {nx} x {ny}")
    case = sized_case(n_inst, nx, ny, 2.0 * max(nx, ny))
    assert case.n_inst == n_inst
    ref = oden.density_map(case.size, case.kind, case.xyz0, geometry_of(case))
    got = gpu_problem(case, precision=place3d.FP32).density(case.xyz0).cpu().numpy()
    assert rel_l2(got, ref) <= 1e-6


@pytest.mark.parametrize("n_inst", [700, 512 * 256, 512 * 256 + 1])
def test_step_size_from_either_reduction(n_inst):
    need_gpu()
    log(f"[launches] step of {n_inst} instances")
    case = sized_case(n_inst, 64, 64, 40.0 + 2.2 * n_inst ** 0.5)
    assert case.n_inst == n_inst and not (case.kind & 2).any()
    prob = gpu_problem(case, precision=place3d.FP32)
    st = prob.gp_init(case.xyz0)
    prob.step(st)
    v, vp, g = st.v.double().clone(), st.v_prev.double().clone(), st.g_prev.double().clone()
    prob.step(st)
    want = float(torch.sqrt(((v - vp) ** 2).sum() / ((st.g_prev.double() - g) ** 2).sum()))
    got = st.read()["step"]
    assert abs(got - want) <= 1e-9 * want
    s = st.read()
    assert np.isfinite([s["ovfl_bot"], s["ovfl_top"], s["hpwl"]]).all() and s["ovfl_bot"] + s["ovfl_top"] > 0


@pytest.mark.parametrize("n", [900, 2048 * 256, 2048 * 256 + 1])
def test_multi_die_step_size_from_either_reduction(n):
    need_gpu()
    log(f"[launches] multi-die step of {n} nodes")
    rng = np.random.default_rng(n)
    die = 40.0 + 2.0 * n ** 0.5
    layer = rng.integers(0, 3, n).astype(np.uint8)
    xy = (die * (0.1 + 0.8 * rng.random((2, n)))).astype(np.float32)
    nets = rng.permutation(n)[:600].reshape(300, 2)
    prob = place3d.MultiDie2D(size=np.ones((2, n), np.float32), kind=np.zeros(n, np.uint8), layer=layer,
                              net_start=np.arange(0, 601, 2, dtype=np.int32), pin2node=nets.reshape(-1).astype(np.int32),
                              pin_off=np.zeros((2, 600), np.float32), fixed_xy=xy, die_x=die, die_y=die, nx=64, ny=64,
                              gamma=10.0)
    st = prob.gp_init(xy)
    prob.step(st)
    v, vp, g = st.v.double().clone(), st.v_prev.double().clone(), st.g_prev.double().clone()
    prob.step(st)
    want = float(torch.sqrt(((v - vp) ** 2).sum() / ((st.g_prev.double() - g) ** 2).sum()))
    assert abs(st.read()["step"] - want) <= 1e-9 * want


@pytest.mark.parametrize("n_inst", [1 << 20, (1 << 20) + 1])
def test_steps_of_large_split_problems_solve_by_contractions(n_inst):
    """Up to 2^20 instances a split-bf16 step takes the float32 transforms (its gradient within 1e-6 of
    the plain form's: the same field, compensated wirelength sums), from there on the split
    contractions, whose field differs by their rounding (some 4e-6); both meet the bar of 1e-4, and
    the field call takes the transforms either way."""
    need_gpu()
    log(f"[launches] split step of {n_inst} instances")
    case = sized_case(n_inst, 64, 64, 2400.0)
    assert case.n_inst == n_inst
    g, f = [], []
    for precision in (place3d.FP32, place3d.BF16X3):
        prob = gpu_problem(case, precision=precision)
        st = prob.new_state()
        x = prob.xyz(case.xyz0)
        for t in (st.u, st.v):
            t.copy_(x)
        st.v_prev.copy_(x + 0.01)
        st.g_prev.zero_()
        st.scalars.zero_()
        st.scalars[place3d.S["a"]] = 1.0
        st.scalars[place3d.S["lam"]] = 1.0
        prob.step(st)
        g.append(st.g_prev.double())
        rho = prob.density(case.xyz0)
        f.append(prob.field(rho, want=("ex", "ez")))
    err = float((g[0] - g[1]).norm() / g[0].norm())
    log(f"[launches] {n_inst}: gradient of the split form {err:.2e} from the plain one")
    assert err <= 1e-4 and (err <= 1e-6) == (n_inst <= 1 << 20)
    assert all(torch.equal(f[0][k], f[1][k]) for k in ("ex", "ez"))
