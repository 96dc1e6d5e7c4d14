"""Timed cases of the placement library: what a placer's program asks of it, over the sizes it meets.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges; ``prepare`` builds what
the program holds before the call (a problem with its context, positions, an optimiser state),
``run`` makes one pass through the public calls and returns what they computed, ``work`` counts the
bytes and operations that a pass cannot do without, and ``exact`` evaluates the same formulas in
float64 with plain torch.

The kinds of pass:
  step     one global-placement iteration (Problem.step), the inner loop of a placer
  md2d     one iteration of the multi-die 2D placement that follows (MultiDie2D.step)
  penalty  density map, field and field-gather gradient by separate calls, as a program with an
           optimiser of its own makes them
  chain    density and potential as autograd functions, forward and backward
  field    the spectral solve alone
  wl       wirelength gradient and metrics (Problem.wl_grad)
  wlfun    the wirelength as an autograd function, forward and backward

Steps run with a constant density weight (lambda_ramp = 1): a weight that grows at every pass would
overflow after some ten thousand of them.  The float64 records (optimiser scalars, metrics) are
kept as float32, as a placer's log holds them: they are sums of terms computed in float32.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2403_09070_amd import autograd, place3d

DEV = "cuda"
MACRO, FIXED, FILLER, ZFIXED = 1, 2, 4, 8
TOP_SCALE = 0.7           # top-die sizes and pin offsets relative to the bottom die's
WINDOW = 256              # index half-window of a local net

_DEFAULT = dict(kind="step", cells=2000, macros=4, macro_share=0.1, fixed=False, fillers=0, degree="geo", local=0.9,
                die=200.0, nx=64, ny=64, nz=2, precision="fp32", dgrad="field", spread="uniform")


def _case(name, **kw):
    c = dict(_DEFAULT, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    mixed = dict(precision="bf16x3")
    c4 = dict(cells=1_200_000, macros=150, macro_share=0.15, degree="mix", die=4000.0, nx=1024, ny=1024, nz=4)
    return [
        # a small block placed interactively: the iteration is launches and latency
        _case("step 2k fp32", fixed=True, macro_share=0.12),
        # an ordinary block: 200k cells under 40 macros that cover a good part of the die
        _case("step 200k mixed", cells=200_000, macros=40, macro_share=0.5, die=2000.0, nx=512, ny=512, nz=4, **mixed),
        # the benchmark's workload in both precisions
        _case("step 1.2M mixed", **c4, **mixed),
        _case("step 1.2M fp32", **c4),
        # a design filled up with dummy cells, stepped with the exact adjoint of the density map
        _case("step 20k+300k fillers adjoint", cells=20_000, macros=12, macro_share=0.2, fillers=300_000, die=600.0,
              nx=256, ny=256, nz=4, dgrad="adjoint"),
        # the start of a placement: every instance around the centre of the die
        _case("penalty 1.2M centred", **dict(c4, kind="penalty", spread="centre")),
        # a differentiable density model on a grid whose sides are no powers of two
        _case("chain 150k 420x380", kind="chain", cells=150_000, macros=20, macro_share=0.2, die=1600.0, nx=420, ny=380,
              nz=4),
        # the solve alone: largest power-of-two grid in use, and a small odd one
        _case("field 2048x2048x4 mixed", kind="field", cells=64, die=8000.0, nx=2048, ny=2048, nz=4, **mixed),
        _case("field 75x61x6 fp32", kind="field", cells=64, die=240.0, nx=75, ny=61, nz=6),
        # wirelength of a netlist without index locality, every member drawn over the whole design
        _case("wl 600k scattered mixed", kind="wl", cells=600_000, macros=80, degree="mix", local=0.0, die=2800.0,
              nx=512, ny=512, nz=4, **mixed),
        # the differentiable wirelength of a small ragged netlist
        _case("wlfun 31k", kind="wlfun", cells=31_013, macros=9, degree="mix", die=800.0, nx=200, ny=200, nz=4),
        # planar refinement of a finished 3D placement on its three layers
        _case("md2d 300k mixed", kind="md2d", cells=300_000, macros=30, macro_share=0.2, die=2400.0, nx=512, ny=512,
              nz=2, **mixed),
    ]


def draw(rng):
    """A case of the listed ranges: 2k to 1.2M cells, grids of about one bin per cell, powers of two
    (as placers choose them) in two draws of three and any sides else."""
    log = lambda lo, hi: math.exp(rng.uniform(math.log(lo), math.log(hi)))  # noqa: E731
    kind = rng.choice(["step", "step", "step", "md2d", "penalty", "chain", "field", "wl", "wlfun"])
    cells = int(log(2000, 300_000 if kind == "md2d" else 1_100_000))
    side = math.sqrt(cells * rng.uniform(0.9, 2.0))
    if rng.random() < 0.67:
        nx = 1 << round(math.log2(side))
        ny = nx if rng.random() < 0.7 else max(64, nx // 2)
        nz = rng.choice([2, 4, 4, 4])
    else:
        nx = int(min(side, 400) * rng.uniform(0.8, 1.1))
        ny = int(min(side, 400) * rng.uniform(0.8, 1.1))
        nz = rng.choice([2, 4, 4, 6])
    nx, ny = min(nx, 1024), min(ny, 1024)
    # separate calls and autograd run in the binding's default precision, steps in both
    spread = "centre" if kind in ("penalty", "chain") and rng.random() < 0.4 else "uniform"
    # (the adjoint on blocks: on large grids the float32 potential leaves its differences few digits)
    adjoint = kind == "step" and cells < 60_000 and rng.random() < 0.5
    mixed = kind not in ("penalty", "chain") and not adjoint and rng.random() < 0.6
    macros = rng.randint(3, 8 + cells // 10_000)
    fillers = int(cells * rng.uniform(0.5, 2.0)) if kind == "step" and cells < 300_000 and rng.random() < 0.3 else 0
    return _case("", kind=kind, cells=cells, macros=macros, macro_share=round(rng.uniform(0.05, 0.4), 3),
                 fixed=kind == "step" and rng.random() < 0.2, fillers=fillers, degree=rng.choice(["geo", "mix"]),
                 local=rng.choice([0.9, 0.9, 0.0]), die=round(3.7 * math.sqrt(cells * rng.uniform(1.0, 1.4)), 1),
                 nx=nx, ny=ny, nz=2 if kind == "md2d" else nz, precision="bf16x3" if mixed else "fp32",
                 dgrad="adjoint" if adjoint else "field", spread=spread)


# ---------------------------------------------------------------- inputs

class _Geo:
    """Bin and region sizes of a case (float64)."""

    def __init__(self, c):
        self.n = (c["nx"], c["ny"], c["nz"])
        self.die = (c["die"], c["die"])
        self.wb, self.hb = c["die"] / c["nx"], c["die"] / c["ny"]
        self.db = 0.5 * (self.wb + self.hb)
        self.dz = c["nz"] * self.db
        self.step = (self.wb, self.hb, self.db)
        self.length = (c["die"], c["die"], self.dz)
        self.vol = self.wb * self.hb * self.db
        self.gamma = 2.0 * self.wb
        eta = 2.0 / 1.7                       # HBT pitch 1, rows 0.7 and 1
        self.alpha = 3.5e-3 * (c["die"] * eta * eta / self.dz) * math.log(900.0 * eta - 1.0)
        self.lam = 0.8 / self.dz              # about one over a mean cell's charge


def _rand(gen, *shape):
    return torch.rand(*shape, generator=gen, device=DEV, dtype=torch.float64)


def _instances(c, gen):
    """size [4][n], kind [n], xyz [3][n]: cells, macros, fillers."""
    g = _Geo(c)
    nc, nm, nf = c["cells"], c["macros"], c["fillers"]
    w, h = torch.floor(1.0 + 4.0 * _rand(gen, nc)), torch.ones(nc, device=DEV, dtype=torch.float64)
    area = 0.5 + 1.5 * _rand(gen, nm)
    area = area / area.sum() * c["macro_share"] * c["die"] ** 2
    aspect = 0.5 + 1.5 * _rand(gen, nm)
    side = math.sqrt(2.5)
    fill = torch.full((nf,), side, device=DEV, dtype=torch.float64)
    w = torch.cat([w, (area * aspect).sqrt(), fill])
    h = torch.cat([h, (area / aspect).sqrt(), fill])
    size = torch.stack([w, h, TOP_SCALE * w, TOP_SCALE * h])
    kind = torch.zeros(nc + nm + nf, device=DEV, dtype=torch.uint8)
    kind[nc:nc + nm] = MACRO | (FIXED if c["fixed"] else 0)
    kind[nc + nm:] = FILLER
    kind[nc + nm:nc + nm + nf // 2] = FILLER | ZFIXED
    n = nc + nm + nf
    xyz = torch.empty(3, n, device=DEV, dtype=torch.float64)
    if c["spread"] == "centre":
        for a, (mid, dev) in enumerate(((0.5 * c["die"], 0.02 * c["die"]), (0.5 * c["die"], 0.02 * c["die"]),
                                        (0.5 * g.dz, 0.05 * g.dz))):
            xyz[a] = mid + dev * torch.randn(n, generator=gen, device=DEV, dtype=torch.float64)
    else:
        xyz[0] = w / 2 + _rand(gen, n) * (c["die"] - w)
        xyz[1] = h / 2 + _rand(gen, n) * (c["die"] - h)
        xyz[2] = g.dz / 4 + _rand(gen, n) * g.dz / 2
    held = (kind & ZFIXED) != 0
    xyz[2, held] = (0.25 + 0.5 * (_rand(gen, int(held.sum())) < 0.5).double()) * g.dz
    return size.float(), kind, xyz.float()


def _nets(c, gen):
    """net_start, pin2node (int64): nets in anchor order, members spread over an index window (or
    the whole design), one in fifty with a macro on one pin."""
    nc, nm = c["cells"], c["macros"]
    m = int(1.08 * nc)
    if c["degree"] == "geo":
        d = torch.arange(2, 21, device=DEV)
        p = 0.621 ** (d - 2.0)
    else:
        d = torch.arange(2, 51, device=DEV)
        body = 0.5 ** (d - 2.0)
        tail = torch.where(d >= 7, d ** -2.5, torch.zeros_like(body))
        p = 0.9545 * body / body.sum() + 0.0455 * tail / tail.sum()
    cdf = torch.cumsum((p / p.sum()).double(), 0)
    deg = d[torch.searchsorted(cdf, _rand(gen, m)).clamp(max=d.numel() - 1)]
    anchor = torch.sort(torch.floor(_rand(gen, m) * nc)).values
    local = _rand(gen, m) < c["local"]
    width = torch.where(local, float(min(2 * WINDOW + 1, nc)), float(nc))
    lo = torch.where(local, torch.minimum((anchor - WINDOW).clamp(min=0), nc - width), 0.0)
    start = torch.zeros(m + 1, device=DEV, dtype=torch.int64)
    torch.cumsum(deg, 0, out=start[1:])
    net = torch.repeat_interleave(torch.arange(m, device=DEV), deg)
    k = torch.arange(net.numel(), device=DEV) - start[net]
    # one member from each of `degree` equal parts of the window: distinct members
    part = torch.floor(width[net] / deg[net])
    node = (lo[net] + k * part + torch.floor(_rand(gen, net.numel()) * part)).long()
    swap = (_rand(gen, m) < 0.02)[net] & (k == torch.floor(_rand(gen, m) * deg)[net])
    macro = nc + torch.floor(_rand(gen, m) * nm).long()
    return start, torch.where(swap, macro[net], node)


def _offsets(size, node, gen):
    off = torch.stack([(_rand(gen, node.numel()) - 0.5) * size[a, node] for a in range(2)])
    return torch.cat([off, TOP_SCALE * off]).float()


def _inputs(case, seed):
    """Every array of a case, from its seed alone (device tensors)."""
    c = dict(_DEFAULT, **case)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    g = _Geo(c)
    d = {}
    if c["kind"] == "field":
        nx, ny, nz = g.n
        size, kind, xyz = _instances(dict(c, cells=64, macros=1, macro_share=0.001), gen)
        # a map like a placement's: occupancy that changes from bin to bin, over broad hills
        rho = 1.5 * _rand(gen, nz, ny, nx) ** 2
        x = torch.arange(nx, device=DEV, dtype=torch.float64) / nx
        y = torch.arange(ny, device=DEV, dtype=torch.float64) / ny
        hill = _rand(gen, nz, 4).cpu().tolist()
        for z in range(nz):
            cx, cy, s, top = hill[z]
            sy, sx = torch.exp(-(y - cy) ** 2 * (9 + 40 * s)), torch.exp(-(x - cx) ** 2 * 20)
            rho[z] += top * sy[:, None] * sx[None, :]
        d["rho"] = rho.float()
    elif c["kind"] == "md2d":
        return _md_inputs(c, gen)
    else:
        size, kind, xyz = _instances(c, gen)
    d.update(size=size, kind=kind, xyz=xyz)
    n = kind.numel()
    if c["kind"] in ("step", "wl", "wlfun"):
        d["start"], d["node"] = _nets(c, gen)
        d["off"] = _offsets(size, d["node"], gen)
    else:
        d["start"] = torch.zeros(1, device=DEV, dtype=torch.int64)
        d["node"], d["off"] = d["start"][:0], torch.zeros(4, 0, device=DEV)
    if c["kind"] == "chain":
        # what a loss with an overflow term on the map and an energy term on the potential sends back;
        # the second's share reaches the map with about the size of the first
        bins = math.prod(g.n)
        d["g_rho"] = (_rand(gen, *reversed(g.n)) - 0.5).float()
        d["g_phi"] = (5.0 * math.sqrt(bins) / c["die"] ** 2 * (_rand(gen, *reversed(g.n)) - 0.5)).float()
    if c["kind"] == "step":
        move = torch.tensor([g.wb, g.hb, 0.1 * g.dz], device=DEV, dtype=torch.float64)[:, None]
        fixed = (kind & FIXED) != 0
        held = fixed | ((kind & ZFIXED) != 0)
        v = _clamp(size.double(), kind, xyz.double(), g)
        near = {}
        for name, amp in (("u", 0.2), ("v_prev", 0.4)):
            p = amp * move * torch.randn(3, n, generator=gen, device=DEV, dtype=torch.float64)
            p[:, fixed] = 0
            p[2, held] = 0
            near[name] = _clamp(size.double(), kind, v + p, g).float()
        gp = 0.3 * torch.randn(3, n, generator=gen, device=DEV, dtype=torch.float64)
        gp[:, fixed] = 0
        gp[2, held] = 0
        d.update(u=near["u"], v=v.float(), v_prev=near["v_prev"], g_prev=gp.float(), a=2.5, lam=g.lam)
    return d


def _md_inputs(c, gen):
    """Nodes of three layers (instances at their die's size, a bonding terminal per crossing net)
    and the partial nets, with an optimiser state.  Even instances sit on the bottom die, odd ones
    on top; three nets of five cross."""
    size4, kind, xyz = _instances(dict(c, fixed=False, fillers=0), gen)
    start, node = _nets(c, gen)
    g = _Geo(c)
    n0, m = kind.numel(), start.numel() - 1
    net = torch.repeat_interleave(torch.arange(m, device=DEV), start[1:] - start[:-1])
    k = torch.arange(net.numel(), device=DEV) - start[net]
    crossing = net % 5 < 3
    die = torch.where(crossing, torch.where(k < 2, k, node % 2), net % 2)
    node = torch.where(2 * (node // 2) + die < n0, 2 * (node // 2) + die, die)
    top = torch.arange(n0, device=DEV) % 2
    part = 2 * net + die
    cross = (torch.arange(m, device=DEV) % 5 < 3).nonzero().flatten()
    nb = cross.numel()
    hbt = n0 + torch.arange(nb, device=DEV)
    all_part = torch.cat([part, 2 * cross, 2 * cross + 1])
    all_node = torch.cat([node, hbt, hbt])
    order = torch.sort(all_part, stable=True).indices
    deg = torch.bincount(all_part, minlength=2 * m)
    deg = deg[deg > 0]
    pstart = torch.zeros(deg.numel() + 1, device=DEV, dtype=torch.int64)
    torch.cumsum(deg, 0, out=pstart[1:])
    pnode = all_node[order]
    size = torch.cat([torch.where(top.bool(), size4[2:], size4[:2]), torch.ones(2, nb, device=DEV)], 1)
    first = node[start[:-1]][cross]
    xy = torch.cat([xyz[:2], xyz[:2, first]], 1)
    kind = torch.cat([kind, torch.zeros(nb, device=DEV, dtype=torch.uint8)])
    layer = torch.cat([top, torch.full((nb,), 2, device=DEV)]).to(torch.uint8)
    off = torch.stack([(_rand(gen, pnode.numel()) - 0.5) * size[a, pnode] for a in range(2)])
    off[:, pnode >= n0] = 0
    n = kind.numel()
    v = _clamp2(size.double(), xy.double(), g)
    noise = lambda: torch.randn(2, n, generator=gen, device=DEV, dtype=torch.float64)  # noqa: E731
    near = {k: _clamp2(size.double(), v + amp * g.wb * noise(), g).float() for k, amp in (("u", 0.2), ("v_prev", 0.4))}
    gp = 0.3 * noise()
    return dict(size=size, kind=kind, layer=layer, start=pstart, node=pnode, off=off.float(), u=near["u"], v=v.float(),
                v_prev=near["v_prev"], g_prev=gp.float(), a=2.5, lam=0.4)


def _precision(c):
    return place3d.BF16X3 if c["precision"] == "bf16x3" else place3d.FP32


def prepare(case, seed):
    c = dict(_DEFAULT, **case)
    d = _inputs(c, seed)
    g = _Geo(c)
    h = lambda t, dt=None: t.cpu().numpy() if dt is None else t.to(dt).cpu().numpy()  # noqa: E731
    nets = dict(net_start=h(d["start"], torch.int32), pin2node=h(d["node"], torch.int32), pin_off=h(d["off"]))
    if c["kind"] == "md2d":
        prob = place3d.MultiDie2D(size=h(d["size"]), kind=h(d["kind"]), layer=h(d["layer"]), **nets,
                                  fixed_xy=np.zeros((2, d["kind"].numel()), np.float32), die_x=c["die"], die_y=c["die"],
                                  nx=c["nx"], ny=c["ny"], gamma=g.gamma, lambda_ramp=1.0, precision=_precision(c))
    else:
        prob = place3d.Problem(size=h(d["size"]), kind=h(d["kind"]), **nets, fixed_xyz=h(d["xyz"]), die_x=c["die"],
                               die_y=c["die"], nx=c["nx"], ny=c["ny"], nz=c["nz"], gamma=g.gamma, alpha=g.alpha,
                               lambda_ramp=1.0, precision=_precision(c),
                               dgrad=place3d.DGRAD_ADJOINT if c["dgrad"] == "adjoint" else place3d.DGRAD_FIELD)
    s = dict(kind=c["kind"], prob=prob)
    if c["kind"] in ("step", "md2d"):
        st = prob.new_state()
        for name in ("u", "v", "v_prev", "g_prev"):
            getattr(st, name).copy_(d[name])
        st.scalars[0] = d["a"]
        st.scalars[1:2 if c["kind"] == "step" else 4] = d["lam"]
        s["state"] = st
    elif c["kind"] == "field":
        s["rho"] = d["rho"]
    else:
        s["xyz"] = d["xyz"]
        if c["kind"] == "chain":
            s["g"] = [d["g_rho"], d["g_phi"]]
    return s


# ---------------------------------------------------------------- passes

def run(state):
    kind, prob = state["kind"], state["prob"]
    if kind in ("step", "md2d"):
        st = state["state"]
        prob.step(st)
        return {"u": st.u, "v": st.v, "v_prev": st.v_prev, "g_prev": st.g_prev, "record": st.scalars.float()}
    if kind == "field":
        return prob.field(state["rho"])
    xyz = state["xyz"]
    if kind == "penalty":
        rho = prob.density(xyz)
        f = prob.field(rho, want=("ex", "ey", "ez"))
        return {"rho": rho, **f, "grad": prob.field_force(xyz, f["ex"], f["ey"], f["ez"])}
    if kind == "wl":
        grad, met = prob.wl_grad(xyz)
        return {"grad": grad, "metrics": met.float()}
    x = xyz.detach().requires_grad_()
    if kind == "chain":
        rho = autograd.Density.apply(prob, x)
        phi = autograd.Field.apply(prob, rho)
        torch.autograd.backward([rho, phi], state["g"])
        return {"rho": rho.detach(), "phi": phi.detach(), "grad": x.grad}
    w = autograd.wirelength(prob, x)
    w.backward()
    return {"value": w.detach().float(), "grad": x.grad}


def work(case):
    """Inputs once and outputs once; transforms as fast ones (2.5 N log2 N each), about 12 operations
    per overlapped bin, 120 per pin and 60 per moved node."""
    c = dict(_DEFAULT, **case)
    kind, n = c["kind"], c["cells"] + c["macros"] + c["fillers"]
    bins = c["nx"] * c["ny"] * c["nz"]
    pins = int(1.08 * c["cells"] * 3.5)
    solve = lambda k: 2.5 * k * bins * math.log2(bins)  # noqa: E731
    cells = n * 18 * 12
    net = 24 * pins + 4 * 1.08 * c["cells"]
    if kind == "step":
        return {"bytes": 17 * n + net + 96 * n, "flops": solve(7) + 2 * cells + 120 * pins + 60 * n}
    if kind == "md2d":
        n, pins = int(1.25 * n), int(1.15 * pins)
        return {"bytes": 10 * n + 16 * pins + 64 * n, "flops": 3 * solve(3) + 2 * cells + 80 * pins + 40 * n}
    if kind == "field":
        return {"bytes": 4 * bins * 5, "flops": solve(9)}
    if kind == "penalty":
        return {"bytes": 29 * n + 16 * bins + 12 * n, "flops": solve(7) + 2 * cells}
    if kind == "chain":
        return {"bytes": 29 * n + 12 * bins + 12 * n, "flops": 2 * solve(4) + 2 * cells}
    return {"bytes": net + 12 * n + 12 * n, "flops": (120 if kind == "wl" else 180) * pins}


# ---------------------------------------------------------------- the formulas in float64

def _wh(size, kind, z, g):
    """Widths and heights at z: a cell's by its die, a macro's linear between the dies."""
    top = z > 0.5 * g.dz
    t = 2.0 * z.clamp(0.25 * g.dz, 0.75 * g.dz) / g.dz
    mac = (kind & MACRO) != 0
    return [torch.where(mac, (t - 0.5) * size[2 + k] + (1.5 - t) * size[k], torch.where(top, size[2 + k], size[k]))
            for k in range(2)]


def _clamp2(size, xy, g):
    return torch.stack([torch.minimum(torch.maximum(xy[a], 0.5 * size[a]), g.die[a] - 0.5 * size[a]) for a in range(2)])


def _clamp(size, kind, xyz, g):
    z = xyz[2].clamp(0.25 * g.dz, 0.75 * g.dz)
    w, h = _wh(size, kind, z, g)
    out = torch.stack([torch.minimum(torch.maximum(xyz[0], 0.5 * w), g.die[0] - 0.5 * w),
                       torch.minimum(torch.maximum(xyz[1], 0.5 * h), g.die[1] - 0.5 * h), z])
    return torch.where((kind & FIXED) != 0, xyz, out)


def _clip(e, L):
    """Edges clipped to [0, L]; an edge within 2^-20 L of a face is on it and moves into the region."""
    moves = (e >= -L * 2.0 ** -20) & (e <= L * (1 + 2.0 ** -20))
    c = e.clamp(0.0, L).detach()
    return c + torch.where(moves, e - e.detach(), 0.0) if e.requires_grad else c


def _boxes(w, h, pos, g):
    """Stretched, clipped extents (lo, hi) per axis and the weight of every instance; two axes, or
    three with the depth of half the stack."""
    r2 = math.sqrt(2.0)
    half = [0.5 * w.clamp(min=r2 * g.wb), 0.5 * h.clamp(min=r2 * g.hb)]
    if len(pos) == 3:
        half.append(torch.full_like(w, 0.25 * g.dz))
    box = [(_clip(p - e, L), _clip(p + e, L)) for p, e, L in zip(pos, half, g.length)]
    return box, (w / (r2 * g.wb)).clamp(max=1.0) * (h / (r2 * g.hb)).clamp(max=1.0)


def _overlap(lo, hi, b, step):
    b0, b1 = b.double() * step, (b.double() + 1) * step
    return (torch.where(hi <= b1 * (1 + 1e-12), hi, b1) - torch.where(lo >= b0, lo, b0)).clamp(min=0.0)


def _bins(box, g):
    """First and last bin per axis of every box."""
    out = []
    for (lo, hi), step, n in zip(box, g.step, g.n):
        b0 = torch.floor(lo.detach() / step).long().clamp(0, n - 1)
        b1 = (torch.ceil(hi.detach() / step).long() - 1).clamp(0, n - 1)
        out.append((b0, torch.maximum(b0, b1)))
    return out


def _sweep(box, weight, g, cell, large):
    """Calls cell(flat bins, overlaps) for the small boxes, span by span, and large(slices, overlaps)
    for each box of more than twelve bins on a planar axis."""
    rng = _bins(box, g)
    wide = ((rng[0][1] - rng[0][0]) > 12) | ((rng[1][1] - rng[1][0]) > 12)
    small = (~wide).nonzero().flatten()
    if small.numel():
        spans = [int((r1 - r0)[small].max()) + 1 for r0, r1 in rng]
        per_axis = []
        for a in range(len(box)):
            row = []
            for o in range(spans[a]):
                b = rng[a][0][small] + o
                row.append((b.clamp(max=g.n[a] - 1), torch.where(b <= rng[a][1][small], _overlap(
                    box[a][0][small], box[a][1][small], b, g.step[a]), 0.0)))
            per_axis.append(row)
        zs = per_axis[2] if len(box) == 3 else [(torch.zeros_like(small), 1.0)]
        for bz, lz in zs:
            for by, ly in per_axis[1]:
                for bx, lx in per_axis[0]:
                    cell(small, (bz * g.n[1] + by) * g.n[0] + bx, weight[small] * lx * ly * lz)
    for i in wide.nonzero().flatten().tolist():
        ov, sl = [], []
        for a in range(len(box)):
            b0, b1 = int(rng[a][0][i]), int(rng[a][1][i])
            b = torch.arange(b0, b1 + 1, device=DEV)
            ov.append(_overlap(box[a][0][i], box[a][1][i], b, g.step[a]))
            sl.append(slice(b0, b1 + 1))
        v = weight[i] * ov[1][:, None] * ov[0][None, :]
        large(i, tuple(reversed(sl)), v if len(box) == 2 else ov[2][:, None, None] * v)


def _density(box, weight, g):
    d = len(box)
    shape, vol = tuple(reversed(g.n[:d])), math.prod(g.step[:d])
    rho = torch.zeros(shape, device=DEV, dtype=torch.float64)
    flat = rho.view(-1)

    def large(i, sl, v):
        rho[sl] += v

    _sweep(box, weight, g, lambda i, b, v: flat.index_add_(0, b, v), large)
    return rho / vol


def _gather(box, weight, g, maps):
    """sum_b weight vol(D ∩ b) map_b per instance, for each map."""
    out = torch.zeros(len(maps), weight.numel(), device=DEV, dtype=torch.float64)

    def cell(i, b, v):
        for k, m in enumerate(maps):
            out[k, i] += v * m.reshape(-1)[b]

    def large(i, sl, v):
        for k, m in enumerate(maps):
            out[k, i] = (v * m[sl]).sum()

    _sweep(box, weight, g, cell, large)
    return out


def _along(m, mat, axis):
    """Contract an axis of m with mat[sample, out]."""
    m = m.movedim(axis, -1).contiguous()
    return (m.reshape(-1, m.shape[-1]) @ mat).reshape(*m.shape[:-1], mat.shape[1]).movedim(-1, axis)


def _solve(rho, g, want):
    """Potential and field of a map by cosine series, dense transforms; two or three axes."""
    d = rho.dim()
    cos, sin, om = [], [], []
    a = rho
    for k in range(d):
        n, L = g.n[k], g.length[k]
        i, j = torch.arange(n, device=DEV, dtype=torch.float64), torch.arange(n, device=DEV, dtype=torch.float64)
        arg = math.pi * (i[:, None] + 0.5) * j[None, :] / n
        cos.append(torch.cos(arg))
        om.append(math.pi * j / L)
        sin.append(torch.sin(arg) * om[k][None, :])
        norm = torch.full((n,), 2.0 / n, device=DEV, dtype=torch.float64)
        norm[0] = 1.0 / n
        a = _along(a, cos[k] * norm, d - 1 - k)
    w2 = om[0][None, :] ** 2 + om[1][:, None] ** 2
    if d == 3:
        w2 = w2 + om[2][:, None, None] ** 2
    b = torch.where(w2 > 0, a / w2.clamp(min=1e-300), 0.0)
    out = {}
    for name, axis in (("phi", -1), ("ex", 0), ("ey", 1), ("ez", 2)):
        if name in want:
            m = b
            for k in range(d):
                m = _along(m, (sin if k == axis else cos)[k].T.contiguous(), d - 1 - k)
            out[name] = m.contiguous()
    return out


def _wa(u, mask, gamma):
    """Weighted-average extent of the masked members of each row and its derivative."""
    any_ = mask.any(1, keepdim=True)
    inf = float("inf")
    hi = torch.where(any_, torch.where(mask, u, -inf).amax(1, keepdim=True), 0.0)
    lo = torch.where(any_, torch.where(mask, u, inf).amin(1, keepdim=True), 0.0)
    um = torch.where(mask, u, 0.0)
    ep = torch.where(mask, torch.exp(torch.where(mask, u - hi, 0.0) / gamma), 0.0)
    em = torch.where(mask, torch.exp(torch.where(mask, lo - u, 0.0) / gamma), 0.0)
    sp = torch.where(any_, ep.sum(1, keepdim=True), 1.0)
    sm = torch.where(any_, em.sum(1, keepdim=True), 1.0)
    # relative to the extremes: the sums then do not cancel
    ap = (torch.where(mask, um - hi, 0.0) * ep).sum(1, keepdim=True) / sp
    am = (torch.where(mask, um - lo, 0.0) * em).sum(1, keepdim=True) / sm
    grad = ep / sp * (1 + (u - hi - ap) / gamma) - em / sm * (1 - (u - lo - am) / gamma)
    return torch.where(any_, hi - lo + ap - am, 0.0)[:, 0], torch.where(mask, grad, 0.0)


def _extent(u, mask):
    hi = torch.where(mask, u, -float("inf")).amax(1)
    lo = torch.where(mask, u, float("inf")).amin(1)
    return torch.where(mask.any(1), hi - lo, 0.0)


def _bistratal(u, top):
    return torch.maximum(_extent(u, torch.ones_like(top)), _extent(u, top) + _extent(u, ~top))


def _wirelength(d, pos, g, alpha):
    """Gradient parts per instance and totals of the bistratal model; pos [3][n] (two dies) or
    [2][n] (every net on one layer)."""
    n = pos.shape[1]
    gx, gy, gz, fda = (torch.zeros(n, device=DEV, dtype=torch.float64) for _ in range(4))
    tot = dict(wa_bi=0.0, wa_z=0.0, hpwl=0.0, hpwl3d=0.0, ncut=0.0)
    start, node, off = d["start"], d["node"], d["off"].double()
    deg = start[1:] - start[:-1]
    two = pos.shape[0] == 3
    for k in torch.unique(deg).tolist():
        nets = (deg == k).nonzero().flatten()
        for part in nets.split(max(1, 4_000_000 // max(k, 1))):
            if k == 0:
                continue
            pins = start[part][:, None] + torch.arange(k, device=DEV)
            nd = node[pins]
            top = pos[2, nd] > 0.5 * g.dz if two else torch.zeros_like(nd, dtype=torch.bool)
            cur, oth = [], []
            for a in range(2):
                bot, upp = off[a][pins], off[(2 if two else 0) + a][pins]
                cur.append(pos[a, nd] + torch.where(top, upp, bot))
                oth.append(pos[a, nd] + torch.where(top, bot, upp))
            crossing = top.any(1) & (~top).any(1)
            everyone = torch.ones_like(top)
            now = torch.zeros(part.numel(), device=DEV, dtype=torch.float64)
            for a, grad in ((0, gx), (1, gy)):
                pe, ge = _wa(cur[a], everyone, g.gamma)
                pt, gt = _wa(cur[a], top, g.gamma)
                pb, gb = _wa(cur[a], ~top, g.gamma)
                split = crossing & (pt + pb > pe)
                tot["wa_bi"] += float(torch.where(split, pt + pb, pe).sum())
                share = torch.where(split[:, None], torch.where(top, gt, gb), ge)
                grad.index_add_(0, nd.reshape(-1), share.reshape(-1))
                now = now + _bistratal(cur[a], top)
                tot["hpwl3d"] += float(_extent(cur[a], everyone).sum())
            tot["hpwl"] += float(now.sum())
            tot["ncut"] += float(crossing.sum())
            if not two:
                continue
            z = pos[2, nd]
            pz, gzz = _wa(z, everyone, g.gamma)
            tot["wa_z"] += alpha * float(pz.sum())
            tot["hpwl3d"] += alpha * float(_extent(z, everyone).sum())
            gz.index_add_(0, nd.reshape(-1), alpha * gzz.reshape(-1))
            for j in range(k):                       # every member in turn on the other die
                t2 = top.clone()
                t2[:, j] = ~t2[:, j]
                flip = torch.zeros_like(now)
                for a in range(2):
                    u2 = cur[a].clone()
                    u2[:, j] = oth[a][:, j]
                    flip = flip + _bistratal(u2, t2)
                dw = torch.where(top[:, j], now - flip, flip - now)
                fda.index_add_(0, nd[:, j], 4.0 / g.dz * dw)
    fixed = (d["kind"] & FIXED) != 0
    for t in (gx, gy, gz, fda):
        t[fixed] = 0.0
    norm = [float(t.abs().sum()) for t in (gx, gy, fda)]
    scale = (norm[0] + norm[1]) / (2 * norm[2]) if norm[2] > 0 else 0.0
    met = [tot["wa_bi"], tot["wa_z"], tot["hpwl"], tot["hpwl3d"], tot["ncut"], *norm, scale]
    return torch.stack([gx, gy, scale * fda + gz]), met


def _adjoint(size, kind, xyz, g, gmap):
    """Gradient of sum_b gmap_b rho_b."""
    x = xyz.clone().requires_grad_()
    box, weight = _boxes(*_wh(size, kind, x[2], g), x, g)
    parts = []
    flat = gmap.reshape(-1)
    _sweep(box, weight, g, lambda i, b, v: parts.append((flat[b] * v).sum()),
           lambda i, sl, v: parts.append((gmap[sl] * v).sum()))
    grad, = torch.autograd.grad(torch.stack(parts).sum() / g.vol, x)
    return torch.where((kind & FIXED) != 0, 0.0, grad)


def _move(d, grad, clamp, movable):
    """The optimiser's move from a preconditioned gradient: new u, v and the step."""
    u, v, vp, gp = (d[k].double() for k in ("u", "v", "v_prev", "g_prev"))
    dv, dg = ((v - vp)[:, movable] ** 2).sum(), ((grad - gp)[:, movable] ** 2).sum()
    step = float((dv / dg).sqrt()) if float(dg) > 0 else 0.0
    a1 = 0.5 * (1 + math.sqrt(4 * d["a"] ** 2 + 1))
    un = clamp(v - step * grad)
    vn = clamp(un + (d["a"] - 1) / a1 * (un - u))
    fixed = ~movable
    un[:, fixed], vn[:, fixed] = u[:, fixed], v[:, fixed]
    return un, vn, v, step, a1


def _exact_step(c, d, g):
    size, kind, v = d["size"].double(), d["kind"], d["v"].double()
    fixed, filler, held = (kind & FIXED) != 0, (kind & FILLER) != 0, (kind & ZFIXED) != 0
    w, h = _wh(size, kind, v[2], g)
    box, weight = _boxes(w, h, v, g)
    rho = _density(box, weight, g)
    wl, met = _wirelength(d, v, g, g.alpha)
    energy = 0.0
    if c["dgrad"] == "adjoint":
        phi = _solve(rho, g, ("phi",))["phi"]
        energy = 0.5 * float((rho * phi).sum()) * g.vol
        den = _adjoint(size, kind, v, g, phi * g.vol)
    else:
        f = _solve(rho, g, ("ex", "ey", "ez"))
        den = -_gather(box, weight, g, [f["ex"], f["ey"], f["ez"]])
    wl[2, held] = 0.0
    den[2, held] = 0.0
    q = w * h * 0.5 * g.dz
    npins = torch.bincount(d["node"], minlength=kind.numel()).double()
    H = torch.where((kind & MACRO) != 0, npins + d["lam"] * q, d["lam"] * q).clamp(min=1.0)
    grad = (wl + d["lam"] * den) / H
    grad[:, fixed] = 0.0
    un, vn, vp, step, a1 = _move(d, grad, lambda p: _clamp(size, kind, p, g), ~fixed)
    if bool(filler.any()):
        rb, rw = [(lo[~filler], hi[~filler]) for lo, hi in box], weight[~filler]
        rho = _density(rb, rw, g)
    excess = (rho - 1.0).clamp(min=0.0) * g.vol
    half = g.n[2] // 2
    top = v[2] > 0.5 * g.dz
    rec = torch.zeros(32, dtype=torch.float64)
    rec[0], rec[1], rec[2], rec[3], rec[6] = a1, d["lam"], step, 1.0, energy
    for k, (ex, on) in enumerate(((excess[:half], ~top), (excess[half:], top))):
        charge = float(q[on & ~fixed & ~filler].sum())
        rec[4 + k] = float(ex.sum()) / charge if charge > 0 else 0.0
    rec[8:8 + len(met)] = torch.tensor(met)
    return {"u": un, "v": vn, "v_prev": vp, "g_prev": grad, "record": rec}


def _exact_md2d(c, d, g):
    size, kind, layer, v = d["size"].double(), d["kind"], d["layer"], d["v"].double()
    wl, met = _wirelength(d, v, g, 0.0)
    den = torch.zeros_like(v)
    rec = torch.zeros(32, dtype=torch.float64)
    for L in range(3):
        on = layer == L
        box, weight = _boxes(size[0, on], size[1, on], v[:, on], g)
        rho = _density(box, weight, g)
        f = _solve(rho, g, ("ex", "ey"))
        den[:, on] = -_gather(box, weight, g, [f["ex"], f["ey"]])
        area = float((size[0, on] * size[1, on]).sum())
        rec[10 + L] = float((rho - 1.0).clamp(min=0.0).sum()) * g.wb * g.hb / area
    lq = d["lam"] * size[0] * size[1]
    npins = torch.bincount(d["node"], minlength=kind.numel()).double()
    H = torch.where((kind & MACRO) != 0, npins + lq, lq).clamp(min=1.0)
    grad = (wl[:2] + d["lam"] * den) / H
    movable = torch.ones_like(on)
    un, vn, vp, step, a1 = _move(d, grad, lambda p: _clamp2(size, p, g), movable)
    rec[0], rec[1:4], rec[4], rec[5], rec[8], rec[9] = a1, d["lam"], step, 1.0, met[0], met[2]
    return {"u": un, "v": vn, "v_prev": vp, "g_prev": grad, "record": rec}


def exact(case, seed):
    c = dict(_DEFAULT, **case)
    d, g = _inputs(c, seed), _Geo(c)
    kind = c["kind"]
    if kind == "step":
        return _exact_step(c, d, g)
    if kind == "md2d":
        return _exact_md2d(c, d, g)
    if kind == "field":
        return _solve(d["rho"].double(), g, ("phi", "ex", "ey", "ez"))
    size, xyz = d["size"].double(), d["xyz"].double()
    if kind in ("wl", "wlfun"):
        grad, met = _wirelength(d, xyz, g, g.alpha)
        if kind == "wlfun":
            return {"value": torch.tensor(met[0] + met[1], dtype=torch.float64), "grad": grad}
        return {"grad": grad, "metrics": torch.tensor(met + [0.0] * (16 - len(met)), dtype=torch.float64)}
    box, weight = _boxes(*_wh(size, d["kind"], xyz[2], g), xyz, g)
    rho = _density(box, weight, g)
    if kind == "penalty":
        f = _solve(rho, g, ("ex", "ey", "ez"))
        return {"rho": rho, **f, "grad": -_gather(box, weight, g, [f["ex"], f["ey"], f["ez"]])}
    phi = _solve(rho, g, ("phi",))["phi"]
    back = d["g_rho"].double() + _solve(d["g_phi"].double(), g, ("phi",))["phi"]
    return {"rho": rho, "phi": phi, "grad": _adjoint(size, d["kind"], xyz, g, back)}
