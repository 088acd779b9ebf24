"""What a user of this framework has it do, as measurable cases: whole field
solves (FP64, mixed precision, learned), the field solves of a time step, a
mesh-adaptation step, a fluid step, and the correction network alone (forward,
and one training step), on trees from a few boxes to some 10^5.

The trees are the streamer shapes that the benchmark and the tests use: a
uniform base grid, refined around the charged shell of one or more streamer
channels, 2:1 nested.  They are rebuilt here from a distance criterion, so that
any size of the range can be drawn.  Right-hand sides, densities and network
data are made on the GPU from the seed.
"""
import functools

import numpy as np
import torch

from paper_1708_08434_amd import autotune, mg as M, nn as NN

DEV = "cuda:0"
E_CHARGE, EPS0 = 1.602176634e-19, 8.8541878128e-12
UNIT = dict(lo=(0.0, 0.0, 0.0), length=1.0, bc_type=(0,) * 6, bc_val=(0.0,) * 5 + (1.0,))
# a 40 mm domain between plates at 0 and 80 kV, Neumann sides (SI units)
PLATES = dict(lo=(0.0, 0.0, 0.0), length=0.04, bc_type=(1, 1, 1, 1, 0, 0), bc_val=(0.0,) * 5 + (80e3,))
# the unit domain with Neumann sides
NEUMANN = dict(lo=(0.0, 0.0, 0.0), length=1.0, bc_type=(1, 1, 1, 1, 0, 0), bc_val=(0.0,) * 5 + (1.0,))


def listed():
    return [
        # the smallest solve in use: a uniform 32^3 grid, launches only
        dict(name="solve_uniform32", kind="solve", shape="uniform", top=3, precision="fp64", bc="unit", tuned=False),
        # the small streamer of the parity tests, Neumann sides, no tuning (a mesh that lives for a few solves)
        dict(name="solve_small_neumann", kind="solve", shape="streamer", base=3, top=5, radius=0.04, tip=0.62, channels=1,
             precision="fp64", bc="neumann", tuned=False),
        # one streamer, base 64^3 + 4 levels: the ordinary static mesh, launch schedule tuned once per mesh
        dict(name="solve_streamer", kind="solve", shape="streamer", base=4, top=8, radius=0.02, tip=0.62, channels=1,
             precision="fp64", bc="unit", tuned=True),
        # two streamers, base 64^3 + 7 levels, 1.2e8 cells: the largest single-GPU configuration
        dict(name="solve_two_streamers", kind="solve", shape="streamer", base=4, top=11, radius=0.0068, tip=0.72, channels=2,
             precision="fp64", bc="unit", tuned=True),
        # mixed precision on a mesh of base 64^3 + 6 levels
        dict(name="solve_mixed", kind="solve", shape="streamer", base=4, top=10, radius=0.0115, tip=0.68, channels=2,
             precision="mixed", bc="unit", tuned=True),
        # a forest of independent trees of uneven size
        dict(name="solve_forest", kind="solve", shape="forest", trees=24, base=3, top=7, precision="fp64", bc="unit",
             tuned=False),
        # a field solve of a time-stepped run: new charge, two warm-started V-cycles, the field on every box
        dict(name="time_step", kind="time_step", base=4, top=8, radius=0.02, tip=0.62),
        # a mesh-adaptation step as the head moves: criterion, plan, new tree, transfer of the potential
        dict(name="regrid", kind="regrid", base=4, top=8, radius=0.02, tip=0.62),
        # a fluid step (two stages, two field solves) in SI units
        dict(name="fluid_step", kind="fluid_step", base=4, top=8, radius=0.02, tip=0.62),
        # the learned solve: a correction network after each V-cycle
        dict(name="solve_learned", kind="learned", base=4, top=9, radius=0.015, tip=0.66),
        # the network's forward pass over the leaf boxes of an ordinary mesh
        dict(name="nn_forward", kind="nn_forward", boxes=9473),
        # one training step of the network on a mini-batch (forward, backward, Adam)
        dict(name="nn_train", kind="nn_train", boxes=1024, pool=4096),
    ]


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "forest", "time_step", "regrid", "fluid_step", "learned", "nn_forward",
                       "nn_train"])
    radius, tip = round(rng.uniform(0.008, 0.025), 4), round(rng.uniform(0.55, 0.85), 3)
    if kind == "solve":
        base, prec, tuned = rng.choice([2, 3, 4]), rng.choice(["fp64", "fp64", "mixed"]), rng.random() < 0.5
        up = rng.randrange(8)  # refinement levels over the base grid; none: the uniform grid
        if up == 0:
            return dict(kind="solve", shape="uniform", top=base + rng.randrange(2), precision=prec, bc="unit", tuned=tuned)
        top = base + up
        if top > 9:  # the largest meshes: thin channels, as listed
            radius, tip = round(rng.uniform(0.004, 0.0068), 4), round(rng.uniform(0.72, 0.85), 3)
        return dict(kind="solve", shape="streamer", base=base, top=top, radius=radius, tip=tip, channels=rng.choice([1, 2]),
                    precision=prec, bc=rng.choice(["unit", "neumann", "plates"]), tuned=tuned)
    if kind == "forest":
        return dict(kind="solve", shape="forest", trees=round(2 ** rng.uniform(1, 5.5)), base=3, top=rng.choice([4, 5, 6, 7]),
                    precision=rng.choice(["fp64", "mixed"]), bc="unit", tuned=rng.random() < 0.5)
    if kind == "learned":
        return dict(kind="learned", base=rng.choice([3, 4]), top=rng.choice([6, 7, 8, 9]), radius=radius, tip=tip)
    if kind == "nn_forward":
        return dict(kind="nn_forward", boxes=round(2 ** rng.uniform(5, 17)) | 1)
    if kind == "nn_train":
        n = round(2 ** rng.uniform(4, 11.5))
        return dict(kind="nn_train", boxes=n, pool=n + rng.randrange(1, 3000))
    return dict(kind=kind, base=rng.choice([3, 4]), top=rng.choice([6, 7, 8, 9]), radius=radius, tip=tip)


# ------------------------------------------------------------------- meshes

_SH = 20
_OFF = np.array([(a, b, c) for c in (-1, 0, 1) for b in (-1, 0, 1) for a in (-1, 0, 1)], dtype=np.int64)
_CHILD = np.array([(a, b, c) for c in (0, 1) for b in (0, 1) for a in (0, 1)], dtype=np.int64)


def _pack(v):
    return (v[:, 0] << (2 * _SH)) | (v[:, 1] << _SH) | v[:, 2]


def _unpack(k):
    m = (1 << _SH) - 1
    return np.stack([k >> (2 * _SH), (k >> _SH) & m, k & m], axis=1)


def _grid(level):
    g = np.arange(1 << (level - 1))
    return np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)


def channels_of(case):
    """Streamer channels (top point, head centre) in the unit cube."""
    if case.get("channels", 1) == 1:
        return [((0.5, 0.5, 1.0), (0.5, 0.5, case["tip"]))]
    return [((0.45, 0.5, 1.0), (0.45, 0.5, case["tip"])), ((0.55, 0.5, 1.0), (0.55, 0.5, case["tip"] - 0.1))]


def _near(level, ijk, chans, radius):
    """Boxes that the charged shell of a channel crosses, with a 3-cell buffer."""
    h = 1.0 / (8 << (level - 1))
    c = (8 * ijk + 4) * h
    hit = np.zeros(len(c), dtype=bool)
    for p0, p1 in chans:
        p0, ax = np.array(p0), np.array(p1) - np.array(p0)
        length = np.linalg.norm(ax)
        t = np.clip((c - p0) @ (ax / length), 0.0, length)
        d = np.linalg.norm(c - (p0 + t[:, None] * (ax / length)), axis=1)
        hit |= np.abs(d - radius) <= (4 * np.sqrt(3.0) + 3) * h + 0.1 * radius
    return hit


def _tree(base, top, chans, radius):
    """Uniform to level `base`, then refined around the channels to `top`, 2:1 nested over 26 neighbours."""
    flag, cand = {}, _grid(base)
    for lev in range(base, top):
        cand = cand[_near(lev, cand, chans, radius)]
        flag[lev] = _pack(cand)
        cand = (2 * cand[:, None, :] + _CHILD).reshape(-1, 3)
    refined = {lev: _grid(lev) for lev in range(1, base)}
    below = np.zeros((0, 3), dtype=np.int64)
    for lev in range(top - 1, base - 1, -1):
        nb = (below[:, None, :] + _OFF).reshape(-1, 3)
        nb = nb[((nb >= 0) & (nb < (1 << lev))).all(axis=1)]
        refined[lev] = below = _unpack(np.unique(np.concatenate([flag[lev], _pack(nb >> 1)])))
    level, ijk = [np.ones(1, dtype=np.int32)], [np.zeros((1, 3), dtype=np.int64)]
    for lev in range(1, top):
        ijk.append((2 * refined[lev][:, None, :] + _CHILD).reshape(-1, 3))
        level.append(np.full(len(ijk[-1]), lev + 1, dtype=np.int32))
    return np.concatenate(level), np.concatenate(ijk).astype(np.int32)


def _forest_channels(case):
    """Per tree: its channel, radius and top level, the same for every seed."""
    r = np.random.default_rng(case["trees"])
    out = []
    for _ in range(case["trees"]):
        out.append(([((0.5, 0.5, 1.0), (0.5, 0.5, r.uniform(0.6, 0.85)))], r.uniform(0.015, 0.03),
                    int(r.integers(case["base"] + 1, case["top"] + 1))))
    return out


@functools.lru_cache(maxsize=4)
def _boxes(key):
    case = dict(key)
    if case.get("shape") == "uniform":
        lv = [_grid(lev) for lev in range(1, case["top"] + 1)]
        level = np.concatenate([np.full(len(g), q + 1, dtype=np.int32) for q, g in enumerate(lv)])
        return level, np.concatenate(lv).astype(np.int32), np.zeros(len(level), dtype=np.int32)
    if case.get("shape") == "forest":
        parts = [_tree(case["base"], top, ch, rad) for ch, rad, top in _forest_channels(case)]
        return (np.concatenate([p[0] for p in parts]), np.concatenate([p[1] for p in parts]),
                np.concatenate([np.full(len(p[0]), t, dtype=np.int32) for t, p in enumerate(parts)]))
    level, ijk = _tree(case["base"], case["top"], channels_of(case), case["radius"])
    return level, ijk, np.zeros(len(level), dtype=np.int32)


def boxes_of(case):
    keys = ("shape", "base", "top", "radius", "tip", "channels", "trees")
    return _boxes(tuple((k, case[k]) for k in keys if k in case))


def make_tree(case, dom):
    level, ijk, tree = boxes_of(case)
    return M.Tree(level, ijk, tree, device=DEV, **dom)


# ------------------------------------------------------------------ charges

def gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def shell(x, y, z, chans, radius, delta):
    """Charge of the channels: positive head layer, negative sides."""
    rho = torch.zeros_like(x)
    for p0, p1 in chans:
        r = torch.sqrt((x - p1[0]) ** 2 + (y - p1[1]) ** 2)
        side = -0.2 * torch.exp(-(((r - radius) / delta) ** 2) / 2) * (z >= p1[2])
        d = torch.sqrt(r ** 2 + (z - p1[2]) ** 2)
        head = torch.exp(-(((d - radius) / delta) ** 2) / 2) * (z < p1[2])
        rho += head + side
    return rho


def centres(level, ijk):
    """Cell centres of the boxes in the unit cube, [n][8][8][8] each."""
    h = 1.0 / (8.0 * 2.0 ** (level.double() - 1)).view(-1, 1, 1, 1)
    c = torch.arange(8, device=DEV, dtype=torch.float64) + 0.5
    i, j, k = (8 * ijk[:, a].double().view(-1, 1, 1, 1) for a in range(3))
    n = (len(level), 8, 8, 8)
    return (((i + c.view(1, 1, 1, 8)) * h).expand(n), ((j + c.view(1, 1, 8, 1)) * h).expand(n),
            ((k + c.view(1, 8, 1, 1)) * h).expand(n))


def rhs_of(case, t, seed, dz=0.0, amp=1e4):
    """b = -rho on every box of tree t: the channels' charge (its strength and
    head position from the seed) and 1e-3 of seeded noise."""
    g = gen(seed)
    out = torch.empty((t.n, 8, 8, 8), dtype=torch.float64, device=DEV)
    level, ijk = (torch.from_numpy(t.index(w).copy()).to(DEV) for w in (M.MG_IDX_LEVEL, M.MG_IDX_IJK))
    tree = torch.from_numpy(t.index(M.MG_IDX_TREE).copy()).to(DEV)
    ntree = int(t.info.n_trees)
    strength = (0.8 + 0.4 * torch.rand(ntree, generator=g, device=DEV, dtype=torch.float64)).tolist()
    shift = ((torch.rand(ntree, generator=g, device=DEV, dtype=torch.float64) - 0.5) * 2e-3).tolist()
    forest = _forest_channels(case) if case.get("shape") == "forest" else None
    for tr in range(ntree):
        sel = (tree == tr).nonzero().reshape(-1) if ntree > 1 else torch.arange(t.n, device=DEV)
        for part in sel.split(16384):
            x, y, z = centres(level[part], ijk[part])
            if case.get("shape") == "uniform":
                rho = 0.04 * torch.exp(-((x - 0.5 - shift[tr]) ** 2 + (y - 0.5) ** 2 + (z - 0.5) ** 2) / (2 * 0.05 ** 2))
            else:
                chans, rad = (forest[tr][:2] if forest else (channels_of(case), case["radius"]))
                chans = [(p0, (p1[0], p1[1], p1[2] + shift[tr] - dz)) for p0, p1 in chans]
                rho = shell(x, y, z, chans, rad, 0.1 * rad)
            out[part] = -amp * strength[tr] * rho
    out += 1e-3 * amp * 0.04 * (2 * torch.rand(out.shape, generator=g, device=DEV, dtype=torch.float64) - 1)
    return out


# ------------------------------------------------------------------ network

def params_of(seed):
    """A network whose correction is a damped smoothing step (the identity
    through pairs of channels, then a 27-point average) plus seeded noise: the
    size and the effect of a trained one."""
    r = np.random.default_rng(seed)
    w1, w2, w3 = (r.standard_normal(s) * a for s, a in (((16, 27), 0.05), ((16, 16, 27), 0.02), ((16, 27), 0.002)))
    for c in range(16):
        w1[c, 13] += 1.0 if c % 2 == 0 else -1.0
        w2[c, c, 13] += 1.0
        w3[c] += (-1.0 if c % 2 == 0 else 1.0) * (0.004 + 0.012 * (np.arange(27) == 13))
    b1, b2 = 0.01 * r.standard_normal(16), 0.01 * r.standard_normal(16)
    return np.concatenate([w1.ravel(), b1, w2.ravel(), b2, w3.ravel(), np.zeros(1)]).astype(np.float32)


def inputs_of(g, n):
    """Scaled residuals of n boxes with their ghost layer: smooth and rough
    parts of unit size, some face layers empty (coarser or refined neighbours)."""
    x = torch.randn((n, 10, 10, 10), generator=g, device=DEV)
    x = 0.5 * x + 2.0 * torch.nn.functional.avg_pool3d(x.unsqueeze(1), 3, 1, 1).squeeze(1)
    empty = torch.rand((n, 6), generator=g, device=DEV) < 0.2
    for d in range(6):
        layer = x.select(3 - d // 2, 9 if d % 2 else 0)
        layer.masked_fill_(empty[:, d].view(-1, 1, 1), 0.0)
    return x.contiguous()


# --------------------------------------------------------------- the calls

class State:
    pass


def prepare(case, seed):
    s = State()
    s.kind = case["kind"]
    if s.kind in ("nn_forward", "nn_train"):
        g = gen(seed)
        s.net = NN.Net(params_of(seed), device=DEV)
        n = case.get("pool", case["boxes"])
        s.x = inputs_of(g, n)
        if s.kind == "nn_train":
            s.target = -0.1 * s.x[:, 1:9, 1:9, 1:9].contiguous() + 0.02 * torch.randn((n, 8, 8, 8), generator=g, device=DEV)
            s.idx = torch.randperm(n, generator=g, device=DEV)[:case["boxes"]].to(torch.int32)
        return s
    si = s.kind == "fluid_step"
    s.t = t = make_tree(case, PLATES if si else dict(unit=UNIT, neumann=NEUMANN, plates=PLATES)[case.get("bc", "unit")])
    if case.get("tuned"):
        autotune.tune(t, M.MG_MIXED if case["precision"] == "mixed" else M.MG_FP64, use_cache=False)
    if s.kind == "solve":
        s.opts = dict(precision=M.MG_MIXED if case["precision"] == "mixed" else M.MG_FP64)
        amp = 1e4 if case["bc"] != "plates" else 1e4 * 80e3 / 0.04 ** 2
        t.set_field(M.MG_FIELD_RHS, rhs_of(case, t, seed, amp=amp))
        s.phi = torch.empty((t.n, 8, 8, 8), dtype=torch.float64, device=DEV)
    elif s.kind == "learned":
        s.net = NN.Net(params_of(seed), device=DEV)
        s.learned = NN.Learned(t)
        t.set_field(M.MG_FIELD_RHS, rhs_of(case, t, seed))
    elif s.kind == "time_step":
        # the head moves 1 um of a 40 mm domain per field solve, to and fro
        s.rhs = [rhs_of(case, t, seed, dz=q * 2.5e-5) for q in range(3)]
        s.turn = 0
        s.face = torch.empty((t.n, 3, 9, 8, 8), dtype=torch.float64, device=DEV)
        s.norm = torch.empty((t.n, 8, 8, 8), dtype=torch.float64, device=DEV)
        s.opts = t.opts()
        t.set_field(M.MG_FIELD_RHS, s.rhs[2])
        t.fmg_solve()
    elif s.kind == "regrid":
        # the head has moved since the mesh was made; the thresholds keep the finest level around the charge
        rhs = rhs_of(case, t, seed, dz=0.01)
        t.set_field(M.MG_FIELD_RHS, rhs)
        t.fmg_solve()
        t.set_field(M.MG_FIELD_RHS, rhs)
        s.case, s.c3 = case, 0.15 * float(t.refine_near().max())
    elif s.kind == "fluid_step":
        # 1e15 m^-3 background and a plasma blob at the head, the potential solved once
        g = gen(seed)
        level, ijk = (torch.from_numpy(t.index(w).copy()).to(DEV) for w in (M.MG_IDX_LEVEL, M.MG_IDX_IJK))
        x, y, z = centres(level, ijk)
        blob = 1e19 * torch.exp(-(((x - 0.5) ** 2 + (y - 0.5) ** 2 + (z - case["tip"]) ** 2) / 0.03 ** 2))
        rough = 1 + 0.3 * (2 * torch.rand(blob.shape, generator=g, device=DEV, dtype=torch.float64) - 1)
        s.ne, s.ni = (1e15 + blob * rough).contiguous(), (1e15 + 0.8 * blob).contiguous()
        field = np.linspace(0.0, 35e6, 1000)  # synthetic transport table, the paper's size
        alpha = 912000.0 * np.exp(-25992000.0 / np.maximum(field, 1e-3))
        t.fluid_bind(np.stack([0.03 + 0.02 * np.exp(-field / 1e7), 0.1 + 0.05 * field / 35e6, alpha], axis=1), 35e6)
        t.set_field(M.MG_FIELD_RHS, -E_CHARGE * (s.ni - s.ne) / EPS0)
        t.fmg_solve()
        s.dt = 1e-13
    return s


def run(s):
    if s.kind == "solve":
        st = s.t.fmg_solve(**s.opts)
        M.mg_field_get(s.t.h, M.MG_FIELD_PHI, s.phi.data_ptr())
        return dict(phi=s.phi, cycles=st["n_vcycles"])
    if s.kind == "learned":
        st = s.learned.solve(s.net)
        return dict(phi=s.t.get_field(M.MG_FIELD_PHI, to_numpy=False), cycles=st["n_vcycles"], kept=st["accepted"])
    if s.kind == "time_step":
        M.mg_field_set(s.t.h, M.MG_FIELD_RHS, s.rhs[s.turn].data_ptr())
        s.turn = (s.turn + 1) % 3
        M.mg_vcycle(s.t.h, s.opts, 2, stats=False)
        M.mg_efield(s.t.h, s.face.data_ptr(), s.norm.data_ptr())
        return dict(face=s.face, norm=s.norm)
    if s.kind == "regrid":
        near = s.t.refine_near()
        level, ijk, tree = M.mg_regrid_plan_near(s.t.h, near, s.c3, 0.125, s.case["top"])
        new = M.Tree(level, ijk, tree, device=DEV, **UNIT)
        M.mg_transfer(s.t.h, new.h)
        return dict(near=near, level=level, ijk=ijk, phi=new.get_field(M.MG_FIELD_PHI, to_numpy=False))
    if s.kind == "fluid_step":
        dt, s.dt = s.dt, M.mg_fluid_step(s.t.h, s.ne.data_ptr(), s.ni.data_ptr(), s.dt)
        return dict(ne=s.ne, ni=s.ni, dt=dt, next=s.dt)
    if s.kind == "nn_forward":
        return s.net.forward(s.x)
    loss = s.net.gradient(s.x, s.target, idx=s.idx)
    s.net.adam(lr=1e-3)
    return dict(loss=loss, grad=s.net.get_grad(), params=s.net.get_params())


# ------------------------------------------------------------------- volumes

def _counts(case):
    level, _, _ = boxes_of(case)
    n = np.bincount(level, minlength=int(level.max()) + 1)[1:].astype(float)
    leaves = 512.0 * (1 + (n.sum() - 1) * 7 / 8) if case.get("shape") != "forest" else 512.0 * n.sum() * 7 / 8
    return n, leaves


def _cycle_bytes(n, width):
    """A V(2,2) cycle: four sweeps and the transfers between levels, by 127
    bytes a stored cell in FP64 (three accesses a cell and half-sweep, the
    residual, the restriction and the prolongation)."""
    return 127.0 * width / 8 * 512 * n.sum()


def work(case):
    kind = case["kind"]
    if kind in ("nn_forward", "nn_train"):
        flop = 2.0 * 27 * (16 + 256 + 16) * 512 * case["boxes"]
        if kind == "nn_forward":
            return dict(bytes=case["boxes"] * 4.0 * 1512, flops=flop)
        return dict(bytes=case["boxes"] * 4.0 * (1000 + 512) + 7 * 4.0 * 7809, flops=3 * flop)
    n, leaves = _counts(case)
    cells = 512 * n.sum()
    flops = 9.0 * 4 * cells  # one multiply-add and seven adds a cell and sweep
    if kind in ("solve", "learned"):
        width = 4 if case.get("precision") == "mixed" else 8
        cycles = 5
        fmg = sum(_cycle_bytes(n[:top], width) for top in range(2, len(n) + 1))
        total = fmg + cycles * (_cycle_bytes(n, width) + 16 * leaves) + 16.0 * cells
        w = dict(bytes=total, flops=flops * total / (127.0 * cells))
        if kind == "learned":
            w = dict(bytes=w["bytes"] + 80.0 * leaves, flops=w["flops"] + 2 * 15552.0 * leaves)
        return w
    if kind == "time_step":
        return dict(bytes=2 * _cycle_bytes(n, 8) + cells * 8.0 * (1 + 3 + 27 * 64 / 512), flops=2 * flops)
    if kind == "regrid":
        return dict(bytes=cells * 8.0 * 5, flops=10.0 * cells)
    return dict(bytes=4 * _cycle_bytes(n, 8) + 2 * 8.0 * (cells * (2 + 27 * 64 / 512) + leaves * (4 + 27 * 64 / 512 + 1 + 3)),
                flops=4 * flops + 2 * 200.0 * leaves)


# --------------------------------------------------------------------- exact

def _bf(v):
    """Rounded to BF16 (a gradient passes through unchanged), as the network is defined."""
    return v + (v.detach().to(torch.float32).to(torch.bfloat16).to(v.dtype) - v.detach())


def _conv(a, w, same):
    """3^3 convolution of a [n][z][y][x][in] with w [out][in][27] in a's type."""
    if same:
        a = torch.nn.functional.pad(a, (0, 0, 1, 1, 1, 1, 1, 1))
    out = 0.0
    for t in range(27):
        out = out + a[:, t // 9:t // 9 + 8, t // 3 % 3:t // 3 % 3 + 8, t % 3:t % 3 + 8] @ w[:, :, t].t()
    return out


def _network(p, x):
    w1, b1 = _bf(p[:432]).view(16, 1, 27), p[432:448]
    w2, b2 = _bf(p[448:7360]).view(16, 16, 27), p[7360:7376]
    w3, b3 = _bf(p[7376:7808]).view(1, 16, 27), p[7808]
    a1 = _bf(torch.relu(_conv(_bf(x).unsqueeze(-1), w1, False) + b1))
    a2 = _bf(torch.relu(_conv(a1, w2, True) + b2))
    return (_conv(a2, w3, True) + b3).squeeze(-1)


def _uniform_solution(t, rhs, top):
    """The discrete solution on a uniform grid by diagonalisation of the 7-point
    operator (Dirichlet ghosts 2 g - phi), and its means on the coarser levels."""
    m = 8 << (top - 1)
    level, ijk = t.index(M.MG_IDX_LEVEL).reshape(-1), t.index(M.MG_IDX_IJK).reshape(-1, 3)
    b = np.empty((m, m, m))
    for q in np.nonzero(level == top)[0]:
        i, j, k = 8 * ijk[q]
        b[k:k + 8, j:j + 8, i:i + 8] = rhs[q]
    h2 = 1.0 / m ** 2
    b[-1] -= 2.0 * UNIT["bc_val"][5] / h2
    lap = -2.0 * np.eye(m) + np.eye(m, k=1) + np.eye(m, k=-1)
    lap[0, 0] = lap[-1, -1] = -3.0
    lam, v = np.linalg.eigh(lap)
    f = np.einsum("kjx,xi->kji", np.einsum("kyi,yj->kji", np.einsum("zji,zk->kji", b, v, optimize=True), v, optimize=True),
                  v, optimize=True)
    f *= h2 / (lam[:, None, None] + lam[None, :, None] + lam[None, None, :])
    f = np.einsum("kjx,ix->kji", np.einsum("kyi,jy->kji", np.einsum("zji,kz->kji", f, v, optimize=True), v, optimize=True),
                  v, optimize=True)
    out = np.empty((len(level), 8, 8, 8))
    for lev in range(top, 0, -1):
        for q in np.nonzero(level == lev)[0]:
            i, j, k = 8 * ijk[q]
            out[q] = f[k:k + 8, j:j + 8, i:i + 8]
        if lev > 1:
            f = f.reshape(len(f) // 2, 2, len(f) // 2, 2, len(f) // 2, 2).mean(axis=(1, 3, 5))
    return out


def exact(case, seed):
    """64-bit values where a plain form exists: the solve on a uniform grid and
    the network (with its defined BF16 rounding points).  On refined meshes the
    composite operator has no solution cheaper than a multigrid of its own."""
    if case["kind"] == "solve" and case["shape"] == "uniform":
        t = make_tree(case, UNIT)
        return dict(phi=_uniform_solution(t, rhs_of(case, t, seed).cpu().numpy(), case["top"]), cycles=None)
    if case["kind"] not in ("nn_forward", "nn_train"):
        return None
    s = prepare(case, seed)
    p = torch.from_numpy(params_of(seed)).to(DEV).double()
    if s.kind == "nn_forward":
        return torch.cat([_network(p, q.double()) for q in s.x.split(256)])
    p.requires_grad_(True)
    n, loss = len(s.idx), 0.0
    for part in s.idx.long().split(128):
        e = ((_network(p, s.x[part].double()) - s.target[part].double()) ** 2).sum() / (512.0 * n)
        e.backward()
        loss += float(e.detach())
    grad = p.grad
    m, v = 0.1 * grad, 0.001 * grad ** 2
    new = p.detach() - 1e-3 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
    return dict(loss=np.float64(loss), grad=grad, params=new)
