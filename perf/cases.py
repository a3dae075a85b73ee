"""The work this library is timed on: atoms to grids, and gradients on grids back to atoms.

``listed()`` names what its users run, from one small molecule to a chunk of high-resolution
grids; ``draw(rng)`` gives further cases of the same ranges.  ``prepare`` makes what a program
holds before the call (device arrays and the GridMaker), ``run`` is one pass through the public
entry points, ``work`` the bytes and operations a pass cannot do without, ``tolerance`` how far
another correct implementation in the same precision may lie from this one.

A case:
  op       "forward" (atoms -> grid), "backward" (gradient on the grid -> atoms) or "step" (both,
           through torch.autograd, as a training step does)
  types    "index" (one channel per atom) or "vector" (a weight per atom and channel)
  B N T    examples, atoms per example (the longest), channels
  D res    points per side of a (sub)grid, spacing in Angstrom
  S        subgrids per side (1: a plain grid)
  binary   0/1 occupancy instead of densities
  double   grid (or gradient) of doubles
  radii    "type" (a table by channel) or "atom" (one per atom; index types)
  ragged   examples of different length (natoms), the rest is padding of type -1
  pose     "none", "given" (a rotation and a translation per example) or, for steps, "random"
           (drawn on the device anew for every pass, the usual augmentation)
  out      "new" (the call allocates the grid) or "kept" (into a tensor the program keeps)
"""
from __future__ import annotations

import math

import torch

from paper_1912_04822_amd import molgrid
from paper_1912_04822_amd.autograd import GridLayer

RMIN, RMAX = 1.2, 2.0           # atomic radii, uniform (Angstrom)
CUTOFF = 1.5                    # the density reaches 1.5 radii
DENSITY = 0.076                 # atoms per cubic Angstrom (2000 in a cube of 30)


def _case(name=None, **kw):
    c = dict(op="forward", types="index", B=1, N=2040, T=28, D=48, res=0.5, S=1, binary=False,
             double=False, radii="type", ragged=False, pose="given", out="new")
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # one small molecule on a small grid, called again and again: latency
        _case("small_molecule", N=100, T=4, D=24, pose="none"),
        # scoring a single pose of a complex at the default grid (48 points, 23.5 A): latency
        _case("one_complex"),
        # the training-size batch of complexes, grid kept and refilled (the benchmark's workload)
        _case("batch", B=50, out="kept"),
        # 24 A at 0.5 A is 49 points a side: odd rows; complexes of different length, radii per atom
        _case("odd_ragged_batch", B=20, N=3000, D=49, ragged=True, radii="atom"),
        # occupancy grids of the same batch
        _case("binary_batch", B=50, binary=True, out="kept"),
        # a chunk of high-resolution grids (0.25 A), the largest output: 1.6 GB
        _case("high_resolution", B=16, N=8000, D=96, res=0.25, out="kept"),
        # gradients on the grids of a batch to the atoms (optimising poses through a fixed network)
        _case("batch_gradient", op="backward", B=50),
        # a training step with gradients to the atoms, poses drawn at random
        _case("training_step", op="step", B=32, pose="random"),
        # every atom with a weight per channel (learned or ambiguous types): grids
        _case("vector_batch", types="vector", B=50, out="kept"),
        # a training step that also learns the type weights, odd number of channels
        _case("vector_training_step", op="step", types="vector", B=16, T=21, pose="random"),
        # one large assembly, past what one workgroup can sort, as eight subgrids of doubles
        _case("large_assembly_double", B=2, N=20000, T=18, D=40, S=2, double=True),
        # minimising a single pose against a fixed network: one gradient at a time, latency
        _case("pose_gradient", op="backward"),
    ]


def draw(rng):
    """One more case: sizes spread over the logarithm of their ranges, every option in turn."""
    def span(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        types = rng.choice(["index", "index", "vector"])
        op = rng.choice(["forward", "forward", "backward", "step"])
        c = _case(op=op, types=types, B=span(1, 64), N=span(40, 20000), T=span(2, 40), D=span(12, 96),
                  res=rng.choice([0.25, 0.375, 0.5, 0.5, 0.75, 1.0]))
        c["binary"] = op == "forward" and rng.random() < 0.2
        c["double"] = op != "step" and not c["binary"] and rng.random() < 0.15
        c["S"] = 2 if rng.random() < 0.12 else 1
        c["radii"] = "atom" if types == "index" and rng.random() < 0.3 else "type"
        c["ragged"] = rng.random() < 0.4
        c["pose"] = rng.choice(["none", "given", "given"]) if op != "step" else rng.choice(["given", "random"])
        c["out"] = rng.choice(["new", "kept"]) if op == "forward" else "new"
        w = work(c)
        if w["bytes"] <= 6.0e8 and w["flops"] <= 3.0e9 and c["B"] * c["N"] <= 130000:
            return c


# ---- inputs ----

def _cube(N):
    return (N / DENSITY) ** (1.0 / 3.0)


def _maker(c):
    kw = dict(binary=c["binary"], radius_type_indexed=c["radii"] == "type", subgrids_per_side=c["S"])
    dim = (c["D"] - 1) * c["res"]
    return GridLayer(c["res"], dim, **kw) if c["op"] == "step" else molgrid.GridMaker(c["res"], dim, **kw)


def prepare(case, seed):
    """98 % receptor atoms filling a cube (types of the first half of the channels), the rest a
    ligand about the centre (second half); Dirichlet-like weights; N(0,1) upstream gradients."""
    c = dict(case)
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(int(seed) * 7919 + 12345)
    B, N, T = c["B"], c["N"], c["T"]

    def uni(shape, lo, hi):
        return torch.rand(shape, generator=g, device=dev) * (hi - lo) + lo

    def ints(lo, hi, shape):
        return torch.randint(lo, hi, shape, generator=g, device=dev, dtype=torch.int32)

    nlig = max(1, N // 50)
    half = max(1, T // 2)
    coords = uni((B, N, 3), -_cube(N) / 2, _cube(N) / 2)
    coords[:, N - nlig:] = torch.randn((B, nlig, 3), generator=g, device=dev) * 3.0
    types = ints(0, half, (B, N))
    types[:, N - nlig:] = ints(half if T > 1 else 0, T, (B, nlig))
    radii = uni((T,), RMIN, RMAX) if c["radii"] == "type" else uni((B, N), RMIN, RMAX)
    s = {"case": c, "maker": _maker(c), "coords": coords, "radii": radii, "centers": None,
         "quats": None, "translations": None, "natoms": None, "types": None, "weights": None,
         "grad": None, "out": None}
    if c["ragged"]:
        s["natoms"] = ints(max(1, N // 2), N + 1, (B,))
        types[torch.arange(N, device=dev)[None, :] >= s["natoms"][:, None]] = -1
    if c["pose"] != "none":
        s["centers"] = uni((B, 3), -0.5, 0.5)
    if c["pose"] == "given":
        q = torch.randn((B, 4), generator=g, device=dev)
        s["quats"] = q / q.norm(dim=1, keepdim=True)
        s["translations"] = uni((B, 3), -2.0, 2.0)
    if c["types"] == "index":
        s["types"] = types.contiguous()
    else:
        w = torch.rand((B, N, T), generator=g, device=dev) ** (1.0 / 0.3)
        s["weights"] = w / w.sum(dim=2, keepdim=True)
    dtype = torch.float64 if c["double"] else torch.float32
    gm = s["maker"].gm if c["op"] == "step" else s["maker"]
    if c["op"] != "forward":
        s["grad"] = torch.randn(gm.grid_shape(B, T), generator=g, device=dev, dtype=dtype)
    elif c["out"] == "kept":
        s["out"] = torch.empty(gm.grid_shape(B, T), dtype=dtype, device=dev)
    if c["op"] == "step":
        s["coords"].requires_grad_()
        if s["weights"] is not None:
            s["weights"].requires_grad_()
    return s


# ---- one pass ----

def run(s):
    c, m = s["case"], s["maker"]
    pose = dict(natoms=s["natoms"], centers=s["centers"], quats=s["quats"], translations=s["translations"])
    if c["op"] == "step":
        if c["pose"] == "random":
            pose.update(random_rotation=True, random_translation=2.0)
        grid = m(s["coords"], s["radii"], types=s["types"], weights=s["weights"], T=c["T"], **pose)
        leaves = [s["coords"]] + ([s["weights"]] if s["weights"] is not None else [])
        return [grid.detach()] + list(torch.autograd.grad(grid, leaves, s["grad"]))
    if c["op"] == "backward":
        if c["types"] == "index":
            return m.mg_backward_index(s["coords"], s["types"], s["radii"], c["T"], s["grad"], **pose)
        return m.mg_backward_vector(s["coords"], s["weights"], s["radii"], s["grad"], **pose)
    dtype = torch.float64 if c["double"] else torch.float32
    if c["types"] == "index":
        return m.mg_forward_index(s["coords"], s["types"], s["radii"], c["T"], out=s["out"], dtype=dtype, **pose)
    return m.mg_forward_vector(s["coords"], s["weights"], s["radii"], out=s["out"], dtype=dtype, **pose)


# ---- what a pass cannot do without ----

def work(case):
    c = case
    B, N, T = c["B"], c["N"], c["T"]
    elem = 8 if c["double"] else 4
    side = c["D"] * c["S"]
    voxels = float(T) * side ** 3
    n = N * (0.75 if c["ragged"] else 1.0)
    reach = (1.0 if c["binary"] else CUTOFF) ** 3
    sphere = 4.0 / 3.0 * math.pi * reach * (RMAX ** 4 - RMIN ** 4) / (4.0 * (RMAX - RMIN))   # mean, A^3
    inside = min(1.0, side * c["res"] / _cube(N)) ** 3      # share of the atoms the grid holds
    pairs = n * inside * sphere / c["res"] ** 3             # (atom, voxel) pairs of one channel set
    feeds = T if c["types"] == "vector" else 1              # channels an atom feeds
    # voxels within some atom's cutoff in their channel (atoms spread evenly over the grid's share)
    per_channel = n if c["types"] == "vector" else n / T
    box = min(side * c["res"], _cube(N)) ** 3
    covered = voxels * min(1.0, _cube(N) / (side * c["res"])) ** 3 * (
        1.0 - math.exp(-per_channel * inside * sphere / box))
    inputs = B * n * (12 + (4 * T if c["types"] == "vector" else 4) + (4 if c["radii"] == "atom" else 0))
    bytes_, flops = inputs, 0.0
    if c["op"] != "backward":           # every element of the grid is written
        bytes_ += B * voxels * elem
        flops += B * pairs * feeds * (3.0 if c["binary"] else 8.0)
    if c["op"] != "forward":            # the gradient is needed where some atom reaches
        bytes_ += B * covered * elem + B * n * (12 + (4 * T if c["types"] == "vector" else 0))
        flops += B * pairs * feeds * (16.0 if c["types"] == "vector" else 12.0)
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """Occupancy is decided in a fixed order of float operations: exact.  Densities and gradients
    are sums of float terms: four times the largest errors seen against the same sums in double
    (densities 3.3e-7 and 3.8e-6, weighted ones 1.1e-6 and 8.8e-6, gradients 1.0e-6 and 1.3e-5)."""
    if case["binary"]:
        return "exact"
    if case["op"] != "forward":
        return {"rel": 4e-6, "max": 5e-5}
    return {"rel": 4.4e-6, "max": 3.5e-5} if case["types"] == "vector" else {"rel": 1.3e-6, "max": 1.5e-5}


# ---- the same outputs in 64 bits, in plain torch ----

def _philox(b, draw, block):
    """Philox4x32-10 with key 0: four uniforms of example b (the documented augmentation stream)."""
    c, k = [b, draw & 0xFFFFFFFF, draw >> 32, block], [0, 0]
    for _ in range(10):
        p0, p1 = 0xD2511F53 * c[0], 0xCD9E8D57 * c[2]
        c = [(p1 >> 32) ^ c[1] ^ k[0], p1 & 0xFFFFFFFF, (p0 >> 32) ^ c[3] ^ k[1], p0 & 0xFFFFFFFF]
        k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
    return [(w + 0.5) / 2.0 ** 32 for w in c]


def _first_poses(B, dev):
    """The poses a new GridLayer draws for its first pass: uniform rotations, +-2 A."""
    q, t = [], []
    for b in range(B):
        u, v = _philox(b, 0, 0), _philox(b, 0, 1)
        s1, s2, a1, a2 = math.sqrt(1 - u[0]), math.sqrt(u[0]), 2 * math.pi * u[1], 2 * math.pi * u[2]
        q.append([s2 * math.cos(a2), s1 * math.sin(a1), s1 * math.cos(a1), s2 * math.sin(a2)])
        t.append([2.0 * (2.0 * x - 1.0) for x in v[:3]])
    return torch.tensor(q, device=dev), torch.tensor(t, device=dev)     # float32, as they are applied


def _rotations(q):
    q = q.double()
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).view(-1, 3, 3)


def _density(x):
    """rho(x) and rho'(x), x = d/r: a Gaussian up to 1, a quadratic from there to 3/2."""
    e, A = torch.exp(-2 * x * x), 4 * math.exp(-2.0)
    u = (1.5 - x).clamp(min=0.0)
    return torch.where(x <= 1, e, A * u * u), torch.where(x <= 1, -4 * x * e, -2 * A * u)


def exact(case, seed):
    """Atoms placed in 64 bits and rounded to float (positions are float by definition), every
    voxel in an atom's cutoff box summed in 64 bits.  None for occupancy, which is decided bit
    for bit by a fixed sequence of float operations and compared exactly."""
    c = case
    if c["binary"]:
        return None
    s = prepare(case, seed)
    dev, B, N, T, D, S = s["coords"].device, c["B"], c["N"], c["T"], c["D"], c["S"]
    side, f64 = D * S, torch.float64
    quats, trans = _first_poses(B, dev) if c["pose"] == "random" else (s["quats"], s["translations"])
    cen = s["centers"].double() if s["centers"] is not None else torch.zeros((B, 3), dtype=f64, device=dev)
    R = _rotations(quats) if quats is not None else torch.eye(3, dtype=f64, device=dev).repeat(B, 1, 1)
    pos = torch.einsum("bmk,bnk->bnm", R, s["coords"].detach().double() - cen[:, None]) + cen[:, None]
    if trans is not None:
        pos = pos + trans.double()[:, None]
    pos = pos.float().double() - cen[:, None] + 0.5 * (side - 1) * c["res"]      # from the first lattice point
    alive = torch.ones((B, N), dtype=torch.bool, device=dev)
    if s["natoms"] is not None:
        alive &= torch.arange(N, device=dev)[None, :] < s["natoms"][:, None]
    vector = c["types"] == "vector"
    w = s["weights"].detach().double() if vector else None
    grid = torch.zeros(B * T * side ** 3 if c["op"] != "backward" else 0, dtype=f64, device=dev)
    G = None
    if c["op"] != "forward":
        G = s["grad"].double()
        if S > 1:       # subgrids -> one cube
            G = G.permute(0, 4, 1, 5, 2, 6, 3, 7).reshape(B, T, side, side, side)
        G = G.reshape(-1)
    gpos = torch.zeros((B, N, 3), dtype=f64, device=dev)
    gw = torch.zeros((B, N, T), dtype=f64, device=dev) if vector else None
    K = int(2 * CUTOFF * RMAX / c["res"]) + 3
    o = torch.arange(K, device=dev)
    box = torch.stack(torch.meshgrid(o, o, o, indexing="ij"), -1).view(1, -1, 3)
    bi, ni = torch.nonzero(alive, as_tuple=True)
    step = max(1, 12_000_000 // K ** 3)
    for a0 in range(0, len(bi), step):
        b, n = bi[a0:a0 + step], ni[a0:a0 + step]
        x = pos[b, n]
        lo = torch.floor((x - CUTOFF * RMAX) / c["res"]).long()
        p = lo[:, None] + box
        u = x[:, None] - p * c["res"]                           # atom minus voxel
        d = u.norm(dim=2)
        ok = ((p >= 0) & (p < side)).all(2)
        v = torch.where(ok, (p[..., 0] * side + p[..., 1]) * side + p[..., 2], 0)
        if vector:
            chans = [(torch.full_like(n, t), s["radii"][t].double().expand(len(n))) for t in range(T)]
        else:
            t = s["types"][b, n].long()
            chans = [(t, (s["radii"][t] if c["radii"] == "type" else s["radii"][b, n]).double())]
        for t, r in chans:
            rho, slope = _density(d / r[:, None])
            at = ((b * T + t) * side ** 3)[:, None] + v
            rho = torch.where(ok, rho, 0.0)
            wt = w[b, n, t] if vector else torch.ones_like(r)
            if c["op"] != "backward":
                grid.index_add_(0, at.view(-1), (wt[:, None] * rho).view(-1))
            if c["op"] != "forward":
                g = torch.where(ok, G[at], 0.0)
                f = g * slope / (r[:, None] * d.clamp(min=1e-30))
                gpos[b, n] += wt[:, None] * (f[..., None] * u).sum(1)
                if vector:
                    gw[b, n, t] = (g * rho).sum(1)
    out = []
    if c["op"] != "backward":
        grid = grid.view(B, T, side, side, side)
        if S > 1:
            grid = grid.view(B, T, S, D, S, D, S, D).permute(0, 2, 4, 6, 1, 3, 5, 7).contiguous()
        out.append(grid)
    if c["op"] != "forward":
        out.append(torch.einsum("bmk,bnm->bnk", R, gpos))
        if vector:
            out.append(gw)
    return out if c["op"] == "step" else (tuple(out) if len(out) > 1 else out[0])
