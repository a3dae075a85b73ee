"""The kernels that sort the atoms, at the sizes where another one or another way through it takes over:
vector types up to 2048, 4096 and 8192 atoms (two, four and eight per thread of one workgroup), index types up to
4096 atoms, past 32 examples or in few channels of some grids (one workgroup) and beyond (shares of the types, listed in LDS up to 12288
atoms), bins of thousands of atoms, planes of many bins.  Records have one order: every run gives the same bits."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import GRAD_RTOL, dev, grid_tol, mg  # noqa: E402,F401


def _inputs(B, N, T, D, spread, skew, seed):
    rng = np.random.default_rng(seed)
    dim = (D - 1) * 0.75
    coords = rng.uniform(-dim / 2 - spread, dim / 2 + spread, (B, N, 3)).astype(np.float32)
    types = rng.integers(0, T, (B, N)).astype(np.int32)
    types[rng.random((B, N)) < skew] = 0            # most atoms of one type
    radii = rng.uniform(0.6, 1.5, T).astype(np.float32)
    natoms = np.maximum(N - np.arange(B, dtype=np.int32) * (N // 3), 1)
    pose = dict(natoms=natoms, quats=rng.standard_normal((B, 4)).astype(np.float32))
    return rng, dim, coords, types, radii, pose, {k: dev(v) for k, v in pose.items()}


@pytest.mark.parametrize("B,N,T,D,spread,skew", [
    (2, 4097, 3, 16, 2.0, 0.0), (1, 8192, 5, 16, 20.0, 0.0), (33, 4097, 2, 8, 3.0, 0.0), (28, 4200, 28, 6, 3.0, 0.0), (60, 8300, 7, 6, 3.0, 0.3),
    (1, 12288, 1, 16, 6.0, 0.0), (1, 12289, 1, 16, 6.0, 0.0), (1, 14000, 9, 12, 8.0, 0.95), (2, 9000, 4, 70, 1.0, 0.5),
    (9, 8300, 2, 6, 3.0, 1.0),      # nine examples of two shares, one of them without atoms
    # few channels: one workgroup for grids of up to 14 A, and up to 60 atoms to a plane where all find room; else shares
    (2, 4097, 5, 18, 4.0, 0.0), (2, 4097, 5, 19, 4.0, 0.0), (1, 8192, 1, 18, 9.0, 0.0), (1, 8192, 1, 19, 9.0, 0.0),
    (1, 4200, 3, 70, 1.0, 0.9), (1, 4201, 3, 70, 1.0, 0.9), (1, 4200, 4, 70, 1.0, 0.9),
])
def test_index_types(mg, B, N, T, D, spread, skew):
    rng, dim, coords, types, radii, pose, dpose = _inputs(B, N, T, D, spread, skew, N + D)
    co, ty, ra = dev(coords), dev(types), dev(radii)
    gm = mg.GridMaker(0.75, dim, radius_type_indexed=True)
    ws = gm.mg_prepare(co, ty, ra, T, **dpose)
    outs = [gm.mg_forward_index(co, ty, ra, T, **dpose).cpu().numpy() for _ in range(2)]
    outs.append(gm.mg_forward_index_prepared(B, N, T, ws).cpu().numpy())
    ref = oracle.forward_index(coords, types, radii, T, 0.75, dim, **pose)
    assert np.abs(outs[0] - ref).max() <= grid_tol(ref)
    for o in outs[1:]:
        assert np.array_equal(outs[0].view(np.uint32), o.view(np.uint32))
    G = rng.standard_normal(ref.shape).astype(np.float32)
    want = oracle.backward_index(coords, types, radii, T, 0.75, dim, G, **pose)
    got = gm.mg_backward_index(co, ty, ra, T, dev(G), **dpose).cpu().numpy()
    assert np.abs(got - want).max() <= GRAD_RTOL * np.abs(want).max()


@pytest.mark.parametrize("N,T,D,spread,skew", [
    (4097, 5, 19, 4.0, 0.0), (8192, 1, 19, 9.0, 0.0), (8192, 28, 13, 1.0, 0.9), (4201, 3, 70, 1.0, 0.9), (6001, 2, 33, 6.0, 0.5),
])
@pytest.mark.parametrize("by_type", [True, False])
def test_shares_and_one_workgroup_give_the_same_bits(mg, N, T, D, spread, skew, by_type):
    """An example alone is sorted by shares, among 32 others by one workgroup."""
    rng, dim, coords, types, radii, pose, _ = _inputs(1, N, T, D, spread, skew, N + T)
    types[0, ::700] = -1
    if not by_type:
        radii = rng.uniform(0.6, 1.5, (1, N)).astype(np.float32)
    G = rng.standard_normal((1, T, D, D, D)).astype(np.float32)
    many = lambda v: dev(np.repeat(v, 33, axis=0))          # noqa: E731
    got = []
    for of, B in ((dev, 1), (many, 33)):
        gm = mg.GridMaker(0.75, dim, radius_type_indexed=by_type)
        co, ty, ra = of(coords), of(types), dev(radii) if by_type else of(radii)
        ws = gm.mg_prepare(co, ty, ra, T, natoms=of(np.array([N - 5], np.int32)), quats=of(pose["quats"]))
        grid = gm.mg_forward_index_prepared(B, N, T, ws)
        grad = torch.full((B, N, 3), float("nan"), device="cuda")
        gm.mg_backward_index_prepared(B, N, T, of(G), ws, grad_coords=grad)
        got.append((grid, grad))
    for one, all_of in zip(*got):
        one = one.contiguous().view(torch.int32)
        all_of = all_of.contiguous().view(torch.int32)
        assert not torch.isnan(one.view(torch.float32)).any()
        for b in (0, 15, 32):
            assert torch.equal(one[0], all_of[b])


@pytest.mark.parametrize("main", [0, 4, 8])         # (64 examples: shares of three types each)
def test_index_shares_longer_than_the_list(mg, main):
    """More than 12288 atoms of one type beside two others in a share, with smaller and larger types in other shares."""
    B, N, T, D = 64, 14000, 9, 8
    rng, dim, coords, types, radii, pose, dpose = _inputs(B, N, T, D, 3.0, 0.0, main)
    types[rng.random((B, N)) < 0.96] = main
    types[:, ::1000] = -1 + (T + 1) * (np.arange(0, N, 1000) // 1000 % 2)       # no type's
    co, ty, ra = dev(coords), dev(types), dev(radii)
    gm = mg.GridMaker(0.75, dim, radius_type_indexed=True)
    ref = oracle.forward_index(coords, types, radii, T, 0.75, dim, **pose)
    outs = [gm.mg_forward_index(co, ty, ra, T, **dpose).cpu().numpy() for _ in range(2)]
    assert np.abs(outs[0] - ref).max() <= grid_tol(ref)
    assert np.array_equal(outs[0].view(np.uint32), outs[1].view(np.uint32))
    G = rng.standard_normal(ref.shape).astype(np.float32)
    want = oracle.backward_index(coords, types, radii, T, 0.75, dim, G, **pose)
    ws = gm.mg_prepare(co, ty, ra, T, **dpose)
    got = torch.full((B, N, 3), float("nan"), device="cuda")
    gm.mg_backward_index_prepared(B, N, T, dev(G), ws, grad_coords=got)
    assert np.abs(got.cpu().numpy() - want).max() <= GRAD_RTOL * np.abs(want).max()


@pytest.mark.parametrize("B,N,T,D,spread,crowd", [
    (1, 1, 2, 9, 0.0, 0), (2, 63, 3, 9, 1.0, 0), (3, 2048, 5, 14, 2.0, 0), (2, 2049, 4, 14, 2.0, 0), (1, 4097, 3, 13, 4.0, 3000),
    (1, 8192, 70, 8, 6.0, 0), (1, 8193, 2, 13, 10.0, 0), (1, 20011, 3, 12, 2.0, 9000), (1, 500, 2, 130, 0.5, 0),
])
def test_vector_types(mg, B, N, T, D, spread, crowd):
    rng, dim, coords, _, radii, pose, dpose = _inputs(B, N, T, D, spread, 0.0, N + D)
    if crowd:                       # one plane's bin holds thousands of atoms
        pose["quats"] = dpose["quats"] = None
        coords[:, rng.permutation(N)[:crowd], 0] = 0.4
    # sums of thousands of weights stay within what fixed point holds
    w = (rng.random((B, N, T)) * min(1.0, 60.0 / (N * 0.2))).astype(np.float32)
    co, ra = dev(coords), dev(radii)
    gm = mg.GridMaker(0.75, dim, radius_type_indexed=True)
    ws = gm.mg_prepare(co, None, ra, T, **dpose)
    outs = [gm.mg_forward_vector(co, dev(w), ra, **dpose).cpu().numpy() for _ in range(2)]
    outs.append(gm.mg_forward_vector_prepared(dev(w), ra, ws).cpu().numpy())
    ref = oracle.forward_vector(coords, w, radii, 0.75, dim, **pose)
    assert np.abs(outs[0] - ref).max() <= grid_tol(ref)
    for o in outs[1:]:
        assert np.array_equal(outs[0].view(np.uint32), o.view(np.uint32))
    G = rng.standard_normal(ref.shape).astype(np.float32)
    wc, ww = oracle.backward_vector(coords, w, radii, 0.75, dim, G, **pose)
    gc, gw = gm.mg_backward_vector_prepared(dev(w), ra, dev(G), ws)
    assert np.abs(gc.cpu().numpy() - wc).max() <= GRAD_RTOL * max(np.abs(wc).max(), 1e-30)
    assert np.abs(gw.cpu().numpy() - ww).max() <= GRAD_RTOL * max(np.abs(ww).max(), 1e-30)


@pytest.mark.parametrize("B,N,keep", [(1, 8200, 64), (2, 9001, 2), (1, 16500, 5)])
def test_vector_types_culled_among_live(mg, B, N, keep):
    """Culled atoms between live ones in every pattern of lanes (the first lane of a wavefront live, the rest
    culled, and the other way round): each is recorded once, and its gradients are zeros."""
    rng = np.random.default_rng(N)
    T, D, res = 3, 10, 0.75
    dim = (D - 1) * res
    coords = rng.uniform(-dim / 2, dim / 2, (B, N, 3)).astype(np.float32)
    a = np.arange(N)
    out = (a % keep != 0) ^ ((a // 1024) % 2 == 1)
    coords[:, out] += 40.0
    natoms = np.array([N, N - 77][:B], np.int32)
    w = (rng.random((B, N, T)) * 0.05).astype(np.float32)
    radii = rng.uniform(0.6, 1.5, T).astype(np.float32)
    G = rng.standard_normal((B, T, D, D, D)).astype(np.float32)
    gm = mg.GridMaker(res, dim, radius_type_indexed=True)
    co, ra, dn = dev(coords), dev(radii), dev(natoms)
    ref = oracle.forward_vector(coords, w, radii, res, dim, natoms=natoms)
    wc, ww = oracle.backward_vector(coords, w, radii, res, dim, G, natoms=natoms)
    for _ in range(2):
        ws = gm.mg_prepare(co, None, ra, T, natoms=dn)
        got = gm.mg_forward_vector_prepared(dev(w), ra, ws).cpu().numpy()
        assert np.abs(got - ref).max() <= grid_tol(ref)
        gc = torch.full((B, N, 3), float("nan"), device="cuda")
        gw = torch.full((B, N, T), float("nan"), device="cuda")
        gm.mg_backward_vector_prepared(dev(w), ra, dev(G), ws, grad_coords=gc, grad_weights=gw)
        gc, gw = gc.cpu().numpy(), gw.cpu().numpy()
        assert np.abs(gc - wc).max() <= GRAD_RTOL * np.abs(wc).max()
        assert np.abs(gw - ww).max() <= GRAD_RTOL * np.abs(ww).max()
        assert not gc[:, out].any() and not gw[:, out].any()


@pytest.mark.parametrize("B,N,D,planes,crowd", [
    (1, 20011, 12, (4, 5), 13000),      # one bin, put in order by one wavefront
    (64, 16000, 24, (6, 13), 13900),    # the seven bins of a share, put in order by counting
    (64, 16000, 24, (20, 24), 13900),   # the share that also records the culled atoms
])
def test_vector_shares_longer_than_the_list(mg, B, N, D, planes, crowd):
    """More than 12288 atoms in the planes of one workgroup, culled ones among them: counted and placed in passes
    over all atoms.  (64 examples make shares of seven bins; all but the first two are short.)"""
    rng = np.random.default_rng(crowd + D)
    T, res = 2, 0.75
    dim = (D - 1) * res
    coords = rng.uniform(-dim / 2, dim / 2, (B, N, 3)).astype(np.float32)
    coords[0, :, 0] = rng.uniform(-dim / 2 - 30.0, dim / 2 + 30.0, N)
    at = rng.permutation(N)[:crowd]
    lo, hi = planes
    coords[0, at, 0] = ((lo + np.arange(crowd) % (hi - lo)) + rng.uniform(0.1, 0.8, crowd)) * res - dim / 2
    if B > 1:
        coords[1] = coords[0, ::-1]
    natoms = np.full(B, 9, np.int32)
    natoms[:2] = N
    w = (rng.random((B, N, T)) * (60.0 / N)).astype(np.float32)
    radii = rng.uniform(0.6, 1.5, T).astype(np.float32)
    G = rng.standard_normal((B, T, D, D, D)).astype(np.float32)
    ref = oracle.forward_vector(coords, w, radii, res, dim, natoms=natoms)
    wc, ww = oracle.backward_vector(coords, w, radii, res, dim, G, natoms=natoms)
    co, ra, dn, dw = dev(coords), dev(radii), dev(natoms), dev(w)
    gm = mg.GridMaker(res, dim, radius_type_indexed=True)
    ws = gm.mg_prepare(co, None, ra, T, natoms=dn)
    outs = [gm.mg_forward_vector_prepared(dw, ra, ws).cpu().numpy(), gm.mg_forward_vector(co, dw, ra, natoms=dn).cpu().numpy()]
    assert np.abs(outs[0] - ref).max() <= grid_tol(ref)
    assert np.array_equal(outs[0].view(np.uint32), outs[1].view(np.uint32))
    gc = torch.full((B, N, 3), float("nan"), device="cuda")
    gw = torch.full((B, N, T), float("nan"), device="cuda")
    gm.mg_backward_vector_prepared(dw, ra, dev(G), ws, grad_coords=gc, grad_weights=gw)
    assert np.abs(gc.cpu().numpy() - wc).max() <= GRAD_RTOL * np.abs(wc).max()
    assert np.abs(gw.cpu().numpy() - ww).max() <= GRAD_RTOL * np.abs(ww).max()


@pytest.mark.parametrize("N", [2, 5000, 9000])      # one workgroup's kernels; shares
@pytest.mark.parametrize("radius", [3e9, 1e15])
def test_radii_of_more_steps_than_an_integer_holds(mg, N, radius):
    """Every voxel is inside every atom: occupancy is 1, densities are sums of weights."""
    rng = np.random.default_rng(N)
    T, D, res = 2, 6, 0.5
    coords = rng.uniform(-3, 3, (1, N, 3)).astype(np.float32)
    types = np.ones((1, N), np.int32)
    w = (rng.random((1, N, T)) * (20.0 / N)).astype(np.float32)
    ra = torch.full((T,), radius, device="cuda")
    gmb = mg.GridMaker(res, (D - 1) * res, radius_type_indexed=True, binary=True)
    ws = gmb.mg_prepare(dev(coords), dev(types), ra, T)
    occ = gmb.mg_forward_index_prepared(1, N, T, ws)
    assert float(occ[:, 0].abs().max()) == 0.0 and float(occ[:, 1].min()) == 1.0
    gm = mg.GridMaker(res, (D - 1) * res, radius_type_indexed=True)
    ws = gm.mg_prepare(dev(coords), None, ra, T)
    out = gm.mg_forward_vector_prepared(dev(w), ra, ws).cpu().numpy()
    want = w.astype(np.float64).sum(axis=1)[:, :, None, None, None]
    assert np.abs(out - want).max() <= grid_tol(want)
