"""Grids of index types are exact sums of rounded densities: the same bits in every run, however the
work is split.  Channels with so many atoms that a voxel's sum may pass 32 bits take a second pass;
they are looked at over both kinds of tiles (one, two and four wavefronts), whole and odd channels, and
a channel of more than a million atoms in reach of one tile."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import dev, grid_tol, mg  # noqa: E402,F401


def bits(t):
    return t.cpu().numpy().view(np.uint32)


def problem(B, N, T, D, crowd=0.0):
    rng = np.random.default_rng(N + D)
    half = (D - 1) * 0.25 + 1.0
    coords = rng.uniform(-half, half, (B, N, 3)).astype(np.float32)
    coords[:, : int(crowd * N)] *= 0.02         # on top of each other: sums of hundreds
    types = rng.integers(0, T, (B, N)).astype(np.int32)
    radii = rng.uniform(1.2, 2.0, T).astype(np.float32)
    return coords, types, radii


@pytest.mark.parametrize("B,N,T,D,crowd", [
    (1, 2040, 2, 48, 0.0), (1, 1000, 4, 24, 0.0), (5, 2048, 1, 7, 0.0), (1, 2048, 1, 64, 0.0),
    (1, 64, 1, 16, 1.0), (1, 63, 1, 16, 1.0), (1, 300, 2, 48, 1.0), (1, 2048, 1, 48, 1.0), (2, 2000, 1, 49, 0.9), (1, 2048, 2, 13, 0.5)])
def test_the_same_bits_however_the_work_is_split(mg, B, N, T, D, crowd):
    coords, types, radii = problem(B, N, T, D, crowd)
    args = (dev(coords), dev(types), dev(radii), T)
    gm = mg.GridMaker(0.5, (D - 1) * 0.5, radius_type_indexed=True)
    first = gm.mg_forward_index(*args)
    ref = oracle.forward_index(coords, types, radii, T, 0.5, (D - 1) * 0.5)
    assert np.abs(first.cpu().numpy() - ref).max() <= grid_tol(ref)
    for _ in range(4):
        assert np.array_equal(bits(gm.mg_forward_index(*args)), bits(first))
    # the order of the atoms does not matter
    perm = np.random.default_rng(1).permutation(N)
    again = gm.mg_forward_index(dev(coords[:, perm]), dev(types[:, perm]), dev(radii), T)
    assert np.array_equal(bits(again), bits(first))
    # several wavefronts on tiles from the tables (four of them are two sets where planes allow)
    tables = []
    try:
        for tile, waves in ((1024, 1), (1024, 2), (2048, 4), (4096, 2), (4096, 4)):
            mg.set_option("tile_floats", tile)
            mg.set_option("waves_per_tile", waves)
            runs = [gm.mg_forward_index(*args) for _ in range(3)]
            assert all(np.array_equal(bits(r), bits(runs[0])) for r in runs)
            tables.append(runs[0])
    finally:
        mg.set_option("tile_floats", 0)
        mg.set_option("waves_per_tile", 0)
    assert np.array_equal(bits(tables[0]), bits(tables[1]))            # same tiles, other wavefronts
    assert np.array_equal(bits(tables[3]), bits(tables[4]))
    out64 = gm.mg_forward_index(*args, dtype=torch.float64).cpu().numpy()
    assert np.abs(out64 - ref).max() <= grid_tol(ref)
    # other tiles cut the rows elsewhere: the densities are the same all the same
    assert all(np.array_equal(bits(t), bits(first)) for t in tables)
    assert np.array_equal(out64, first.double().cpu().numpy())


@pytest.mark.parametrize("B,N,T,D", [
    (1, 2040, 28, 48), (1, 2040, 4, 48), (2, 600, 9, 48), (1, 2047, 40, 49),
    (3, 700, 5, 21), (1, 256, 28, 96), (1, 100, 4, 24), (2, 60, 3, 17)])
def test_prepared_calls_give_the_bits_of_ordinary_ones(mg, B, N, T, D):
    """Inside the range of the one-launch route, which cuts other tiles than the tables' kernel and
    takes the atoms in another order; also through the layer, whose grid does not depend on whether a
    gradient will be asked for."""
    from paper_1912_04822_amd.autograd import GridLayer
    coords, types, radii = problem(B, N, T, D)
    rng = np.random.default_rng(7)
    pose = dict(centers=dev(rng.uniform(-1, 1, (B, 3)).astype(np.float32)),
                quats=dev(rng.standard_normal((B, 4)).astype(np.float32)),
                translations=dev(rng.uniform(-1, 1, (B, 3)).astype(np.float32)),
                natoms=dev(rng.integers(N // 2, N + 1, B).astype(np.int32)))
    args = (dev(coords), dev(types), dev(radii), T)
    for binary in (False, True):
        gm = mg.GridMaker(0.5, (D - 1) * 0.5, radius_type_indexed=True, binary=binary)
        out = gm.mg_forward_index(*args, **pose)
        ws = gm.mg_prepare(*args, **pose)
        prepared = gm.mg_forward_index_prepared(B, N, T, ws)
        assert np.array_equal(bits(out), bits(prepared))
    layer = GridLayer(0.5, (D - 1) * 0.5)
    plain = layer(args[0], args[2], types=args[1], T=T, **pose)
    asked = layer(args[0].clone().requires_grad_(), args[2], types=args[1], T=T, **pose)
    assert np.array_equal(bits(plain), bits(asked.detach()))


def test_a_million_atoms_in_reach_of_one_tile(mg):
    """Past 2^19 records the upper and lower bits of the densities are summed share by share."""
    N, D = (1 << 20) + 777, 6
    coords, types, radii = problem(1, N, 1, D)
    gm = mg.GridMaker(0.5, (D - 1) * 0.5, radius_type_indexed=True)
    args = (dev(coords), dev(types), dev(radii), 1)
    runs = [gm.mg_forward_index(*args) for _ in range(2)]
    assert np.array_equal(bits(runs[0]), bits(runs[1]))
    ref = oracle.forward_index(coords, types, radii, 1, 0.5, (D - 1) * 0.5)
    assert np.abs(runs[0].cpu().numpy() - ref).max() <= grid_tol(ref)
