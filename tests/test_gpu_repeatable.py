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
