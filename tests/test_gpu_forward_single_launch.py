"""Small problems in one launch: every tile's workgroup lists the atoms of its type and places them
itself.  The same grids as with the prep kernel's tables, to the bit, over the edges of
the rule (atoms, points per side, tiles) and the forms a call takes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import dev, mg  # noqa: E402,F401


@pytest.mark.parametrize("B,N,T,D,kind", [
    (1, 65, 3, 36, "type"), (3, 512, 2, 24, "atom"), (2, 513, 5, 13, "type"), (5, 2048, 1, 7, "type"),
    (1, 2048, 9, 37, "atom"), (1, 700, 3, 63, "type"), (2, 1000, 4, 64, "type"), (1, 300, 28, 48, "type"),
    (1, 2047, 40, 49, "type"), (4, 900, 11, 48, "type"), (1, 64, 2, 40, "type")])
def test_equals_the_tables(mg, B, N, T, D, kind):
    rng = np.random.default_rng(N + D)
    res = 0.5
    half = (D - 1) * 0.25 + 3.0
    coords = rng.uniform(-half, half, (B, N, 3)).astype(np.float32)
    coords[0, 1], coords[0, 2, 1], coords[0, 3] = np.nan, np.inf, 1e30
    types = rng.integers(-2, T + 2, (B, N)).astype(np.int32)
    radii = rng.uniform(0.5, 2.0, (B, N) if kind == "atom" else T).astype(np.float32)
    natoms = rng.integers(0, N + 1, B).astype(np.int32)
    natoms[0] = N
    pose = dict(natoms=dev(natoms), centers=dev(rng.uniform(-1, 1, (B, 3)).astype(np.float32)),
                quats=dev(rng.standard_normal((B, 4)).astype(np.float32)), translations=None)
    for binary in (False, True):
        gm = mg.GridMaker(res, (D - 1) * res, radius_type_indexed=kind != "atom", binary=binary)
        got = []
        try:
            for single in (1, 0):
                mg.set_option("single_launch", single)
                out = torch.full(gm.grid_shape(B, T), float("nan"), device="cuda")
                gm.mg_forward_index(dev(coords), dev(types), dev(radii), T, out=out, **pose)
                got.append(out.cpu().numpy())
        finally:
            mg.set_option("single_launch", 1)
        assert np.array_equal(got[0].view(np.uint32), got[1].view(np.uint32))
