"""Few atoms: the backward kernel alone places every atom itself.  Bit for bit what the prep kernel's
tables give, over the forms a call takes: padding, types out of range, dead radii, coordinates that
are not finite, odd grids, radii by type or by atom, gradients of doubles, both kinds of types."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import dev, mg  # noqa: E402,F401


@pytest.mark.parametrize("B,N,T,D", [(1, 1, 1, 1), (3, 5, 70, 12), (2, 130, 4, 13), (7, 1170, 3, 10),
                                     (24, 2048, 5, 8),      # the most atoms of index types ...
                                     (4, 2048, 5, 8)])      # ... and of vector types
@pytest.mark.parametrize("kind", ["type", "atom", "vector"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_equals_the_tables_bit_for_bit(mg, B, N, T, D, kind, dtype):
    rng = np.random.default_rng(B * N + T)
    res, half = 0.5, (D - 1) * 0.25 + 3.0
    coords = rng.uniform(-half, half, (B, N, 3)).astype(np.float32)
    if N > 4:
        coords[0, 1], coords[0, 2, 1], coords[0, 3] = np.nan, np.inf, 1e30
    types = rng.integers(-2, T + 2, (B, N)).astype(np.int32)
    radii = rng.uniform(0.5, 2.0, (B, N) if kind == "atom" else T).astype(np.float32)
    radii.flat[0] = -1.0 if radii.size > 1 else 1.0
    pose = dict(natoms=dev(rng.integers(0, N + 1, B).astype(np.int32)), centers=dev(rng.uniform(-1, 1, (B, 3)).astype(np.float32)),
                quats=dev(rng.standard_normal((B, 4)).astype(np.float32)),
                translations=dev(rng.uniform(-1, 1, (B, 3)).astype(np.float32)))
    gm = mg.GridMaker(res, (D - 1) * res, radius_type_indexed=kind != "atom")
    G = torch.randn(gm.grid_shape(B, T), device="cuda", dtype=dtype, generator=torch.Generator("cuda").manual_seed(1))
    got = []
    try:
        for single in (1, 0):
            mg.set_option("single_launch", single)
            gc = torch.full((B, N, 3), float("nan"), device="cuda")
            if kind == "vector":
                w = rng.random((B, N, T)).astype(np.float32) if not got else w  # noqa: F821
                gw = torch.full((B, N, T), float("nan"), device="cuda")
                gm.mg_backward_vector(dev(coords), dev(w), dev(radii), G, grad_coords=gc, grad_weights=gw, **pose)
                got.append((gc.cpu().numpy().view(np.uint32), gw.cpu().numpy().view(np.uint32)))
            else:
                gm.mg_backward_index(dev(coords), dev(types), dev(radii), T, G, grad_coords=gc, **pose)
                got.append((gc.cpu().numpy().view(np.uint32),))
    finally:
        mg.set_option("single_launch", 1)
    for a, b in zip(*got):
        assert np.array_equal(a, b)
