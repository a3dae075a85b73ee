"""Which calls run as one launch: those leave the workspace as it is, the others build tables in it.
On both sides of each rule, and the same results either way."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import dev, mg  # noqa: E402,F401


def route(mg, call, B, N, T, D, res):
    """(whether the call left the workspace alone, its result)"""
    rng = np.random.default_rng(B * N + T)
    gm = mg.GridMaker(res, (D - 1) * res, radius_type_indexed=True)
    coords = dev(rng.uniform(-D / 4, D / 4, (B, N, 3)).astype(np.float32))
    radii = dev(rng.uniform(1.2, 2.0, T).astype(np.float32))
    types = dev(rng.integers(0, T, (B, N)).astype(np.int32))
    ws = torch.full((gm.workspace_bytes(B, N, T),), 7, dtype=torch.uint8, device="cuda")
    if call == "forward":
        out = gm.mg_forward_index(coords, types, radii, T, workspace=ws)
    else:
        grad = torch.randn(gm.grid_shape(B, T), device="cuda", generator=torch.Generator("cuda").manual_seed(2))
        if call == "backward":
            out = gm.mg_backward_index(coords, types, radii, T, grad, workspace=ws)
        else:
            w = dev(rng.random((B, N, T)).astype(np.float32))
            out = torch.cat([o.flatten() for o in gm.mg_backward_vector(coords, w, radii, grad, workspace=ws)])
    return bool((ws == 7).all()), out.cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("call,B,N,T,D,res,single", [
    ("backward_vector", 2, 2040, 28, 48, 0.5, True), ("backward_vector", 3, 2040, 28, 48, 0.5, False),
    ("backward_vector", 1, 2040, 8, 96, 0.5, True), ("backward_vector", 1, 2040, 9, 96, 0.5, False),
    ("backward_vector", 1, 4096, 4, 100, 0.5, False), ("backward_vector", 1, 4097, 4, 100, 0.5, True),
    ("backward_vector", 1, 8192, 4, 128, 0.5, False), ("backward_vector", 1, 8192, 4, 128, 0.25, True),
    ("backward_vector", 1, 6000, 12, 64, 0.5, True), ("backward_vector", 1, 4500, 28, 64, 0.5, False),
    ("backward_vector", 1, 8000, 28, 56, 1.0, True), ("backward_vector", 1, 8000, 28, 64, 1.0, False),
    ("backward_vector", 1, 5000, 20, 96, 0.25, True), ("backward_vector", 1, 5000, 5, 96, 0.5, True),
    ("backward_vector", 1, 5000, 8, 96, 0.5, False),
    ("backward_vector", 2, 4096, 1, 12, 0.5, True), ("backward_vector", 2, 4097, 1, 12, 0.5, False),
    ("forward", 1, 2048, 28, 48, 0.5, True), ("forward", 1, 2049, 28, 48, 0.5, False),
    ("forward", 4, 2040, 28, 48, 0.5, False), ("forward", 100, 65, 8, 16, 1.0, True),
    ("forward", 129, 65, 8, 16, 1.0, False), ("forward", 146, 70, 28, 8, 1.0, True),
    ("forward", 147, 70, 28, 8, 1.0, False), ("forward", 146, 70, 28, 9, 1.0, True),
    ("forward", 29, 70, 28, 15, 1.0, True), ("forward", 30, 70, 28, 15, 1.0, False), ("forward", 32, 64, 14, 24, 0.5, True),
    ("forward", 33, 64, 14, 24, 0.5, False), ("forward", 8, 256, 28, 48, 0.5, False),
    ("backward", 24, 2048, 3, 16, 0.5, True), ("backward", 24, 2049, 3, 16, 0.5, False)])
def test_one_launch_or_tables(mg, call, B, N, T, D, res, single):
    alone, result = route(mg, call, B, N, T, D, res)
    assert alone == single
    mg.set_option("single_launch", 0)
    try:
        alone, tables = route(mg, call, B, N, T, D, res)
    finally:
        mg.set_option("single_launch", 1)
    assert not alone
    assert np.array_equal(result, tables)
