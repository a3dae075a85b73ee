"""Backward, vector types: channels in groups of four and lanes of 64 (one group in any order, dead channels,
a second set of lanes), rows shorter than a slot and rows whose last slot reaches past their end."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import GRAD_RTOL, dev, mg  # noqa: E402,F401


@pytest.mark.parametrize("T", [1, 3, 4, 5, 8, 64, 65, 69])
@pytest.mark.parametrize("D,res", [(2, 1.1), (3, 0.7), (5, 0.9), (7, 0.25), (16, 0.5)])
def test_channel_groups(mg, T, D, res):
    B, N = 2, 60
    rng = np.random.default_rng(100 * T + D)
    dim = (D - 1) * res
    coords = rng.uniform(-dim / 2 - 1.5, dim / 2 + 1.5, (B, N, 3)).astype(np.float32)
    coords[0, 0] = 0.5 * res * (1 - D % 2)          # on a voxel: its distance from it is 0
    w = rng.standard_normal((B, N, T)).astype(np.float32)
    radii = rng.uniform(1.0, 1.9, T).astype(np.float32)
    if T > 4:
        radii[[1, T - 1]] = [0.0, -1.0]             # dead channels: no gradient, nothing for the others
    G = rng.standard_normal((B, T, D, D, D)).astype(np.float32)
    wc, ww = oracle.backward_vector(coords, w, radii, res, dim, G)
    gm = mg.GridMaker(res, dim, radius_type_indexed=True)
    outs = []
    for single in (1, 0):                           # one launch; on tables
        mg.set_option("single_launch", single)
        try:
            outs.append(gm.mg_backward_vector(dev(coords), dev(w), dev(radii), dev(G)))
        finally:
            mg.set_option("single_launch", 1)
    for gc, gw in outs:
        assert np.abs(gc.cpu().numpy() - wc).max() <= GRAD_RTOL * np.abs(wc).max()
        assert np.abs(gw.cpu().numpy() - ww).max() <= GRAD_RTOL * np.abs(ww).max()
    for a, b in zip(*outs):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("radius", [1e-3, 1e-11, 1e-13, 1e-15, 1e-20, 1e-30])
@pytest.mark.parametrize("T", [3, 9])
def test_radii_far_below_a_grid_step(mg, T, radius):
    """An atom on a voxel counts there in full (rho(0) = 1) and nowhere else; beside channels of usual radii."""
    B, N, D, res = 1, 40, 9, 0.5
    rng = np.random.default_rng(T)
    dim = (D - 1) * res
    coords = (rng.integers(0, D, (B, N, 3)) * res - dim / 2).astype(np.float32)
    w = rng.standard_normal((B, N, T)).astype(np.float32)
    radii = np.where(np.arange(T) % 3 == 1, 1.4, radius).astype(np.float32)
    G = rng.standard_normal((B, T, D, D, D)).astype(np.float32)
    wc, ww = oracle.backward_vector(coords, w, radii, res, dim, G)
    gm = mg.GridMaker(res, dim, radius_type_indexed=True)
    for single in (1, 0):
        mg.set_option("single_launch", single)
        try:
            gc, gw = gm.mg_backward_vector(dev(coords), dev(w), dev(radii), dev(G))
        finally:
            mg.set_option("single_launch", 1)
        assert np.abs(gc.cpu().numpy() - wc).max() <= GRAD_RTOL * np.abs(wc).max()
        for t in range(T):      # (by channel: the narrow ones beside the wide)
            assert np.abs(gw.cpu().numpy() - ww)[..., t].max() <= GRAD_RTOL * np.abs(ww[..., t]).max(), t
