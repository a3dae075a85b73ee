"""Vector types: chords of every length (one voxel to a whole row), signed and large weights about the
limits of the fixed-point tiles, groups of channels with dead ones, other Gaussian radii."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import GRAD_RTOL, dev, grid_tol, mg  # noqa: E402,F401


@pytest.mark.parametrize("D,res,T,N,scale,signed,grm", [
    (16, 1.9, 4, 300, 1.0, False, 1.0),         # chords of one to three voxels
    (24, 0.5, 7, 700, 1.0, True, 1.0),          # many atoms, signed
    (48, 0.06, 3, 60, 1.0, False, 1.0),         # chords as long as the grid
    (130, 0.03, 1, 9, 1.0, True, 1.0),          # ... of 130 voxels, rows longer than a store
    (17, 0.4, 5, 500, 1.0, False, 0.6),         # odd rows; the tail begins at 0.6 radii
    (16, 0.6, 9, 300, 1.0, False, 1.7),         # ... at 1.7
    (12, 0.5, 4, 160, 1.0, True, 1.0),          # sums of the weights on either side of 60, signed
    (12, 0.5, 4, 300, 1.0, False, 1.0),         # ... of 120
    (12, 0.5, 6, 40, 30.0, True, 1.0),          # large weights: float tiles
])
def test_against_the_oracle(mg, D, res, T, N, scale, signed, grm):
    rng = np.random.default_rng(1000 * D + N)
    B, dim = 2, (D - 1) * res
    side = dim / 2 + 2.0
    centers = rng.uniform(-1, 1, (B, 3)).astype(np.float32)
    coords = (centers[:, None] + rng.uniform(-side, side, (B, N, 3))).astype(np.float32)
    w = (scale * rng.random((B, N, T)) ** 2).astype(np.float32)
    w[:, ::7, 0] = 0.0
    w[0, 3] = 0.0
    if signed:
        w[:, :, T // 2] *= rng.choice([-1.0, 1.0], (B, N)).astype(np.float32)
    radii = rng.uniform(0.9, 1.6, T).astype(np.float32)
    if T > 4:
        radii[2] = 0.0          # a dead channel inside a group
    kw = dict(centers=centers, quats=rng.standard_normal((B, 4)).astype(np.float32))
    dkw = {k: dev(v) for k, v in kw.items()}
    gm = mg.GridMaker(res, dim, radius_type_indexed=True, gaussian_radius_multiple=grm)
    ref = oracle.forward_vector(coords, w, radii, res, dim, grm=grm, **kw)
    outs = [gm.mg_forward_vector(dev(coords), dev(w), dev(radii), **dkw).cpu().numpy() for _ in range(2)]
    assert np.array_equal(outs[0].view(np.uint32), outs[1].view(np.uint32))
    # grid_tol covers sums of terms up to 1; larger weights scale the rounding of every term
    assert np.abs(outs[0] - ref).max() <= grid_tol(ref) * max(1.0, scale)
    out64 = gm.mg_forward_vector(dev(coords), dev(w), dev(radii), dtype=torch.float64, **dkw).cpu().numpy()
    assert np.abs(out64 - ref).max() <= grid_tol(ref) * max(1.0, scale)
    G = rng.standard_normal(ref.shape).astype(np.float32)
    wc, ww = oracle.backward_vector(coords, w, radii, res, dim, G, grm=grm, **kw)
    gc, gw = gm.mg_backward_vector(dev(coords), dev(w), dev(radii), dev(G), **dkw)
    assert np.abs(gc.cpu().numpy() - wc).max() <= GRAD_RTOL * np.abs(wc).max()
    assert np.abs(gw.cpu().numpy() - ww).max() <= GRAD_RTOL * np.abs(ww).max()
