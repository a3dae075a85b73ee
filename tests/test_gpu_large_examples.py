"""Examples past what one workgroup sorts (8192 atoms): several workgroups each sort their share of
the keys.  Sizes around a round of the workgroup's threads, channels that no share divides evenly,
atoms crowded into one x-plane (bins past 2048 atoms take another route), skipped types, natoms."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import GRAD_RTOL, dev, grid_tol, mg  # noqa: E402,F401


@pytest.mark.parametrize("B,N,T,D,crowd", [(1, 8193, 3, 13, 0), (2, 12289, 1, 16, 0),
                                           (3, 9001, 37, 9, 0), (1, 10007, 2, 12, 5000),
                                           (1, 300, 1300, 8, 0)])
def test_against_the_oracle(mg, B, N, T, D, crowd):
    rng = np.random.default_rng(N + T)
    res, dim = 0.75, (D - 1) * 0.75
    centers = rng.uniform(-2, 2, (B, 3)).astype(np.float32)
    coords = (centers[:, None] + rng.uniform(-dim / 2 - 3, dim / 2 + 3, (B, N, 3))).astype(np.float32)
    if crowd:                   # more than 2048 atoms of one type in one plane's bin, out of order
        coords[:, rng.permutation(N)[:crowd], 0] = centers[:, :1] + 0.4
    types = rng.integers(-1, T + 1, (B, N)).astype(np.int32)
    radii = rng.uniform(0.6, 1.5, T).astype(np.float32)
    natoms = rng.integers(N // 2, N + 1, B).astype(np.int32)
    quats = None if crowd else rng.standard_normal((B, 4)).astype(np.float32)
    pose = dict(natoms=natoms, centers=centers, quats=quats)
    dpose = {k: dev(v) for k, v in pose.items()}
    gm = mg.GridMaker(res, dim, radius_type_indexed=True)
    co, ty, ra = dev(coords), dev(types), dev(radii)
    outs = [gm.mg_forward_index(co, ty, ra, T, **dpose).cpu().numpy() for _ in range(2)]
    ref = oracle.forward_index(coords, types, radii, T, res, dim, **pose)
    assert np.array_equal(outs[0].view(np.uint32), outs[1].view(np.uint32))
    assert np.abs(outs[0] - ref).max() <= grid_tol(ref)
    gmb = mg.GridMaker(res, dim, radius_type_indexed=True, binary=True)
    refb = oracle.forward_binary(coords, radii, T, res, dim, types=types, **pose)
    assert np.array_equal(gmb.mg_forward_index(co, ty, ra, T, **dpose).cpu().numpy(), refb)
    G = rng.standard_normal(ref.shape).astype(np.float32)
    want = oracle.backward_index(coords, types, radii, T, res, dim, G, **pose)
    got = gm.mg_backward_index(co, ty, ra, T, dev(G), **dpose).cpu().numpy()
    assert np.abs(got - want).max() <= GRAD_RTOL * np.abs(want).max()
    if T > 8:
        return
    w = rng.dirichlet(np.full(T, 0.4), size=(B, N)).astype(np.float32)
    outs = [gm.mg_forward_vector(co, dev(w), ra, **dpose).cpu().numpy() for _ in range(2)]
    refv = oracle.forward_vector(coords, w, radii, res, dim, **pose)
    assert np.array_equal(outs[0].view(np.uint32), outs[1].view(np.uint32))
    assert np.abs(outs[0] - refv).max() <= grid_tol(refv)
    wc, ww = oracle.backward_vector(coords, w, radii, res, dim, G, **pose)
    gc, gw = gm.mg_backward_vector(co, dev(w), ra, dev(G), **dpose)
    assert np.abs(gc.cpu().numpy() - wc).max() <= GRAD_RTOL * np.abs(wc).max()
    assert np.abs(gw.cpu().numpy() - ww).max() <= GRAD_RTOL * np.abs(ww).max()
