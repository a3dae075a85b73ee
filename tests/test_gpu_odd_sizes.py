"""Grids whose channels are no multiple of 16 bytes: forward tiles on the boundaries of the whole
output (short first and last tiles, an empty last one), outputs that begin off 16 bytes, and backward
slots at the end of rows of 1 to 49 points.  Around every output lie values that must stay."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import GRAD_RTOL, dev, grid_tol, mg  # noqa: E402,F401


def framed(shape, dtype, offset):
    """A contiguous tensor `offset` elements into a buffer of sevens, and the buffer."""
    n = int(np.prod(shape))
    buf = torch.full((n + offset + 64,), 7.0, dtype=dtype, device="cuda")
    return buf, buf[offset:offset + n].view(shape)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("D,N,T", [(1, 20, 3), (3, 30, 5), (5, 60, 9), (10, 200, 6), (13, 300, 7), (18, 500, 4),
                                   (21, 900, 5), (31, 2100, 9), (49, 2500, 3)])
def test_against_the_oracle(mg, D, N, T, offset):
    rng = np.random.default_rng(D + N)
    B, res = 3, 0.5
    dim = (D - 1) * res
    side = dim / 2 + 1.5
    centers = rng.uniform(-1, 1, (B, 3)).astype(np.float32)
    coords = (centers[:, None] + rng.uniform(-side, side, (B, N, 3))).astype(np.float32)
    types = rng.integers(0, T, (B, N)).astype(np.int32)
    radii = rng.uniform(0.8, 1.8, T).astype(np.float32)
    w = rng.dirichlet(np.full(T, 0.4), size=(B, N)).astype(np.float32)
    kw = dict(centers=centers)
    dkw = dict(centers=dev(centers))
    co, ty, ra = dev(coords), dev(types), dev(radii)
    ref = oracle.forward_index(coords, types, radii, T, res, dim, **kw)
    refv = oracle.forward_vector(coords, w, radii, res, dim, **kw)
    refb = oracle.forward_binary(coords, radii, T, res, dim, types=types, **kw)
    for single in (1, 0):
        mg.set_option("single_launch", single)
        try:
            for binary, dtype in ((False, torch.float32), (False, torch.float64), (True, torch.float32)):
                gm = mg.GridMaker(res, dim, radius_type_indexed=True, binary=binary)
                buf, out = framed(ref.shape, dtype, offset)
                gm.mg_forward_index(co, ty, ra, T, out=out, **dkw)
                if binary:
                    assert np.array_equal(out.cpu().numpy(), refb)
                else:
                    assert np.abs(out.cpu().numpy() - ref).max() <= grid_tol(ref)
                frame = torch.cat([buf[:offset], buf[offset + out.numel():]])
                assert bool((frame == 7.0).all())
            gm = mg.GridMaker(res, dim, radius_type_indexed=True)
            buf, out = framed(ref.shape, torch.float32, offset)
            gm.mg_forward_vector(co, dev(w), ra, out=out, **dkw)
            assert np.abs(out.cpu().numpy() - refv).max() <= grid_tol(refv)
            assert bool((torch.cat([buf[:offset], buf[offset + out.numel():]]) == 7.0).all())
            G = rng.standard_normal(ref.shape).astype(np.float32)
            for dtype in (torch.float32, torch.float64):
                buf, g = framed(ref.shape, dtype, offset)
                buf.fill_(float("nan"))         # nothing beyond the gradient counts, whatever it holds
                g.copy_(torch.from_numpy(G))
                want = oracle.backward_index(coords, types, radii, T, res, dim, G, **kw)
                got = gm.mg_backward_index(co, ty, ra, T, g, **dkw).cpu().numpy()
                assert np.abs(got - want).max() <= GRAD_RTOL * max(np.abs(want).max(), 1e-3)
                wc, ww = oracle.backward_vector(coords, w, radii, res, dim, G, **kw)
                gc, gw = gm.mg_backward_vector(co, dev(w), ra, g, **dkw)
                assert np.abs(gc.cpu().numpy() - wc).max() <= GRAD_RTOL * max(np.abs(wc).max(), 1e-3)
                assert np.abs(gw.cpu().numpy() - ww).max() <= GRAD_RTOL * max(np.abs(ww).max(), 1e-3)
        finally:
            mg.set_option("single_launch", 1)
