"""Vector types: the error against 64 bits follows the values, whatever the size of the weights."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import dev, mg  # noqa: E402,F401

# A term is a product of a square root, an exponential, a weight and the squared tail: relative to its
# value some four roundings of at most 2^-24 each, which are independent from term to term, plus half a
# fixed-point step (2^-26) where weights are about one.
REL = 2.0 ** -22


@pytest.mark.parametrize("low,high,signed", [(1, 1, False), (1, 2, False), (4, 8, False), (0.5, 2, True), (30, 50, True)])
@pytest.mark.parametrize("one_hot", [True, False])
def test_error_does_not_grow_with_the_weights(mg, low, high, signed, one_hot):
    B, N, T, D = 2, 1500, 12, 40
    rng = np.random.default_rng(5)
    half = (D - 1) * 0.25 + 1
    coords = rng.uniform(-half, half, (B, N, 3)).astype(np.float32)
    radii = rng.uniform(1.2, 2.0, T).astype(np.float32)
    w = rng.uniform(low, high, (B, N, T))
    if signed:
        w *= rng.choice([-1.0, 1.0], (B, N, T))
    if one_hot:
        w *= np.eye(T)[rng.integers(0, T, (B, N))]
    w = w.astype(np.float32)
    ref = oracle.forward_vector(coords, w, radii, 0.5, (D - 1) * 0.5, out_dtype=np.float64)
    gm = mg.GridMaker(0.5, (D - 1) * 0.5, radius_type_indexed=True)
    got = gm.mg_forward_vector(dev(coords), dev(w), dev(radii)).cpu().numpy()
    assert np.sqrt(((got - ref) ** 2).sum() / (ref ** 2).sum()) <= REL


@pytest.mark.parametrize("D", [48, 41])
@pytest.mark.parametrize("top,share", [(0.32, 0.5), (0.32, 1.0), (0.39, 0.9), (0.39, 0.02), (60.0, 0.3)])
def test_signed_tiles_are_exact_up_to_120(mg, D, top, share):
    """300 atoms on top of each other: a tile's weights add up to some 72 or 90 in magnitude (with one of
    60, to 116), any share of them negative.  Sums in fixed point do not depend on the order of the
    atoms; in floats they would."""
    N, T = 300, 4
    rng = np.random.default_rng(int(D + 100 * share))
    coords = rng.uniform(-1, 1, (1, N, 3)).astype(np.float32)
    radii = rng.uniform(1.2, 2.0, T).astype(np.float32)
    w = rng.uniform(0.5, 1.0, (1, N, T)) * (top if top < 1 else 0.24)
    w *= np.where(rng.random((1, N, T)) < share, -1.0, 1.0)
    if top > 1:
        w[0, 7] = top
    w = w.astype(np.float32)
    assert 60 < np.abs(w).sum(1).max() < 118
    gm = mg.GridMaker(0.5, (D - 1) * 0.5, radius_type_indexed=True)
    outs = []
    for order in (np.arange(N), rng.permutation(N)):
        outs.append(gm.mg_forward_vector(dev(coords[:, order]), dev(w[:, order]), dev(radii)).cpu().numpy())
    mg.set_option("waves_per_tile", 1)
    try:
        outs.append(gm.mg_forward_vector(dev(coords), dev(w), dev(radii)).cpu().numpy())
    finally:
        mg.set_option("waves_per_tile", 0)
    for o in outs[1:]:
        assert np.array_equal(outs[0].view(np.uint32), o.view(np.uint32))
    ref = oracle.forward_vector(coords, w, radii, 0.5, (D - 1) * 0.5, out_dtype=np.float64)
    # every term: half a step, and four roundings of its own size
    assert np.abs(outs[0] - ref).max() <= N * 2.0 ** -26 + REL * np.abs(w).sum(1).max()
