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
