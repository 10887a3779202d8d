"""The early-stop classifier's matrix kernels at the edges of their tiles: 16 samples a
tile, one or four tiles per wavefront in inference, up to 2048 wavefronts in training.

The bars are those of the classifier's oracle tests: probabilities within 1e-5 and loss
within 1e-5 relative of the binary64 forward, gradients within 1e-4 in the 2-norm.
"""
import numpy as np
import pytest

import oracle as orc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible to torch")
    from paper_2004_03972_amd import hqa
    hqa.lib()
    return hqa


def _es(H, seed):
    es = H.ES(seed=1)
    es.params = np.random.default_rng(seed).normal(0, 0.25, size=5187)
    return es, es.params.astype(np.float64)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 65536, 65537, 65600 + 49])
def test_predict_tile_edges(H, n):
    es, P = _es(H, n)
    x = np.random.default_rng(n).normal(size=(n, 12)).astype(np.float32)
    pr = es.predict(x)
    assert np.max(np.abs(pr - orc.mlp_forward(P, x.astype(np.float64)))) < 1e-5
    # a sample's result does not depend on its place among the tiles
    m = min(n, 40)
    assert np.array_equal(pr[n - m:], es.predict(x[n - m:]))
    pb = es.predict(x, bf16=True)
    assert np.array_equal(pb[n - m:], es.predict(x[n - m:], bf16=True))
    assert np.max(np.abs(pb - pr)) < 5e-2


@pytest.mark.parametrize("n", [1, 15, 16, 17, 64, 65, 131, 8192 + 3, 32768 + 70])
def test_gradient_tile_edges(H, n):
    es, P = _es(H, n + 1)
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, 12)).astype(np.float32)
    y = rng.integers(0, 3, size=n).astype(np.int32)
    cw = np.array([1.0, 1.5, 6.0])
    loss, g = es.grad(x, y, cw)
    lo, go = orc.mlp_loss_grad(P, x.astype(np.float64), y, cw)
    assert loss == pytest.approx(lo, rel=1e-5)
    assert np.linalg.norm(g - go) <= 1e-4 * np.linalg.norm(go)
    l2, g2 = es.grad(x, y, cw)                       # fixed order of every sum
    assert l2 == loss and np.array_equal(g, g2)
