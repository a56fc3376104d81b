"""Infinities in the training kernels: a gradient is infinite where the sum over the rows is, and not a number only
where that sum is.  The values are chosen so that no sum holds infinities of both signs or an infinity times 0."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2202_12567_amd import api  # noqa: E402

DEV = torch.device("cuda", 0)
H, K = 128, 12


def gradient(W1, b1, W2, b2, W3, F, dy):
    """The gradient's tensors W1, b1, W2, b2, W3, b3."""
    pv = np.concatenate([np.ravel(a) for a in (W1, b1, W2, b2, W3, [0.0])]).astype(np.float32)
    t = [torch.as_tensor(np.ascontiguousarray(a, np.float32)).to(DEV) for a in (pv, F, dy)]
    g = np.split(api.mlp_grad(api.Context(0), *t).cpu().numpy(), np.cumsum([H * K, H, H * H, H, H]))
    return g[0].reshape(H, K), g[1], g[2].reshape(H, H), g[3], g[4], g[5]


@pytest.mark.parametrize("rows", [32, 256])
def test_infinite_activation(rows):
    """gelu(inf) = inf with slope 1: of two units with an infinite bias dW3 is infinite, db2 finite."""
    b2 = np.ones(H)
    b2[[3, 100]] = np.inf
    _, _, _, gb2, gw3, _ = gradient(np.zeros((H, K)), np.zeros(H), np.zeros((H, H)), b2, np.ones(H), np.ones((rows, K)),
                                    np.ones(rows))
    assert np.array_equal(np.isposinf(gw3), np.isinf(b2)) and np.isfinite(gw3[b2 == 1]).all()
    assert np.all(gb2[[3, 100]] == rows) and np.isfinite(gb2).all()


@pytest.mark.parametrize("rows", [1, 5, 33, 300])
def test_rows_past_the_end_add_nothing(rows):
    """Row counts that fill no tile: an infinite bias of either layer must not meet the 0 of a row past the end."""
    b1, b2 = np.ones(H), np.ones(H)
    b1[7] = b2[3] = np.inf
    W2 = np.full((H, H), 0.01)
    gw1, gb1, gw2, gb2, gw3, gb3 = gradient(np.zeros((H, K)), np.zeros(H), np.zeros((H, H)), b2, np.ones(H),
                                            np.ones((rows, K)), np.ones(rows))
    assert np.array_equal(np.isposinf(gw3), np.isinf(b2)) and np.isfinite(gw3[b2 == 1]).all()
    # first layer: every z2 is infinite then, every slope of the second layer 1
    gw1, gb1, gw2, gb2, gw3, gb3 = gradient(np.zeros((H, K)), b1, W2, np.zeros(H), np.ones(H), np.ones((rows, K)),
                                            np.ones(rows))
    assert np.isposinf(gw3).all() and np.all(gb2 == rows) and np.all(gb3 == rows)
    assert np.isposinf(gw2[:, 7]).all() and np.isfinite(np.delete(gw2, 7, 1)).all()
    assert np.isfinite(gw1).all() and np.isfinite(gb1).all()


@pytest.mark.parametrize("dy,w3", [(np.inf, 1.0), (-np.inf, 1.0), (3e38, 2.0)])
def test_infinite_slope_of_the_second_layer(dy, w3):
    """dz2 infinite (given so, or by overflow) reaches the first layer's gradients as an infinity."""
    W2 = np.random.default_rng(5).uniform(0.01, 0.02, (H, H))
    gw1, gb1, gw2, gb2, gw3, _ = gradient(np.zeros((H, K)), np.full(H, 32.0), W2, np.full(H, 1000.0), np.full(H, w3),
                                          np.ones((1, K)), np.array([dy]))
    for g in (gw1, gb1, gw2, gb2, gw3):
        assert np.array_equal(g, np.full(g.shape, np.copysign(np.inf, dy)))
