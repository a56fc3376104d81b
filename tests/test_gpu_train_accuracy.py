"""Accuracy of the training kernels' parts, each read off a gradient whose other factors are exact.

With W2 = 0 and W3 = 1, one row of dy = 1 leaves db2 = gelu'(b2) and dW3 = bf16(gelu(b2)) of 128 chosen arguments.
With every pre-activation far in GELU's linear range all slopes are 1, so dz2 = dy w3 and, the features being rows of
the identity, dW1 = W2^T dz2: the contraction alone.  The bounds are the errors of the plain FP32 forms against 64
bits, relative RMS with every operation rounded to nearest: 0.5 (1 + tanh u) + 0.5 x (1 - tanh^2 u) u' 6.5e-8 on
N(0, 1.5), a chain of 128 fmas 2.0e-7."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_2202_12567_amd import api  # noqa: E402

DEV = torch.device("cuda", 0)
H, K = 128, 12


def gradient(W1, b1, W2, b2, W3, F, dy):
    """The gradient's tensors in parameter order (W1, b1, W2, b2, W3, b3)."""
    pv = np.concatenate([np.ravel(a) for a in (W1, b1, W2, b2, W3, [0.0])]).astype(np.float32)
    t = [torch.as_tensor(np.ascontiguousarray(a, np.float32)).to(DEV) for a in (pv, F, dy)]
    g = api.mlp_grad(api.Context(0), *t).cpu().numpy()
    return np.split(g, np.cumsum([H * K, H, H * H, H, H]))


def at(x):
    """gelu'(x) and bf16(gelu(x)) of 128 arguments."""
    g = gradient(np.zeros((H, K)), np.zeros(H), np.zeros((H, H)), x, np.ones(H), np.zeros((1, K)), np.ones(1))
    return g[3], g[4]


def exact(x):
    x = x.astype(np.float64)
    a = np.sqrt(2 / np.pi)
    u = a * (x + 0.044715 * x ** 3)
    e = np.exp(-2 * np.abs(u))
    s, c = np.where(u >= 0, 1, e) / (1 + e), np.where(u >= 0, e, 1) / (1 + e)
    return x * s, s + 2 * x * a * (1 + 3 * 0.044715 * x * x) * s * c


def bf16(x):
    return torch.as_tensor(x.astype(np.float32)).bfloat16().double().numpy()


def rms(parts):
    err, ref = (sum(p[k] for p in parts) for k in (0, 1))
    return np.sqrt(err / ref)


@pytest.mark.parametrize("spread", [0.5, 1.5, 4.0])
def test_slope(spread):
    rng = np.random.default_rng(1)
    parts = []
    for _ in range(64):
        x = rng.normal(0, spread, H).astype(np.float32)
        act, want = exact(x)
        got, h = at(x)
        parts.append((((got - want) ** 2).sum(), (want ** 2).sum()))
        # activations are rounded to bfloat16 from FP32 values good to a few ulp: the rounding of the 64-bit value but
        # for near ties, never more than one bfloat16 step away
        assert (h == bf16(act)).mean() > 0.95 and np.all(np.abs(h - bf16(act)) <= np.abs(act) / 128 + 1e-30)
    assert rms(parts) <= {0.5: 4.0e-8, 1.5: 6.5e-8, 4.0: 1.51e-7}[spread]


def test_saturates_far_from_zero():
    """Where the sigmoid is 0 or 1 in FP32 the slope is 0 or 1, at every finite argument whose cube may overflow too."""
    x = np.array([s * 10.0 ** e for e in np.linspace(1.2, 38, 64) for s in (1, -1)], np.float32)
    got, h = at(x)
    assert np.array_equal(got, np.where(x > 0, 1.0, 0.0))
    assert np.array_equal(h, np.where(x > 0, bf16(x), 0.0))


def test_contraction_of_the_second_layer():
    rng = np.random.default_rng(2)
    parts = []
    for _ in range(40):
        W2, W3 = rng.normal(0, np.sqrt(2 / H), (H, H)), rng.normal(0, np.sqrt(1 / H), H)
        dy = rng.normal(0, 1, K).astype(np.float32)
        g = gradient(np.zeros((H, K)), np.full(H, 32.0), W2, np.full(H, 1000.0), W3, np.eye(K), dy)
        dz2 = dy[:, None] * bf16(W3).astype(np.float32)
        want = dz2.astype(np.float64) @ bf16(W2)
        parts.append((((g[0].reshape(H, K).T - want) ** 2).sum(), (want ** 2).sum()))
    assert rms(parts) <= 2.0e-7
