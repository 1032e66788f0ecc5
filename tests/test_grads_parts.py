"""What the bar of the matrix-core gradients' GPU tests can see, on the CPU: the six products of bf16
parts, in 64-bit sums, stay far below it, and each of them left out, in either product, goes past it."""
import numpy as np
import pytest

from test_grads_gpu import BAR


def bf16(v, nearest):
    b = v.astype(np.float32).view(np.uint32)
    if nearest:
        b = b + 0x7fff + ((b >> 16) & 1)
    return (b & np.uint32(0xffff0000)).view(np.float32)


def parts(v, nearest):
    out, left = [], v.astype(np.float32)
    for _ in range(3):
        out.append(bf16(left, nearest))
        left = left - out[-1]
    return out


KEPT = [(0, 0), (0, 1), (1, 0), (0, 2), (1, 1), (2, 0)]


def product(a, b, kept):
    """a @ b from the kept products of parts; a is split to nearest, b by truncation."""
    pa, pb = parts(a, True), parts(b, False)
    return sum(pa[i].astype(np.float64) @ pb[j].astype(np.float64) for i, j in kept)


def gradient_error(n, d, b, loss, kept_z, kept_g):
    rng = np.random.default_rng([n, d, b])
    X = (rng.standard_normal((n, d)) * d ** -0.5).astype(np.float32)
    y = (rng.random(n) < 0.5).astype(np.float32)
    W = rng.standard_normal((b, d)).astype(np.float32)
    act = (lambda z: z) if loss == "linear" else (lambda z: 1 / (1 + np.exp(-z)))
    U = (act(product(X, W.T, kept_z)) - y[:, None]).astype(np.float32)
    G = product(X.T, U, kept_g)
    ref = X.T.astype(np.float64) @ (act(X.astype(np.float64) @ W.T.astype(np.float64)) - y[:, None])
    return (np.linalg.norm(G - ref, axis=0) / np.linalg.norm(ref, axis=0)).max()


@pytest.mark.parametrize("n,d,b", [(64, 4096, 4), (33, 8191, 31), (17, 2001, 64), (300, 70, 60)])
def test_bar_sees_every_product(n, d, b):
    assert gradient_error(n, d, b, "linear", KEPT, KEPT) < 0.2 * BAR
    assert gradient_error(n, d, b, "logistic", KEPT, KEPT) < 0.2 * BAR
    for k in KEPT:
        left = [p for p in KEPT if p != k]
        assert gradient_error(n, d, b, "linear", left, KEPT) > BAR
        assert gradient_error(n, d, b, "linear", KEPT, left) > BAR
