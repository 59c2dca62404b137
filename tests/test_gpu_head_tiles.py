"""Length head and its training step at the edges of their tiles, against the fp64 oracle: 32 prompts x 32
hidden units and depth ranges of 16 waves in the first layer (64 x 64 and 8 waves in larger calls), 32 x 128
tiles of the gradients, four outputs at a time in the second layer."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_15592_amd as estp
from tests._util import check_order_margin, dev, host, rel_l2

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _head(g, d, Hd, K):
    return ((g.standard_normal((Hd, d)) * 0.1).astype(np.float32), (g.standard_normal(Hd) * 0.1).astype(np.float32),
            (g.standard_normal((K, Hd)) * 0.3).astype(np.float32), (g.standard_normal(K) * 0.1).astype(np.float32))


@pytest.mark.parametrize("B,d,Hd,K", [
    (1, 1, 1, 1),          # one of everything
    (31, 7, 33, 5),        # rows that are not 16-byte aligned: single loads
    (33, 127, 31, 17),     # one prompt and one output past a tile, odd depth
    (32, 128, 32, 16),     # whole tiles, one step of each wave
    (64, 260, 129, 2),     # depth ends inside the last wave's range
    (257, 4096, 40, 3),    # deep and narrow: several depth shares
    (5, 4100, 1000, 1024), # the most outputs
    (1100, 64, 70, 50),    # more than one LDS round of the order
    (257, 132, 1000, 16),  # 64 x 64 tiles, one prompt past a tile, depth past a step
    (300, 131, 961, 4),    # the same with single loads, one hidden unit past a tile
])
def test_predict_tiles(B, d, Hd, K):
    g = np.random.default_rng(B + d)
    P = g.standard_normal((B, d)).astype(np.float32)
    W1, b1, W2, b2 = _head(g, d, Hd, K)
    c = np.linspace(50, 3000, K).astype(np.float32)
    y, bins, order = estp.predict(dev(P), dev(W1), dev(b1), dev(W2), dev(b2), dev(c) if K > 1 else None)
    ref, bin_ref, _ = oracle.predict(P, W1, b1, W2, b2, c)
    # ReLU is 1-Lipschitz, so an output is within gamma_(d + Hd + 4) of the sum of its terms' sizes; the
    # expectation over the centres moves by at most that times their range, plus a few ulp of the softmax
    absz = np.abs(P.astype(np.float64)) @ np.abs(W1.astype(np.float64)).T + np.abs(b1)
    do = (d + Hd + 4) * U * (absz @ np.abs(W2.astype(np.float64)).T + np.abs(b2))
    bound = do[:, 0] if K == 1 else do.max(axis=1) * (c[-1] - c[0]) + (K + 20) * U * c[-1]
    assert np.all(np.abs(host(y) - ref) <= bound)
    check_order_margin(host(order), ref, 2 * bound)
    if K > 1:
        a = np.maximum(P.astype(np.float64) @ W1.T + b1, 0)
        o = a @ W2.T.astype(np.float64) + b2
        got = host(bins)
        assert np.all(o[np.arange(B), got] >= o.max(axis=1) - 2 * do.max(axis=1))


@pytest.mark.parametrize("B,d,Hd,K", [
    (1, 4, 1, 2),
    (2, 132, 33, 3),       # one column and one row past a tile
    (17, 128, 32, 33),     # outputs past one tile of W2
    (33, 260, 130, 16),    # W2 rows that are not 16-byte aligned
    (65, 1000, 257, 130),
    (300, 64, 96, 10),
])
def test_head_train_step_tiles(B, d, Hd, K):
    g = np.random.default_rng(B + d + 1)
    W1, b1, W2, b2 = _head(g, d, Hd, K)
    h = g.standard_normal((B, d)).astype(np.float32)
    edges = (np.arange(K + 1) * (4096.0 / K)).astype(np.float32)
    centres = ((edges[1:] + edges[:-1]) / 2).astype(np.float32)
    y = g.uniform(0, 4096, B).astype(np.float32)
    shapes = {"W1": (Hd, d), "b1": (Hd,), "W2": (K, Hd), "b2": (K,)}
    cat = lambda D: np.concatenate([np.asarray(D[k]).ravel() for k in shapes])
    params = {"W1": W1, "b1": b1, "W2": W2, "b2": b2}
    grads = oracle.head_train_step(h, y, edges, centres, params, {k: np.zeros(s) for k, s in shapes.items()},
                                   {k: np.zeros(s) for k, s in shapes.items()}, 1, 0.5, 1e-3)[1]
    size = float(np.sqrt(np.mean(cat(grads) ** 2)))
    # moments of the gradients' size, as in the middle of training: the update is smooth in the gradient
    M = {k: (size * g.standard_normal(s)).astype(np.float32) for k, s in shapes.items()}
    V = {k: (size ** 2 * g.uniform(0.5, 2, s)).astype(np.float32) for k, s in shapes.items()}
    th, m, v = (dev(cat(D).astype(np.float32)) for D in (params, M, V))
    # hyperparameters that are exact in fp32
    hyper = dict(beta1=0.875, beta2=0.9375, eps=2.0 ** -24, weight_decay=0.0625)
    loss = host(estp.head_train_step(dev(h), dev(y), dev(edges), dev(centres), th, m, v, Hd, 50, 0.5, 2.0 ** -10,
                                     **hyper))[0]
    ref_loss, _, Pr, Mr, Vr = oracle.head_train_step(h, y, edges, centres, params, M, V, 50, 0.5, 2.0 ** -10, **hyper)
    # sums of up to d + Hd + K + B fp32 terms of mixed sign: their errors add up like the square root of
    # that many roundings, and the residual y - yhat and the ReLU's edge amplify them a few times
    tol = 16 * U * np.sqrt(d + Hd + K + B)
    print(f"loss {abs(loss / ref_loss - 1):.2e}, m {rel_l2(host(m), cat(Mr)):.2e}, v {rel_l2(host(v), cat(Vr)):.2e}, "
          f"theta {rel_l2(host(th), cat(Pr)):.2e}, bound {tol:.2e}")
    assert abs(loss / ref_loss - 1) <= tol
    for got, want in ((m, Mr), (v, Vr), (th, Pr)):
        assert rel_l2(host(got), cat(want)) <= tol
