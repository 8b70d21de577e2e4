"""Precision of the split float32 products, per tile shape, against 64 bits.

The networks are built so that every product under test is a sum of positive
terms whose operands have all three bf16 pieces positive and near their
largest (1 + i/128, then j 2^-15, then k 2^-23, times a power of two): losing
any one of the six piece products moves every result the same way, by 2^-18
of it or more, and the bounds here are 2^-20 and 2^-21.  The output weights
are negative and those of class 0 zero, so that the softmax is exactly
(1, 0, ...), every loss is -z_y and every output gradient +-1/m: what comes
back is a product of known operands.

The exponents also take the operands, one after the other, to where bf16 has
no values for the low pieces of an unscaled split, and the results above
2^96, where a tile is computed again in float32 (one rounding per two
products there: bound 2^-18)."""
import os
import re

import numpy as np
import pytest

from tests.helpers import to_device

pytestmark = pytest.mark.gpu

SPLIT_BOUND, REDO_BOUND = 2.0 ** -21, 2.0 ** -18
SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1710_02368_amd", "csrc",
                      "gemm_f32_split.hip")


def rule(name):
    """A threshold of the dispatch, from the source that states it."""
    with open(SOURCE) as f:
        return int(re.search(r"\b%s = (\d+)" % name, f.read()).group(1))


def tiles(n, rows, cols, bm=64, bn=64):
    return n * -(-rows // bm) * -(-cols // bn)


def forward_shape(n, m, out, inp):
    if n > 1 and m > 64 and tiles(n, m, out, 128) >= rule("kWideTiles"):
        return "wide"
    t = tiles(n, m, out)
    if t >= rule("kMidTiles"):
        return "mid"
    if inp % 4:  # (single-float loads)
        return "small" if t < rule("kFlatTilesWords") else "flat"
    return "small" if t < rule("kFlatTiles") else "deep" if t <= rule("kDeepTiles") else "flat"


def dw_shape(n, out, inp):
    return "midw" if tiles(n, out, inp) >= rule("kMidWTiles") else "small"


def bwd_shape(n, m, out, inp):
    if dw_shape(n, out, inp) == "small":
        return "small"
    return "flat+midw" if tiles(n, m, inp) >= rule("kFlatDxTiles") else "small+midw"


def structured(rng, shape, e):
    i, j, k = rng.integers(0, 128, shape), rng.integers(64, 127, shape), rng.integers(32, 63, shape)
    return np.ldexp(1.0 + i / 128.0 + j * 2.0 ** -15 + k * 2.0 ** -23, e).astype(np.float32)


def output_weights(rng, C, d, e):
    w = -structured(rng, (C, d), e)
    w[0] = 0.0
    return w


def one_round(dims, n, m, weights, X, y, eta):
    """Losses and committed deltas (not normalized, lambda = 1) of one round."""
    import torch

    import paper_1710_02368_amd as agn
    vec = np.concatenate([np.concatenate([w.ravel(), np.zeros(w.shape[0], np.float32)]) for w in weights])
    g = agn.AGN(dims, n, 1, eta, m, seed=1, normalize=False)
    g.set_central(torch.from_numpy(vec).cuda())
    g.round(*to_device(X, y), list(range(n)))
    loss, deltas = g.loss().cpu().numpy(), [g.delta(k).cpu().numpy() for k in range(n)]
    g.close()
    at = np.cumsum([0] + [w.size + w.shape[0] for w in weights])
    return loss, [[d[at[l]:at[l] + w.size].reshape(w.shape).astype(np.float64) for l, w in enumerate(weights)]
                  for d in deltas]


def step_rate(w, grads):
    """A power of two that makes every step 2^14 times the weights or more, so
    that the rounding of weight plus step is that of the step (two roundings,
    2^-23 of it)."""
    need = 2.0 ** 14 * np.max(np.abs(w)) / np.min([g[g != 0].min() for g in grads])
    return float(2.0 ** np.clip(np.ceil(np.log2(need)), -20, 100))


def check_step(delta, grad, eta, redo, what):
    ref = -eta * grad
    err = np.max(np.abs(delta - ref)[ref != 0] / np.abs(ref)[ref != 0])
    print(what, "step", err * 2.0 ** 21, "x 2^-21", flush=True)
    assert np.all(delta[ref == 0] == 0)
    assert err <= (REDO_BOUND if redo else SPLIT_BOUND), (what, err)


# dims, n, m, shape of the first layer's forward product, of its weight gradient
TWO_LAYERS = {
    "small": ((100, 70, 10), 2, 32, "small", "small"),
    "small_unaligned": ((101, 70, 10), 2, 32, "small", "small"),
    "small_linear": ((64, 96, 40), 3, 32, "small", "small"),         # (logits by the split product)
    "small_full": ((132, 514, 10), 16, 64, "small", "midw"),
    "deep": ((132, 900, 10), 16, 64, "deep", "midw"),
    "flat": ((132, 1100, 10), 16, 64, "flat", "midw"),
    "flat_unaligned": ((131, 514, 10), 16, 64, "flat", "midw"),
    "mid": ((68, 580, 10), 40, 128, "mid", "midw"),
    "wide": ((36, 900, 10), 40, 256, "wide", "midw"),
    "wide_unaligned": ((37, 900, 10), 40, 256, "wide", "midw"),
}
# exponents of X, W0, W1; results of at least 2^96 in the forward product, in the weight gradient
TWO_LAYER_RANGES = {
    "ordinary": (0, 0, 0, False, False),
    "tiny_rows": (-120, 42, 81, False, False),
    "tiny_weights": (58, -120, 65, False, True),
    "tiny_gradients": (95, 22, -115, True, False),
}


@pytest.mark.parametrize("rng_name", TWO_LAYER_RANGES)
@pytest.mark.parametrize("case", TWO_LAYERS)
def test_forward_and_first_layer(case, rng_name):
    dims, n, m, fwd, dw = TWO_LAYERS[case]
    assert (forward_shape(n, m, dims[1], dims[0]), dw_shape(n, dims[1], dims[0])) == (fwd, dw)
    ex, e0, e1, redo_fwd, redo_dw = TWO_LAYER_RANGES[rng_name]
    print(case, rng_name, dims, n, m, flush=True)
    rng = np.random.default_rng(5)
    X, W0, W1 = structured(rng, (n * m, dims[0]), ex), structured(rng, (dims[1], dims[0]), e0), output_weights(
        rng, dims[2], dims[1], e1)
    y = rng.integers(1, dims[2], n * m).astype(np.int32)
    x64, w0, w1 = (v.astype(np.float64) for v in (X, W0, W1))
    want = -np.sum((x64 @ w0.T) * w1[y], axis=1).reshape(n, m).mean(axis=1)
    assert want.min() > 400  # (every other class's probability is exactly zero)
    grads = [(-w1[y[k * m:(k + 1) * m]] / m).T @ x64[k * m:(k + 1) * m] for k in range(n)]
    eta = step_rate(W0, grads)
    loss, deltas = one_round(dims, n, m, [W0, W1], X, y, eta)
    err = np.max(np.abs(loss / want - 1.0))
    print(case, rng_name, "loss", err * 2.0 ** 20, "x 2^-20", flush=True)
    assert err <= (REDO_BOUND if redo_fwd else 2 * SPLIT_BOUND), err  # (the output layer's float32 sums among them)
    for k in range(n):
        check_step(deltas[k][0], grads[k], eta, redo_dw, (case, rng_name, k))


# dims, n, m, shape of the second layer's backward launch
THREE_LAYERS = {
    "small": ((20, 70, 66, 10), 2, 32, "small"),
    "small_linear": ((20, 70, 66, 40), 2, 32, "small"),
    "flat+midw": ((24, 520, 500, 10), 16, 64, "flat+midw"),
    "small+midw": ((24, 260, 520, 10), 16, 64, "small+midw"),
}
# exponents of W0, W1, W2, the layer whose step is checked, results of at least 2^96 on the way to it
THREE_LAYER_RANGES = {
    "ordinary": (0, 0, 0, 1, False),
    "ordinary_dx": (0, 0, 0, 0, False),
    "tiny_inputs": (-120, 37, 81, 1, False),
    "large_dx": (-120, 37, 81, 0, True),
    "tiny_weights_dx": (40, -118, 82, 0, False),
    "large_dw": (40, -118, 82, 1, True),
    "tiny_gradients": (72, 39, -113, 1, False),
    "tiny_gradients_dx": (10, 101, -113, 0, False),
}


@pytest.mark.parametrize("rng_name", THREE_LAYER_RANGES)
@pytest.mark.parametrize("case", THREE_LAYERS)
def test_backward_launch(case, rng_name):
    """Rows of X with a single one: the first layer's activations are columns
    of W0 and its step is a sum of rows of the input gradient, so that both
    products of the second layer's launch have known operands."""
    dims, n, m, bwd = THREE_LAYERS[case]
    assert bwd_shape(n, m, dims[2], dims[1]) == bwd
    e0, e1, e2, layer, redo = THREE_LAYER_RANGES[rng_name]
    print(case, rng_name, dims, n, m, flush=True)
    rng = np.random.default_rng(6)
    W0, W1 = structured(rng, (dims[1], dims[0]), e0), structured(rng, (dims[2], dims[1]), e1)
    W2 = output_weights(rng, dims[3], dims[2], e2)
    X = np.eye(dims[0], dtype=np.float32)[rng.integers(0, dims[0], n * m)]
    y = rng.integers(1, dims[3], n * m).astype(np.int32)
    x64, w0, w1, w2 = (v.astype(np.float64) for v in (X, W0, W1, W2))
    h1 = x64 @ w0.T
    assert -np.max(np.sum((h1 @ w1.T) * w2[y], axis=1)) > 400
    dz2 = -w2[y] / m
    a, b = (dz2, h1) if layer else (dz2 @ w1, x64)
    grads = [a[k * m:(k + 1) * m].T @ b[k * m:(k + 1) * m] for k in range(n)]
    eta = step_rate((W0, W1)[layer], grads)
    _, deltas = one_round(dims, n, m, [W0, W1, W2], X, y, eta)
    for k in range(n):
        check_step(deltas[k][layer], grads[k], eta, redo, (case, rng_name, k))
