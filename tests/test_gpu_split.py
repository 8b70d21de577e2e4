"""The split float32 products at the edges of their tiles: every tile shape of
the forward, input-gradient and weight-gradient products with ragged rows,
columns and K, data rows that no 16-byte load fits, batches that wrap round
their shard or exceed it, and operands that are not finite."""
import numpy as np
import pytest

import workloads as W
from oracle import AGNOracle, evaluate, unflat_params
from tests.helpers import to_device

pytestmark = pytest.mark.gpu

# dims, n, m, N: one layer of each case lands on the named shape
CASES = {
    "small_unaligned": ((101, 71, 60, 40), 2, 20, 400),         # 32 x 32 tiles, single-float loads of the data
    "small_k1": ((1, 33, 5, 3), 3, 7, 100),                     # K = 1, one column past a tile
    "flat_midw": ((130, 514, 66, 10), 16, 70, 16 * 90),         # 32 x 64 forward, 64 x 64 weight gradient, m > 64
    "flat_midw_unaligned": ((131, 514, 66, 12), 16, 70, 16 * 90),
    "flat_bwd": ((64, 260, 514, 10), 16, 70, 16 * 90),          # 32 x 64 input gradient beside 64 x 64 weight tiles
    "deep": ((132, 450, 66, 10), 16, 70, 16 * 90),              # 64 x 64 forward, three stages
    "mid": ((68, 385, 33, 10), 40, 130, 40 * 200),              # 64 x 64 forward
    "wide": ((36, 700, 33, 10), 48, 130, 48 * 200),             # 128 x 64 forward, the second row tile of 2 rows
    "wide_unaligned": ((37, 700, 33, 10), 48, 130, 48 * 200),
    "batch_over_shard": ((50, 70, 66, 10), 2, 50, 60),          # m = 50 rows of shards of 30
    "batch_over_shard_unaligned": ((51, 70, 66, 10), 2, 50, 60),
}


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("adam", [None, (0.9, 0.999, 1e-5)], ids=["sgd", "adam"])
def test_round_matches_oracle(case, adam):
    import paper_1710_02368_amd as agn
    dims, n, m, N = CASES[case]
    print(case, dims, n, m, N, adam, flush=True)
    wl = W.small_workload(case, dims, n, 2, m, 0.02 if adam is None else 0.001, 1, N, order="permutation")
    X, y = W.make_data(wl)
    xd, yd = to_device(X, y)
    g = agn.AGN(dims, n, wl.lam, wl.eta, m, seed=3, adam=adam)
    o = AGNOracle(dims, n, wl.lam, wl.eta, m, seed=3, adam=adam)
    order = W.commit_orders(wl)[0]
    g.round(xd, yd, order)
    o.round(X, y, order)
    np.testing.assert_allclose(g.loss().cpu().numpy(), o.last_loss, rtol=2e-6)
    a, b = g.central().cpu().numpy().astype(np.float64), o.central_flat().astype(np.float64)
    # float32 sums of up to 700 terms; a unit at a ReLU edge moves its own row
    assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b)
    assert np.max(np.abs(a - b)) <= 1e-3 * np.max(np.abs(b))
    # each worker's step, against the displacement the oracle takes: 1e-2 in
    # the 2-norm per tensor leaves room for such a unit and for the rounding
    # of theta itself (half an ulp per step)
    theta = unflat_params(o.central_flat(), dims)
    for k in range(0, n, 7):
        d = unflat_params(g.delta(k).cpu().numpy(), dims)
        ref = unflat_params(np.concatenate([np.concatenate([w.ravel(), v.ravel()]) for w, v in o.last_deltas[k]]), dims)
        for (dw, db), (rw, rb), (tw, tb) in zip(d, ref, theta):
            for got, want, t in ((dw, rw, tw), (db, rb, tb)):
                tol = 1e-2 * np.linalg.norm(want) + 2.0 ** -22 * np.linalg.norm(t)
                assert np.linalg.norm(got.astype(np.float64) - want) <= tol, k
    g.close()


def test_infinities_and_largest_values_stay_what_they_are():
    """An infinite weight makes infinities, not NaN, where the float32 product
    has them; a value that rounds to infinity in bf16 still gives its finite
    product."""
    import torch

    import paper_1710_02368_amd as agn
    dims = (20, 40, 36, 6)
    wl = W.small_workload("inf", dims, 2, 1, 8, 0.05, 1, 70)
    X, y = W.make_data(wl)
    vec = W.random_params(dims, 7)
    p = unflat_params(vec, dims)
    p[0][0][3, 5] = np.inf
    big = X.copy()
    big[:, 9] = 3.395e38       # above the largest bf16 value
    q = unflat_params(vec, dims)
    q[0][0][:, 9] *= 1e-36     # (products of about 100, weights no subnormals)
    for what, params, data in (("inf", p, X), ("big", q, big)):
        flat = np.concatenate([np.concatenate([w.ravel(), b.ravel()]) for w, b in params])
        g = agn.AGN(dims, 2, 1, 0.05, 8, seed=1)
        g.set_central(torch.from_numpy(flat).cuda())
        xd, yd = to_device(data, y)
        _, rl, rp = g.evaluate(xd, yd, row_outputs=True)
        with np.errstate(invalid="ignore"):
            row_loss, pred, logits = evaluate(params, data, y)
        rl, rp = rl.cpu().numpy(), rp.cpu().numpy()
        np.testing.assert_array_equal(rp, pred, err_msg=what)
        np.testing.assert_array_equal(np.isfinite(rl), np.isfinite(row_loss))
        ok = np.isfinite(row_loss)
        np.testing.assert_allclose(rl[ok], row_loss[ok], rtol=1e-4, atol=1e-5)
        g.close()


@pytest.mark.parametrize("rows,width", [(70, 40), (7000, 70), (16300, 70), (16300, 200)],
                         ids=["small", "deep", "flat", "mid"])
def test_infinity_beside_nan(rows, width):
    """A unit whose weights are all NaN (its results are NaN whichever way they
    are computed) beside one with an infinite weight, which has to stay an
    infinity where its input is positive, and beside a unit with a single NaN
    between the places that are looked at."""
    import torch

    import paper_1710_02368_amd as agn
    dims = (20, width, 36, 6)
    print(rows, dims, flush=True)
    rng = np.random.default_rng(3)
    X, y = rng.standard_normal((rows, 20)).astype(np.float32), rng.integers(0, 6, rows).astype(np.int32)
    p = unflat_params(W.random_params(dims, 7), dims)
    p[0][0][3] = np.nan
    p[0][0][7, 14] = np.nan
    p[0][0][5, 2] = np.inf
    g = agn.AGN(dims, 2, 1, 0.05, 8, seed=1)
    flat = np.concatenate([np.concatenate([w.ravel(), b.ravel()]) for w, b in p])
    g.set_central(torch.from_numpy(flat).cuda())
    _, rl, _ = g.evaluate(*to_device(X, y), row_outputs=True)
    g.close()
    h = X.astype(np.float64)
    with np.errstate(invalid="ignore"):
        for l, (w, b) in enumerate(p):
            h = _product(h, w) + b
            if l < 2:
                h = np.where(h > 0, h, 0.0)
        lse = h.max(axis=1) + np.log(np.exp(h - h.max(axis=1, keepdims=True)).sum(axis=1))
        want = lse - h[np.arange(rows), y]
    rl = rl.cpu().numpy()
    ok = X[:, 2] < 0  # (minus infinity before the rectifier)
    assert not np.any(np.isfinite(rl[~ok])) and not np.any(np.isfinite(want[~ok]))
    np.testing.assert_allclose(rl[ok], want[ok], rtol=1e-4, atol=1e-5)


def _product(h, w):
    """h w^T in 64 bits with infinities as IEEE has them (a blocked library
    product may differ: inf * 0 in its padding)."""
    return np.concatenate([(h[r:r + 256, None, :] * w.astype(np.float64)[None]).sum(axis=2)
                           for r in range(0, len(h), 256)])


def test_a_model_of_nan_keeps_its_speed():
    """Tiles of NaN weights are not computed twice (2.5 times the round when
    they were)."""
    import time

    import torch

    import paper_1710_02368_amd as agn
    dims, n, m, rows = (784, 1000, 1000, 10), 8, 128, 8 * 1920
    x = torch.rand(rows, 784, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    y = torch.zeros(rows, dtype=torch.int32, device="cuda")
    took = {}
    for what in ("finite", "nan"):
        g = agn.AGN(dims, n, 15, 0.001, m, seed=1)
        if what == "nan":
            g.set_central(torch.full((g.P,), float("nan"), device="cuda"))
        times = []
        for i in range(12):
            t = time.perf_counter()
            g.round(x, y, list(range(n)))
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t)
        took[what] = float(np.median(times[2:]))
        g.close()
    print(took, flush=True)
    assert took["nan"] <= 1.6 * took["finite"], took
