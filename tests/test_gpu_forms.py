"""Forms of one kernel that only some batch sizes or layer widths reach, bit for
bit against the form that the others take."""
import numpy as np
import pytest

import cases
import oracle as O
from gpu_common import announce, need_gpu, planner

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _case(n_cath, n_dwell, M, seed=5):
    return cases.make_case(n_cath, n_dwell, (M - 3 * (M // 5), M // 5, M // 5, M // 5), seed=seed)


def _result(pl):
    m = pl.metrics()
    return [pl.weights_x(), m["F_run"], m["evaluations"], m["iterations"], m["status"]]


# A batch of at most 256 plans has the split partials summed by seven wavefronts,
# in chunks of 28,672 / (padded dwells) splits; grouped launches use one wavefront
# for any batch.  Sizes: one and two float4 columns per lane, 512 padded dwells
# with 56 splits (one whole chunk), 58 and 114 (a second and a third chunk), both
# history capacities.
@pytest.mark.parametrize("n_cath,n_dw,M,m", [(5, 6, 64, 4), (16, 10, 2400, 10), (20, 25, 896, 10),
                                             (20, 25, 928, 4), (20, 25, 1824, 10), (18, 20, 4096, 4)])
def test_wide_update_agrees_with_grouped_bitwise(n_cath, n_dw, M, m):
    from paper_1904_01567_amd import optimize_many
    announce(f"wide update K={n_cath * n_dw} M={M} m={m}")
    c = _case(n_cath, n_dw, M)
    W = cases.hidden_weights(3, seed=6)
    alone = planner(c, W, history=m)
    alone.optimize(max_iter=15)
    pair = [planner(c, W, history=m) for _ in range(2)]
    optimize_many(pair, max_iter=15)
    for pl in pair:
        for a, b in zip(_result(alone), _result(pl)):
            np.testing.assert_array_equal(a, b)


# The same against the one-wavefront form of a batch of its own: 300 copies of a
# plan advance together, so every round keeps its five plan tiles and the split
# set for them.  85 splits at 384 padded dwells are a chunk of 74 and a remainder.
@pytest.mark.parametrize("n_cath,n_dw,M,m,split", [(5, 6, 64, 4, 4), (18, 20, 1005, 4, 32), (18, 20, 5440, 10, 85)])
def test_wide_update_agrees_with_large_batch_bitwise(n_cath, n_dw, M, m, split):
    announce(f"wide update against 300 plans K={n_cath * n_dw} M={M} m={m} split={split}")
    c = _case(n_cath, n_dw, M)
    W = cases.hidden_weights(2, seed=6)
    for w in W:
        out = []
        for P in (1, 300):
            pl = planner(c, np.tile(w, (P, 1)), history=m)
            pl.set_split(split)
            pl.optimize(max_iter=12)
            out.append(_result(pl))
        for a, b in zip(*out):
            np.testing.assert_array_equal(np.broadcast_to(a, b.shape), b)


# Weight gradients take 64 x 64 tiles from 512 of them (1,536 x 1,500: 24 x 24)
# and 32 x 32 below.  The first 96 outputs alone are 48 tiles, and their gradient
# is 16 times as large (the mean is over a sixteenth of the outputs), a scaling
# that no rounding sees.
@pytest.mark.parametrize("B", [5, 64, 200])
def test_weight_gradient_tiles_agree_bitwise(B):
    from oracle import mlp_oracle as MO
    from paper_1904_01567_amd import Network
    announce(f"weight gradient tiles B={B}")
    n_in, n_out, part = 1500, 1536, 96
    rng = np.random.default_rng(B)
    p = cases.mlp_init([n_in, n_out], seed=1).astype(np.float32)
    X = rng.uniform(0, 1, size=(B, n_in)).astype(np.float32)
    Y = rng.uniform(0, 2, size=(B, n_out)).astype(np.float32)
    net = Network([n_in, n_out], max_batch=B)
    net.set_params(p)
    L, g = net.loss_grad(X, Y)
    gW, gb = g[:n_in * n_out].reshape(n_out, n_in), g[n_in * n_out:]
    Lr, gr = MO.loss_and_grad(p.astype(np.float64), [n_in, n_out], X.astype(np.float64), Y.astype(np.float64))
    assert L == pytest.approx(Lr, rel=2e-2)
    assert np.abs(g - gr).max() <= 5e-2 * np.abs(gr).max()
    W = p[:n_in * n_out].reshape(n_out, n_in)
    small = Network([n_in, part], max_batch=B)
    small.set_params(np.concatenate([W[:part].ravel(), p[n_in * n_out:][:part]]))
    _, h = small.loss_grad(X, np.ascontiguousarray(Y[:, :part]))
    np.testing.assert_array_equal(h[:n_in * part].reshape(part, n_in), np.float32(n_out / part) * gW[:part])
    np.testing.assert_array_equal(h[n_in * part:], np.float32(n_out / part) * gb[:part])
    # the form that updates the parameters in place of storing the gradient: the
    # first Adam step from this gradient, within a few FP32 roundings
    net.set_data(X, Y)
    lr = 1e-3
    net.train(np.arange(B, dtype=np.int32), B, lr)
    m = np.float32(0.1) * g
    v = g * (np.float32(0.001) * g)
    step = lr * (m.astype(np.float64) / 0.1) / (np.sqrt(v.astype(np.float64) / 0.001) + 1e-8)
    # (the first step's moments and their corrections have the same factors)
    assert np.abs(net.params() - (p - step)).max() <= 2.0 ** -23 * np.abs(p).max() + 2e-6 * lr
    assert np.abs(net.params() - p).max() > 0.5 * lr


# A range of more than 65,536 point blocks in one workgroup (a million points and
# one split, as batches of thousands of plans have): the form for few plans walks
# it in chunks whose places were once computed in 32 bits past their range.
@pytest.mark.parametrize("dtype", ["f32", "f32acc64"])
def test_few_plans_over_a_long_range(dtype):
    M = 1_300_000
    announce(f"few plans over {M} points in one split, {dtype}")
    c = _case(1, 5, M)
    W = cases.hidden_weights(64, seed=6)
    x = 0.5 + cases.uniform_draws((64, c.K), seed=7)
    out = []
    for P in (64, 1):
        pl = planner(c, W[:P], dtype=dtype)
        pl.set_split(1)
        out.append(pl.evaluate(x[:P]))
        pl.close()
    (F, g), (F1, g1) = out
    np.testing.assert_array_equal(F1, F[:1])
    np.testing.assert_array_equal(g1, g[:1])
    assert np.all(np.isfinite(F)) and np.all(F > 0.0)
