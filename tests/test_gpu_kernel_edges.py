"""Kernel variants at the sizes where their dispatch or their tiles change,
against the FP64 oracle or, where the order of the arithmetic is part of the
contract, bit for bit against the other variant."""
import numpy as np
import pytest

import cases
import oracle as O
from gpu_common import PARAMS, announce, need_gpu, planner

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


def _case(n_cath, n_dwell, M, seed=5):
    return cases.make_case(n_cath, n_dwell, (M - 3 * (M // 5), M // 5, M // 5, M // 5), seed=seed)


# Sums over the split partials of an evaluation: one wavefront up to 48 splits,
# eight in chunks of 128 splits above.  FP32 bounds of the evaluation: 2e-5 on
# F, 2e-4 of the gradient's scale.
@pytest.mark.parametrize("M,splits", [(4096, (1, 15, 16, 17, 47, 48, 49, 127, 128, 129, 256)), (32, (1, 2))])
@pytest.mark.parametrize("P,n_cath,n_dw", [(3, 5, 7), (65, 8, 16)])
def test_evaluation_sums_every_split(M, splits, P, n_cath, n_dw):
    announce(f"evaluate split sums M={M} P={P} K={n_cath * n_dw}")
    c = _case(n_cath, n_dw, M)
    D = O.dose_rate_matrix(c.dwell_xyz, c.pt_xyz)
    W = cases.hidden_weights(P, seed=P)
    x = np.sqrt(O.uniform_start_time(D, c.group, 15.0)) * (0.2 + 1.6 * cases.uniform_draws((P, c.K), seed=7))
    Fr, gr = O.objective_and_gradient_x(D, x, c.group, PARAMS, W)
    pl = planner(c, W)
    cap = pl.tuning()["split"]
    for s in splits:
        if s > max(cap, min(32, (M + 31) // 32 * 2)):
            continue
        pl.set_split(s)
        F, g = pl.evaluate(x)
        assert np.max(np.abs(F - Fr) / Fr) <= 2e-5, s
        assert np.abs(g - gr).max() <= 2e-4 * np.abs(gr).max(), s


# The update kernel sums the split partials with seven wavefronts in batches of
# at most 256 plan slots and with one above; both in split order, so the same
# plans in a small and in a large context give the same bits.  Sizes: one and
# two float4 columns per lane, splits at and past a chunk of 56 (512 padded
# dwells), short and full histories.
@pytest.mark.parametrize("n_cath,n_dw,M,m", [(5, 6, 64, 4), (16, 10, 2400, 10), (20, 25, 896, 10),
                                             (20, 25, 928, 4), (20, 25, 1824, 10), (18, 20, 4096, 10)])
def test_update_forms_agree_bitwise(n_cath, n_dw, M, m):
    announce(f"update forms K={n_cath * n_dw} M={M} m={m}")
    c = _case(n_cath, n_dw, M)
    W = cases.hidden_weights(3, seed=6)
    out = []
    for cap in (3, 300):
        pl = planner(c, W, max_plans=cap, history=m)
        pl.optimize(max_iter=15)
        out.append((pl.weights_x(), pl.metrics()["F_run"], pl.metrics()["evaluations"]))
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


# At most 16 plans in a workgroup take the form that shares a chunk of three
# (FP32) or two (FP64-accumulated) point blocks among all waves; the chains and
# the order of every sum are those of the form for more plans, so the same plans
# alone and among others give the same bits.  Sizes: one dwell slice and more
# than eight, ranges of one block, of whole chunks and of a remainder, batches
# that fill the group, leave it ragged, and end in a second tile of few plans.
@pytest.mark.parametrize("n_cath,n_dw,M", [(1, 5, 15), (3, 11, 75), (5, 13, 160), (18, 20, 1005), (20, 20, 4096),
                                           (20, 25, 333)])
@pytest.mark.parametrize("dtype", ["f32", "f32acc64"])
def test_few_plans_agree_bitwise(n_cath, n_dw, M, dtype):
    announce(f"few plans K={n_cath * n_dw} M={M} {dtype}")
    c = _case(n_cath, n_dw, M)
    D = O.dose_rate_matrix(c.dwell_xyz, c.pt_xyz)
    W = cases.hidden_weights(64, seed=6)
    x = np.sqrt(O.uniform_start_time(D, c.group, 15.0)) * (0.2 + 1.6 * cases.uniform_draws((64, c.K), seed=7))
    x[2] = 0.0
    full = planner(c, W, dtype=dtype)
    alone = [(P, planner(c, np.concatenate([np.tile(W[:1], (P // 64 * 64, 1)), W[:P % 64]]), dtype=dtype))
             for P in (1, 5, 16, 17, 67)]
    for s in (1, 2, 3, (M + 15) // 16 // 2):
        if s < 1 or s > min(32, (M + 31) // 32 * 2):
            continue
        full.set_split(s)
        F, g = full.evaluate(x)
        for P, pl in alone:
            pl.set_split(s)
            Fp, gp = pl.evaluate(np.concatenate([x] * (P // 64) + [x[:P % 64]]))
            np.testing.assert_array_equal(Fp[P // 64 * 64:], F[:P % 64])
            np.testing.assert_array_equal(gp[P // 64 * 64:], g[:P % 64])


# The set-up kernel takes 32 rows and 64 columns at a time; the row sums of the
# start time start and end inside a block of rows when the target does not
# come first.  Tolerances: the matrix within 8 FP64 roundings of the oracle's,
# the start time within 1e-13; the run-precision copies bit for bit.
@pytest.mark.parametrize("n_cath,n_dw,M", [(1, 1, 15), (3, 11, 75), (5, 13, 160), (8, 12, 1005), (20, 25, 333)])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
def test_dose_setup_edges(n_cath, n_dw, M, dtype):
    import torch
    announce(f"dose set-up K={n_cath * n_dw} M={M} {dtype}")
    c = _case(n_cath, n_dw, M)
    target = 2 if M > 100 else 0
    D = O.dose_rate_matrix(c.dwell_xyz, c.pt_xyz)
    from paper_1904_01567_amd import Planner
    pl = Planner(dtype=dtype, max_plans=2)
    pl.load(c, PARAMS, target_group=target)
    Dg = pl.dose_rate()
    np.testing.assert_allclose(Dg, D, rtol=4e-16 * 8, atol=0)
    tb = 15.0 / Dg[c.group == target].sum(axis=1).mean()
    assert pl.start_time() == pytest.approx(tb, rel=1e-13)
    D32 = Dg.astype(np.float32)
    if dtype == "f32":
        ref = D32.astype(np.float64)
    elif dtype == "bf16":
        ref = torch.tensor(D32).to(torch.bfloat16).double().numpy()
    else:
        s = (Dg.max(axis=0) / 224.0).astype(np.float32)
        ref = torch.tensor(D32 / s[None, :]).to(torch.float8_e4m3fn).double().numpy() * s[None, :].astype(np.float64)
    np.testing.assert_array_equal(pl.dose_rate(run_dtype=True), ref)
    # the dwell-major copy feeds the back-projection: the gradient of one plan
    x = np.full((1, c.K), np.sqrt(tb)) * (0.3 + cases.uniform_draws((1, c.K), seed=9))
    W = cases.hidden_weights(1, seed=3)
    pl.set_weights(W)
    _, g = pl.evaluate(x)
    _, gr = O.objective_and_gradient_x(D, x, c.group, PARAMS, W)
    tol = {"f32": 2e-4, "bf16": 5e-2, "fp8": 0.25}[dtype]
    assert np.abs(g - gr).max() <= tol * np.abs(gr).max()


# The network's products at the edges of their tiles (32 x 32, slices of 64)
# and past six layers (the weight gradients of one launch).  BF16 operands in
# every product: the tolerances of the network's own parity test.
@pytest.mark.parametrize("sizes,B", [([1, 1], 1), ([33, 65, 31], 33), ([64, 32, 64], 128), ([68, 40, 277], 129),
                                     ([9, 8, 8, 8, 8, 8, 8, 8, 5], 70)])
def test_network_products_at_tile_edges(sizes, B):
    from oracle import mlp_oracle as MO
    from paper_1904_01567_amd import Network
    announce(f"network {sizes} B={B}")
    rng = np.random.default_rng(B)
    p = cases.mlp_init(sizes, seed=1).astype(np.float32)
    X = rng.uniform(0, 1, size=(B + 7, sizes[0])).astype(np.float32)
    Y = rng.uniform(0, 2, size=(B + 7, sizes[-1])).astype(np.float32)
    order = rng.permutation(B + 7)[:B].astype(np.int32)
    net = Network(sizes, max_batch=B)
    net.set_params(p)
    L, g = net.loss_grad(X[order], Y[order])
    Lr, gr = MO.loss_and_grad(p.astype(np.float64), sizes, X[order].astype(np.float64), Y[order].astype(np.float64))
    assert L == pytest.approx(Lr, rel=2e-2)
    assert np.abs(g - gr).max() <= 5e-2 * np.abs(gr).max()
    # rows gathered by index, and the same rows laid out in order: the same step
    got = []
    for Xd, Yd, o in ((X, Y, order), (X[order], Y[order], np.arange(B, dtype=np.int32))):
        net.set_params(p)
        net.set_data(Xd, Yd)
        loss = net.train(np.concatenate([o, o]), B, 1e-3)
        got.append((loss, net.params()))
    assert got[0][0] == got[1][0]
    np.testing.assert_array_equal(got[0][1], got[1][1])
    assert np.abs(got[0][1] - p).max() > 1e-4


def test_network_tile_sizes_agree_bitwise():
    # 64 x 64 tiles from 512 of them (2,048 rows x 1,100 columns), 32 x 32 below
    from paper_1904_01567_amd import Network
    announce("network tile sizes")
    sizes = [70, 1100, 1030]
    rng = np.random.default_rng(3)
    p = cases.mlp_init(sizes, seed=2).astype(np.float32)
    X = rng.uniform(0, 1, size=(2048, 70)).astype(np.float32)
    out = []
    for mb in (2048, 100):
        net = Network(sizes, max_batch=mb)
        net.set_params(p)
        out.append(net.predict(X))
    np.testing.assert_array_equal(out[0], out[1])
    Y = rng.uniform(0, 2, size=(2048, 1030)).astype(np.float32)
    net = Network(sizes, max_batch=2048)
    net.set_params(p)
    L, g = net.loss_grad(X, Y)
    from oracle import mlp_oracle as MO
    Lr, gr = MO.loss_and_grad(p.astype(np.float64), sizes, X.astype(np.float64), Y.astype(np.float64))
    assert L == pytest.approx(Lr, rel=2e-2)
    assert np.abs(g - gr).max() <= 5e-2 * np.abs(gr).max()


# Rows of whole, aligned float4 are read 16 bytes at a time, others by element.
# A network of 67 inputs and the same one with a 68th that is always zero take
# different forms of the first forward product: the same bits.
@pytest.mark.parametrize("hidden,B", [(32, 33), (64, 130)])
def test_network_row_loads_agree_bitwise(hidden, B):
    from paper_1904_01567_amd import Network
    announce(f"network row loads hidden={hidden} B={B}")
    rng = np.random.default_rng(B)
    narrow, wide = [67, hidden, 8], [68, hidden, 8]
    p = cases.mlp_init(narrow, seed=2).astype(np.float32)
    W0 = p[:67 * hidden].reshape(hidden, 67)
    q = np.concatenate([np.pad(W0, ((0, 0), (0, 1))).ravel(), p[67 * hidden:]])
    X = rng.uniform(0, 1, size=(B, 67)).astype(np.float32)
    Y = rng.uniform(0, 2, size=(B, 8)).astype(np.float32)
    out = []
    for sizes, par, x in ((narrow, p, X), (wide, q, np.pad(X, ((0, 0), (0, 1))))):
        net = Network(sizes, max_batch=B)
        net.set_params(par)
        L, g = net.loss_grad(x, Y)
        gW = g[:sizes[0] * hidden].reshape(hidden, sizes[0])
        out.append((np.float64(L), net.predict(x), gW[:, :67], g[sizes[0] * hidden:]))
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


def _check_metrics(pl, D, t, c, W, params=PARAMS):
    m = pl.metrics()
    mref = O.plan_metrics(D, t, c.group, params, W, c.volume_cc, 15.0)
    for p, q in enumerate(mref):
        assert m["F64"][p] == pytest.approx(q["F"], rel=1e-12, abs=1e-300)
        np.testing.assert_allclose(m["f_organ"][p], q["f_organ"], rtol=1e-12, atol=1e-300)
        np.testing.assert_array_equal(m["V100_pct"][p], q["V100_pct"])
        np.testing.assert_array_equal(m["V75_cc"][p], q["V75_cc"])
        np.testing.assert_allclose(m["D10_pct"][p], q["D10_pct"], rtol=1e-13)
        np.testing.assert_allclose(m["D90_pct"][p], q["D90_pct"], rtol=1e-13)
    best, cls, nd, frac = pl.select_plan()
    np.testing.assert_array_equal(cls, [O.plan_class(q) for q in mref])
    np.testing.assert_array_equal(nd, O.nondominated(np.array([q["f_organ"] for q in mref])))
    assert best == O.select_plan(mref)
    assert frac == pytest.approx(nd.mean())


# FP64 doses in tiles of 16, 32 and 64 plans and steps of 16 dwells; the
# tolerances of the metrics' parity test (FP64 sums in another order).
@pytest.mark.parametrize("P", [1, 16, 17, 32, 33, 64, 65])
@pytest.mark.parametrize("n_cath,n_dw,M", [(1, 5, 40), (3, 16, 129), (5, 7, 1007)])
def test_metrics_tile_edges(P, n_cath, n_dw, M):
    announce(f"metrics P={P} K={n_cath * n_dw} M={M}")
    c = _case(n_cath, n_dw, M)
    D = O.dose_rate_matrix(c.dwell_xyz, c.pt_xyz)
    W = cases.hidden_weights(P, seed=P)
    t0 = O.uniform_start_time(D, c.group, 15.0) * (0.1 + 1.9 * cases.uniform_draws((P, c.K), seed=303))
    pl = planner(c, W, t0=t0)
    x = np.sqrt(t0).astype(np.float32).astype(np.float64)
    _check_metrics(pl, D, x * x, c, W)


# D10 / D90 by histogram and ranking; bins of more than 1,024 doses by the
# radix select: an organ of equal doses, one of two values around the rank, and
# doses far outside the histogram's 2^-4 .. 2^12 Gy, where its end bins hold all.
@pytest.mark.parametrize("scale", [1.0, 1e-6, 1e6])
def test_metrics_of_equal_and_extreme_doses(scale):
    announce(f"metrics of equal doses x {scale}")
    from paper_1904_01567_amd import Planner
    c = _case(3, 5, 10000)
    rng = np.random.default_rng(8)
    D = np.empty((c.M, c.K))
    D[c.group == 0] = 1.0                                            # one dose
    two = rng.uniform(size=(c.group == 1).sum()) < 0.1               # two doses
    D[c.group == 1] = np.where(two, 2.0, 1.0)[:, None]
    D[c.group >= 2] = rng.uniform(0.5, 2.0, size=((c.group >= 2).sum(), 1))
    D *= scale
    W = cases.hidden_weights(3, seed=2)
    t0 = np.full((3, c.K), 1.0) * np.array([[1.0], [4.0], [0.25]])   # exact square roots
    pl = Planner(max_plans=3)
    pl.load_case(c.dwell_xyz, None, c.group, PARAMS, c.volume_cc, 15.0, 0, dose_rate=D)
    pl.set_weights(W, t0)
    _check_metrics(pl, D, t0, c, W)


# The test for finite values runs on blocks of 2,048; every place counts, and
# the largest finite FP64 values pass it (they overflow FP32, so the objective
# does not stay finite).
def test_nonfinite_inputs_are_refused_at_every_place():
    from paper_1904_01567_amd import GmcoError
    announce("non-finite inputs")
    c = cases.make_case(8, 16, (40, 10, 15, 15), seed=4)  # 128 dwells
    W = cases.hidden_weights(40, seed=1)
    pl = planner(c, W)
    x = np.full((40, c.K), 0.1)
    F0, g0 = pl.evaluate(x)
    for at in (0, 2047, 2048, 4095, 40 * c.K - 1):
        for bad in (np.inf, -np.inf, np.nan):
            y = x.copy()
            y.reshape(-1)[at] = bad
            with pytest.raises(GmcoError) as e:
                pl.evaluate(y)
            assert e.value.code == -1 and "finite" in str(e.value)
    y = x.copy()
    y[3, 5] = -np.finfo(np.float64).max
    y[4, 6] = np.finfo(np.float64).tiny / 8
    F1, _ = pl.evaluate(y)
    keep = np.arange(40) != 3
    assert not np.isfinite(F1[3]) and np.all(np.isfinite(F1[keep]))
    F2, g2 = pl.evaluate(x)  # a refused call leaves nothing behind
    np.testing.assert_array_equal(F2, F0)
    np.testing.assert_array_equal(g2, g0)
