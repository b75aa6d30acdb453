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
