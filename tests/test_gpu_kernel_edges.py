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
