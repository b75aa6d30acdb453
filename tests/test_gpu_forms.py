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
