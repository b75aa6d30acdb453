"""Device memory that calls hold after they return."""
import numpy as np
import pytest

import cases
from gpu_common import announce, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    need_gpu()


# The order of a training call goes to the device whole: 64 MiB here.  A network
# keeps at most 16 MiB of it for the next call.
def test_long_training_call_gives_its_order_back():
    import torch
    from paper_1904_01567_amd import Network
    announce("training order of 64 MiB")
    B, steps = 16384, 1024
    net = Network([1, 1], max_batch=B)
    net.set_params(cases.mlp_init([1, 1], seed=1).astype(np.float32))
    r = np.random.default_rng(3)
    X = r.uniform(0, 1, size=(64, 1)).astype(np.float32)
    net.set_data(X, 2 * X + 1)
    order = r.integers(0, 64, size=steps * B).astype(np.int32)
    first = net.train(order[:B], B, 1e-2)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    loss = net.train(order, B, 1e-2)
    assert free - torch.cuda.mem_get_info()[0] <= 16 << 20
    assert loss < first
    again = net.train(order[:B], B, 1e-2)  # (a short call after it allocates anew)
    assert again < loss
