"""The order in which the scorer's kernels add: the sums of what a call stores,
taken on the host in FP32 in the stated order, bit for bit."""
import numpy as np
import pytest
import torch

from synth import weights as W
from tests.test_gpu_mlp_shapes import _case, _dev, _empty, _prepared, ctx  # noqa: F401
from tests.test_sum_orders import logit_sum

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 16, 17, 1000, 40001])
def test_logits_add_in_order(ctx, n):    # noqa: F811
    """terms h2 w3 of the stored second layer"""
    print(f"case logit sum n={n}", flush=True)
    f, mean, istd, P, _ = _case(n, n + 11)
    x = _prepared(ctx, f, mean, istd)
    lg, h1, h2 = _empty(n, torch.float32), _empty((n, 64), torch.int16), _empty((n, 64), torch.float32)
    ctx.mlp_forward(_dev(P), x, lg, h1, h2)
    terms = h2.cpu().numpy() * P[-65:-1]
    want = logit_sum(terms) + P[-1]
    assert np.array_equal(lg.cpu().numpy().view(np.uint32), want.view(np.uint32))
