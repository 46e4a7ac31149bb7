"""The order in which the scorer's kernels add: the sums of what a call stores,
taken on the host in FP32 in the stated order, bit for bit."""
import numpy as np
import pytest
import torch

from synth import weights as W
from tests.test_gpu_mlp_shapes import _case, _dev, _empty, _prepared, ctx  # noqa: F401
from tests.test_sum_orders import chunk_sum, logit_sum

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


@pytest.mark.parametrize("few", [False, True])
@pytest.mark.parametrize("n", [1, 64, 65, 4096, 4097, 8192, 8193, 20001])
def test_gradients_add_the_chunks(ctx, n, few):    # noqa: F811
    """the chunks' partial gradients as the workspace holds them after the call"""
    print(f"case chunk sum n={n} few={few}", flush=True)
    f, mean, istd, P, y = _case(n, n + 12)
    x, p = _prepared(ctx, f, mean, istd), _dev(P)
    lg, h1, h2 = _empty(n, torch.float32), _empty((n, 64), torch.int16), _empty((n, 64), torch.float32)
    size = 4 * (n + 64 * W.N_PARAM) if few else ctx.mlp_workspace_bytes(n)
    work, g, loss = _empty(size, torch.uint8), _empty(W.N_PARAM, torch.float32), _empty(1, torch.float32)
    ctx.mlp_forward(p, x, lg, h1, h2)
    ctx.mlp_backward(p, x, _dev(y.astype(np.uint8)), lg, h1, h2, work, g, loss)
    most = (size // 4 - n) // W.N_PARAM
    batches = -(-n // 64)
    chunks = -(-batches // -(-batches // most))
    parts = work.view(torch.float32)[n:n + chunks * W.N_PARAM].cpu().numpy().reshape(chunks, -1)
    want = chunk_sum(np.ascontiguousarray(parts.T))
    assert np.array_equal(g.cpu().numpy().view(np.uint32), want.view(np.uint32))
