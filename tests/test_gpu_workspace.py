"""Training with a workspace of 64 row chunks, 4 (n + 64 x parameters) bytes:
accepted for every n, nothing written past it, gradients within the FP64
oracle's bound, and a fused step equal to the separate calls bit for bit."""
import numpy as np
import pytest
import torch

from oracle import mlp as M
from synth import weights as W
from tests.test_gpu_mlp_shapes import _case, _dev, _empty, _prepared, ctx  # noqa: F401

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
GUARD = 4096


@pytest.mark.parametrize("n", [1, 64, 4096, 4097, 5000, 8192, 8193, 20001])
def test_workspace_of_64_chunks(ctx, n):    # noqa: F811
    import paper_2209_13711_amd as lst
    print(f"case workspace n={n}", flush=True)
    f, mean, istd, P, y = _case(n, n + 3)
    x, yd = _prepared(ctx, f, mean, istd), _dev(y.astype(np.uint8))
    lg, h1, h2 = _empty(n, torch.float32), _empty((n, 64), torch.int16), _empty((n, 64), torch.float32)
    least = 4 * (n + 64 * W.N_PARAM)
    whole = torch.full((least + GUARD,), 0x5a, dtype=torch.uint8, device=DEV)
    work = whole[:least]
    p, g, m, v = _dev(P), _dev(P * 0), _dev(P * 0), _dev(P * 0)
    loss = _empty(1, torch.float32)
    ctx.mlp_forward(p, x, lg, h1, h2)
    ctx.mlp_backward(p, x, yd, lg, h1, h2, work, g, loss)
    loss_ref, g_ref = M.loss_and_grad(P, M.standardise(f, mean, istd), y)
    assert float(loss[0]) == pytest.approx(loss_ref, rel=1e-5, abs=1e-6)
    got, o = g.cpu().numpy().astype(np.float64), 0
    for name, shape in M.SIZES:
        k = int(np.prod(shape))
        assert np.linalg.norm(got[o:o + k] - g_ref[o:o + k]) <= 1e-3 * np.linalg.norm(g_ref[o:o + k]) + 1e-9, name
        o += k
    p2, g2, m2, v2 = _dev(P), _dev(P * 0), _dev(P * 0), _dev(P * 0)
    loss2 = _empty(1, torch.float32)
    ctx.mlp_adam(p, g, m, v, 1, 1e-3)
    ctx.mlp_train_steps(p2, x, yd, n, [0], 0, lg, h1, h2, work, g2, m2, v2, loss2, 1e-3)
    for a, b in ((p, p2), (g, g2), (m, m2), (v, v2), (loss, loss2)):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    assert bool((whole[least:] == 0x5a).all())
    # up to 4096 rows it is the whole workspace; a byte less is refused
    if n <= 4096:
        assert ctx.mlp_workspace_bytes(n) == least
    for call in (lambda: ctx.mlp_backward(p, x, yd, lg, h1, h2, work[:-1], g, loss),
                 lambda: ctx.mlp_train_steps(p2, x, yd, n, [0], 0, lg, h1, h2, work[:-1], g2, m2, v2,
                                             loss2, 1e-3)):
        with pytest.raises(lst.LSTError) as ei:
            call()
        assert ei.value.code == lst.LST_E_CAPACITY
