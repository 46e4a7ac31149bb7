"""Scorer training and scoring calls at the sizes where their kernels change:
one chunk per 64 rows up to 128 chunks, then several batches per chunk; tiles
of 16 rows per wave beyond the grid; arrays whose alignment rules out wide
loads and stores.  References as in the scorer tests: the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import mlp as M
from synth import geometry as G
from synth import params as PR
from synth import weights as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def ctx():
    import paper_2209_13711_amd as lst
    geo = G.get("barrel_toy")
    return lst.Context(PR.make(), geo.f32, geo.i32, device=0)


def _case(n, seed):
    rng = np.random.default_rng(seed)
    f = rng.normal(0, 1, (n, 40)).astype(np.float32)
    mean, istd = np.zeros(40, np.float32), np.ones(40, np.float32)
    P = W.random_params(rng, bias=0.2)
    return f, mean, istd, P, rng.integers(0, 2, n)


def _dev(a, shift=0):
    """on the device, `shift` elements past an aligned address"""
    t = torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    if not shift:
        return t
    out = torch.empty(t.numel() + shift, dtype=t.dtype, device=DEV)[shift:].reshape(t.shape)
    out.copy_(t)
    return out


def _empty(shape, dtype, shift=0):
    return torch.empty(int(np.prod(shape)) + shift, dtype=dtype, device=DEV)[shift:].reshape(shape)


def _prepared(ctx, f, mean, istd, shift=0):
    x = torch.empty((len(f), 64), dtype=torch.int16, device=DEV)
    ctx.mlp_prepare(_dev(f, shift), _dev(mean, shift), _dev(istd, shift), x)
    return x


@pytest.mark.parametrize("n", [63, 65, 4097, 8192, 8193, 20001])
def test_gradient_chunks(ctx, n):
    """gradients within the FP64 bound, and one fused training step equals the
    separate calls bit for bit"""
    print(f"case gradient chunks n={n}", flush=True)
    f, mean, istd, P, y = _case(n, n)
    x, yd = _prepared(ctx, f, mean, istd), _dev(y.astype(np.uint8))
    lg, h1, h2 = (_empty(n, torch.float32), _empty((n, 64), torch.int16), _empty((n, 64), torch.float32))
    work = _empty(ctx.mlp_workspace_bytes(n), torch.uint8)
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


@pytest.mark.parametrize("n", [1, 15, 17, 64, 65, 40000])
def test_forward_tiles(ctx, n):
    """logits within the oracle's bound, with and without saved layers, the
    saved layers those of the logits"""
    print(f"case forward tiles n={n}", flush=True)
    f, mean, istd, P, _ = _case(n, 7 * n + 1)
    x, p = _prepared(ctx, f, mean, istd), _dev(P)
    lg, only = _empty(n, torch.float32), _empty(n, torch.float32)
    h1, h2 = _empty((n, 64), torch.int16), _empty((n, 64), torch.float32)
    ctx.mlp_forward(p, x, lg, h1, h2)
    ctx.mlp_forward(p, x, only)
    assert torch.equal(lg.view(torch.int32), only.view(torch.int32))
    ref, bound = M.forward(P, M.standardise(f, mean, istd))
    got = lg.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= bound)
    w3, b3 = P[-65:-1].astype(np.float64), float(P[-1])
    h = h2.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(h @ w3 + b3 - got) <= 1e-5 * (np.abs(h) @ np.abs(w3) + abs(b3)))
    assert ((h1.cpu().numpy().view(np.uint16) & 0x8000) == 0).all() and (h >= 0).all()


@pytest.mark.parametrize("n", [1, 3, 4097])
def test_unaligned_arrays(ctx, n):
    """the same bits from arrays one element past an aligned address"""
    print(f"case unaligned n={n}", flush=True)
    f, mean, istd, P, y = _case(n, n + 5)
    x, xs = _prepared(ctx, f, mean, istd), _prepared(ctx, f, mean, istd, shift=1)
    assert torch.equal(x, xs)
    out = []
    for sh in (0, 1):
        p = _dev(P, sh)
        lg, g, loss = _empty(n, torch.float32, sh), _empty(W.N_PARAM, torch.float32, sh), _empty(1, torch.float32)
        h1, h2 = _empty((n, 64), torch.int16, 4 * sh), _empty((n, 64), torch.float32, sh)
        ctx.mlp_forward(p, x, lg, h1, h2)
        saved = [h1.clone(), h2.clone()]
        # the stored first layer is read 16 bytes at a time, as the inputs are
        ctx.mlp_backward(p, x, _dev(y.astype(np.uint8)), lg, h1.clone(), h2,
                         _empty(ctx.mlp_workspace_bytes(n), torch.uint8), g, loss)
        h1b = _empty((n, 64), torch.int16, 1)
        ctx.mlp_forward(p, x, lg, h1b, h2)
        out.append([lg.clone(), g.clone(), loss.clone(), h1b.clone()] + saved)
    for a, b in zip(*out):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
