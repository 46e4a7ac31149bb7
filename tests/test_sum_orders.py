"""Orders in which the scorer's kernels add, on the CPU in FP32: none may be
further off than the orders used before (16 lanes of four terms each for a
logit, at most 64 chunks of rows one after the other for a gradient), against
sums in FP64."""
import numpy as np
import pytest

F = np.float32


def serial(t):
    """terms along the last axis, one after the other"""
    a = t[..., 0]
    for k in range(1, t.shape[-1]):
        a = a + t[..., k]
    return a


def logit_sum(t):
    """units 16 nt + 4 q + r of [n, 64]: nt in order, then the sums (q, r) by
    q ^ 2, q ^ 1, r ^ 2, r ^ 1, as the lanes of the kernels add"""
    s = serial(t.reshape(-1, 4, 4, 4).transpose(0, 2, 3, 1))     # q, r
    s = s[:, :2] + s[:, 2:]
    s = s[:, 0] + s[:, 1]
    s = s[:, :2] + s[:, 2:]
    return s[:, 0] + s[:, 1]


def logit_sum_lanes(t):
    """units 16 nt + c: nt in order, then the 16 lanes by halves"""
    a = serial(t.reshape(-1, 4, 16).transpose(0, 2, 1))
    for d in (8, 4, 2, 1):
        a = a[:, :d] + a[:, d:2 * d]
    return a[:, 0]


def chunk_sum(p):
    """partial sums of up to 128 chunks [.., chunks]: every fourth in order, the
    four sums by pairs"""
    p = np.concatenate([p, np.zeros(p.shape[:-1] + (128 - p.shape[-1],), F)], -1)
    w = [serial(np.concatenate([np.zeros(p.shape[:-1] + (1,), F), p[..., k::4]], -1)) for k in range(4)]
    return (w[0] + w[1]) + (w[2] + w[3])


def rms(got, terms):
    ref = terms.astype(np.float64).sum(-1)
    return float(np.sqrt(((got - ref) ** 2).mean() / (ref ** 2).mean()))


@pytest.mark.parametrize("seed", range(4))
def test_logit_sum_is_no_further_off(seed):
    rng = np.random.default_rng(seed)
    h2 = np.maximum(rng.normal(0.1, 1, (50000, 64)), 0).astype(F)
    t = h2 * rng.normal(0, 0.125, 64).astype(F)
    assert logit_sum(t).dtype == F
    assert rms(logit_sum(t), t) <= rms(logit_sum_lanes(t), t)


@pytest.mark.parametrize("rows", [64, 4096, 5056, 8192])
def test_chunk_sum_is_no_further_off(rows):
    """rows of random terms, 64 to a chunk, or twice as many where that would
    be more than 64 chunks"""
    t = np.random.default_rng(rows).normal(0.02, 1, (4000, rows)).astype(F)
    batches = serial(t.reshape(4000, -1, 64))
    per = 2 if rows > 4096 else 1
    was = serial(np.stack([serial(t[:, k:k + 64 * per]) for k in range(0, rows, 64 * per)], -1))
    assert rms(chunk_sum(batches), t) <= rms(was, t)
