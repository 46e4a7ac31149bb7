"""The tie list of one hit in duplicate removal, on a model of its first pass:
quintuplets arrive in any order at a minimum of (score, index), and of two that
tie there the one left without the minimum's index is recorded."""
import numpy as np
import pytest


def first_pass(scores, order):
    best, ties = None, []
    for t in order:
        key = (scores[t], t)
        if best is not None and best[0] == key[0]:
            ties.append(best[1] if key < best else t)
        if best is None or key < best:
            best = key
    return best, ties


@pytest.mark.parametrize("values", [1, 2, 5, 40])
def test_ties_are_listed_once(values):
    """the list and the minimum's index hold all that reach the minimum, once
    each; records are one per tie, so as many as those but one when every
    score is the same"""
    rng = np.random.default_rng(values)
    for n in list(range(1, 20)) * 20 + [60] * 20:
        scores = rng.integers(0, values, n)
        order = rng.permutation(n)
        (low, at), ties = first_pass(scores, order)
        reach = np.flatnonzero(scores == scores.min()).tolist()
        assert low == scores.min() and at == reach[0]
        assert sorted([t for t in ties if scores[t] == low] + [at]) == reach
        assert len(ties) == len(set(ties))
        if values == 1:
            assert len(ties) == n - 1
