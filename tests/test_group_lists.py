"""The lists of the one-launch hit grouping, on a model of a wave's lanes: a
wave walks the hits in groups of four per lane, then its first lanes take the
last one to three hits, and each ballot places the hits of the wave's range in
its list.  Lanes without a hit sit a ballot out, so their own count of the
list falls behind; every place has to come from the first lane's count."""
import numpy as np
import pytest

BLOCK, LANES = 1024, 64     # threads of a block, lanes of a wave


def steps(n_hits, wave):
    """hit of each lane at each ballot (-1: the lane sits it out)"""
    t = LANES * wave + np.arange(LANES)
    n_g = n_hits // 4
    for g in range(0, n_g, BLOCK):
        for k in range(4):
            yield np.where(g + t < n_g, 4 * (g + t) + k, -1)
    yield np.where(4 * n_g + t < n_hits, 4 * n_g + t, -1)


def listed(n_hits, wave, in_range, one_count):
    """the list a wave writes: place -> hits written there, and its length"""
    own = np.zeros(LANES, np.int64)
    places = {}
    for h in steps(n_hits, wave):
        act = h >= 0
        if not act.any():
            continue
        assert act[0] and not (np.diff(act.astype(int)) > 0).any()   # a prefix of the lanes
        on = act & in_range(h)
        if one_count:
            own[act] = own[0]
        for lane, rank in zip(np.flatnonzero(on), range(int(on.sum()))):
            places.setdefault(int(own[lane] + rank), []).append(int(h[lane]))
        own[act] += int(on.sum())
    return places, int(own[0])


def whole(n_hits, in_range, one_count, waves=(0,)):
    """every hit of the range once, and no place left out or written twice"""
    for w in waves:
        want = sorted(x for h in steps(n_hits, w) for x in h[(h >= 0) & in_range(h)].tolist())
        places, length = listed(n_hits, w, in_range, one_count)
        got = [x for at in range(length) for x in places.get(at, [None])]
        if length != len(want) or len(places) != length or sorted(got, key=lambda x: -1 if x is None else x) != want:
            return False
    return True


COUNTS = list(range(0, 300)) + [k * 4096 + d for k in (1, 2, 13) for d in range(-8, 17)]


@pytest.mark.parametrize("last", [None, 16, 3])
def test_one_count_lists_every_hit_once(last):
    """all hits in the range, or the last 16 or 3"""
    for n in COUNTS:
        assert whole(n, lambda h: h >= (0 if last is None else n - last), True), n
    for n in (5000, 8191, 8192):
        assert whole(n, lambda h: h % 5 == 0, True, waves=range(16)), n


def test_each_lanes_own_count_does_not():
    """where the lists were wrong: 6, 7 or 11 hits past a multiple of 4096"""
    bad = [n for n in COUNTS if not whole(n, lambda h: h >= 0, False)]
    assert bad == [n for n in COUNTS if n % 4096 in (6, 7, 11)]
    places, length = listed(6, 0, lambda h: h >= 0, False)
    assert length == 6 and 5 not in places and places[1] == [1, 5]
