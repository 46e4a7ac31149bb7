"""Hit grouping of one event in one launch, at the sizes where it changes:
hits outnumbering a wave's list of its range, hit counts that split the
16-byte loads, no hit, invalid ids before, between and after the others; and
the event counts next to it, which take other kernels."""
import numpy as np
import pytest

import oracle
from synth import events as E
from synth import geometry as G
from synth import params as PR
from tests.parity import assert_parity

pytestmark = pytest.mark.gpu


def _run(cid, evs, chains=("stages", "graph", "persistent")):
    import paper_2209_13711_amd as lst
    cfg = E.CONFIGS[cid]
    geo = G.get(cfg.geometry)
    params = PR.make(w=cfg.window)
    orc = oracle.Oracle(params, geo.f32, geo.i32)
    ctx = lst.Context(params, geo.f32, geo.i32, device=0)
    b = E.concat(evs)
    ctx.run_batch(b.offsets, b.x, b.y, b.z, b.module, b.sensor)
    refs = []
    for ev in evs:
        ok = (ev.module >= 0) & (ev.module < geo.n_mod) & (ev.sensor <= 1)
        back = np.nonzero(ok)[0]
        r = orc.run(ev.x[ok], ev.y[ok], ev.z[ok], ev.module[ok], ev.sensor[ok])
        refs.append((r, back))
    bad = any((ev.module < 0).any() or (ev.module >= geo.n_mod).any() or (ev.sensor > 1).any()
              for ev in evs)
    for chain in chains:
        ctx.load_hits(b.offsets, b.x, b.y, b.z, b.module, b.sensor)
        dict(stages=ctx.run_chain, graph=ctx.run_chain_graph,
             persistent=ctx.run_chain_persistent)[chain]()
        for e, (ref, back) in enumerate(refs):
            got = {k: ctx.objects(e, k) for k in range(5)}
            for k in range(5):
                want = set(map(tuple, back[ref.tuples[k]].tolist())) if len(ref.tuples[k]) else set()
                assert set(map(tuple, got[k].tolist())) == want, (chain, e, k)
            c = ctx.counts(e)
            assert c["error_flags"] == int(bad)
            assert [c["cand_md"], c["cand_seg"], c["cand_t3"], c["cand_t5"]] == ref.cands.tolist()


def _with(ev, module, sensor, n, at_front=False):
    """n more hits on (module, sensor) at spread positions"""
    rng = np.random.default_rng(n)
    cat = (lambda a, b: np.r_[b, a]) if at_front else (lambda a, b: np.r_[a, b])
    out = E.Event(*[cat(getattr(ev, k), rng.uniform(-1, 1, n).astype(np.float32)) for k in "xyz"],
                  cat(ev.module, np.full(n, module, np.int32)),
                  cat(ev.sensor, np.full(n, sensor, np.uint8)),
                  cat(ev.truth, np.full(n, -1, np.int32)))
    return out


def _empty():
    z = np.zeros(0, np.float32)
    return E.Event(z, z, z, np.zeros(0, np.int32), np.zeros(0, np.uint8), np.zeros(0, np.int32))


@pytest.mark.parametrize("n", [255, 4097, 9001])
def test_more_hits_in_a_range_than_its_lists(n):
    """all of them lower hits of one module, so they form no pairs"""
    print(f"case group list {n}", flush=True)
    ev = E.generate(1, 40)
    free = np.setdiff1d(np.arange(G.get("barrel_toy").n_mod), ev.module)[0]
    _run(1, [_with(ev, free, 0, n)])


@pytest.mark.parametrize("extra", [1, 2, 3, 4])
def test_hit_counts_and_invalid_ids(extra):
    """every remainder of four hits; invalid ids first, last and on a module
    whose lists overflow"""
    print(f"case group remainder {extra}", flush=True)
    ev = E.generate(1, 41, n_tracks=30)
    _run(1, [_with(ev, 17, 0, extra)])
    _run(1, [_with(_with(_with(ev, -7, 1, extra, at_front=True), 3, 1, 5000), 8244, 0, 1)])


@pytest.mark.parametrize("n_events", [1, 2, 3, 7, 8])
def test_uneven_events_with_invalid_hits(n_events):
    """odd event sizes, empty events, invalid module and sensor ids in the
    first event and in the middle of others"""
    print(f"case group events {n_events}", flush=True)
    evs = [E.generate(1, 50 + e, n_tracks=15 + 13 * e) for e in range(n_events)]
    evs[0] = _with(evs[0], -1, 0, 3, at_front=True)
    if n_events > 2:
        evs[1] = _empty()
        evs[2] = _with(_with(evs[2], 5, 2, 1, at_front=True), 1 << 30, 0, 2)
    if n_events > 3:
        evs[-1] = _empty()
    _run(1, evs)


@pytest.mark.parametrize("tracks", [0, 1, 2])
def test_almost_nothing(tracks):
    print(f"case group tracks {tracks}", flush=True)
    _run(2, [E.generate(2, 60, n_tracks=tracks) if tracks else _empty()])
