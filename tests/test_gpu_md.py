"""Mini-doublet enumeration at the sizes where its walk changes: lower hits
around one wave's 64, one lower hit with many upper hits, more accepted pairs
than a wave stages, several dense modules of a wave, in the barrel and the
endcap, one event and several.  Object sets, counts and indices must equal the
oracle's."""
import numpy as np
import pytest

import oracle
from synth import events as E
from synth import geometry as G
from synth import params as PR

pytestmark = pytest.mark.gpu
CID = 2


def _seeds(geo, orc, barrel):
    """an event, and (lower hit, upper hit) of one mini-doublet of the oracle
    on each of its modules of one kind"""
    ev = E.generate(CID, 70, n_tracks=60)
    first = {}
    for lo, up in orc.run(ev.x, ev.y, ev.z, ev.module, ev.sensor).tuples[0].tolist():
        first.setdefault(int(ev.module[lo]), (lo, up))
    kind = geo.i32[G.I_SUBDET] == G.SUBDET_BARREL
    return ev, [p for m, p in sorted(first.items()) if kind[m] == barrel]


def _dense(ev, pairs, n_lo, n_up):
    """n_lo lower and n_up upper hits next to each given pair's"""
    rng = np.random.default_rng(n_lo * 1000 + n_up)
    idx = np.concatenate([np.r_[np.full(n_lo, lo), np.full(n_up, up)] for lo, up in pairs])
    x, y, z = ((a[idx] + rng.uniform(-2e-3, 2e-3, idx.size)).astype(np.float32)
               for a in (ev.x, ev.y, ev.z))
    return E.Event(x, y, z, ev.module[idx], ev.sensor[idx], ev.truth[idx])


@pytest.mark.parametrize("n_ev", [1, 3])
@pytest.mark.parametrize("barrel", [True, False])
@pytest.mark.parametrize("n_lo,n_up,n_mod", [(1, 1, 1), (63, 1, 1), (64, 1, 2), (65, 2, 1),
                                             (1, 130, 3), (65, 5, 1), (130, 9, 4)])
def test_dense_modules(n_lo, n_up, n_mod, barrel, n_ev):
    import paper_2209_13711_amd as lst
    print(f"case md {n_lo} {n_up} {n_mod} barrel={barrel} events={n_ev}", flush=True)
    cfg = E.CONFIGS[CID]
    geo = G.get(cfg.geometry)
    params = PR.make(w=cfg.window)
    orc = oracle.Oracle(params, geo.f32, geo.i32)
    ev, pairs = _seeds(geo, orc, barrel)
    evs = [_dense(ev, pairs[e:e + n_mod], n_lo, n_up) for e in range(n_ev)]
    refs = [orc.run(v.x, v.y, v.z, v.module, v.sensor) for v in evs]
    assert sum(len(r.tuples[0]) for r in refs) > 0
    ctx = lst.Context(params, geo.f32, geo.i32, device=0)
    b = E.concat(evs)
    ctx.run_batch(b.offsets, b.x, b.y, b.z, b.module, b.sensor)
    for e, ref in enumerate(refs):
        c = ctx.counts(e)
        assert c["error_flags"] == 0
        assert [c["cand_md"], c["cand_seg"], c["cand_t3"], c["cand_t5"]] == ref.cands.tolist()
        for k in range(5):
            assert sorted(map(tuple, ctx.objects(e, k).tolist())) == sorted(map(tuple, ref.tuples[k].tolist()))
