"""After a kernel-side time-out the stored indices may be of any value: the
getters' kernels look at the error word before they follow one.  The time-out
is raised from the host, and everything behind the chain's counters in the
arena is overwritten with indices out of every range."""
import numpy as np
import pytest

from synth import events as E
from synth import geometry as G
from synth import params as PR
from tests.test_gpu_group_fault import GROUP, GROUP_BYTES, counters

pytestmark = pytest.mark.gpu


def _overwrite(ctx):
    ctx.arena[counters(ctx) + 4 * GROUP + GROUP_BYTES:] = 0x7f


def _all_refuse(lst, calls):
    for fn in calls:
        with pytest.raises(lst.LSTError) as ei:
            fn()
        assert ei.value.code == lst.LST_E_FAULT, ei.value


@pytest.mark.parametrize("n_events", [1, 3])
def test_objects_are_not_followed(n_events):
    import paper_2209_13711_amd as lst
    geo = G.get("barrel_toy")
    ctx = lst.Context(PR.make(), geo.f32, geo.i32, device=0)
    b = E.concat([E.generate(1, 70 + e) for e in range(n_events)])
    caps = lst.default_caps(n_events, int(b.offsets[-1]))
    ctx.reserve(dict(caps, features=1))
    print(f"case fault first {n_events} events", flush=True)
    ctx.run_batch(b.offsets, b.x, b.y, b.z, b.module, b.sensor)
    ctx.run_t3_features()
    ctx.run_t5_features()
    assert len(ctx.objects(0, lst.LST_T5)) > 0
    _overwrite(ctx)
    for e in range(n_events):
        _all_refuse(lst, [lambda k=k: ctx.objects(e, k) for k in range(5)]
                    + [lambda f=f: f(e) for f in (ctx.t5_scores, ctx.t5_logits, ctx.t3_logits,
                                                  ctx.t3_features, ctx.t5_features, ctx.counts)])
        c = ctx.counts(e, check=False)
        assert c["rc"] == lst.LST_E_FAULT and c["error_flags"] == 2
        assert c["n_hits"] == b.offsets[e + 1] - b.offsets[e]


def test_pixel_rows_are_not_followed():
    import paper_2209_13711_amd as lst
    geo = G.get("full")
    ctx = lst.Context(PR.make(), geo.f32, geo.i32, device=0)
    ev = E.generate(2, 71, n_tracks=300)
    print("case fault first pixel", flush=True)
    assert len(ctx.run_event_pixel(ev, E.pixel_seeds(ev, 2, 1), PR.make_pixel())) > 0
    assert len(ctx.pixel_candidates(0, 0)) > 0
    _overwrite(ctx)
    _all_refuse(lst, [lambda: ctx.track_candidates(0), lambda: ctx.pixel_candidates(0, 0),
                      lambda: ctx.pixel_candidates(0, 1), lambda: ctx.objects(0, lst.LST_T5_KEPT)])
