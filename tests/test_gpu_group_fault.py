"""The one-launch grouping reports hits that do not fit the positions it
counted (error bit 2) through a byte per wave behind the chain's counters, 16
for each of 256 ranges of modules.  No hits do that, so the bytes are written
from the host: counts and getters refuse, and the next chain runs clean."""
import numpy as np
import pytest

import oracle
from synth import events as E
from synth import geometry as G
from synth import params as PR
from tests.parity import assert_parity

pytestmark = pytest.mark.gpu

# counters: the error word is the second, the waves' bytes follow 64 words and a
# line of 64 for each of 4 object types x 32 shards
GROUP = 64 + 4 * 32 * 64
GROUP_BYTES = 256 * 16


def counters(ctx):
    """byte offset of the counters in the arena: the error word is the one
    that the error hook changes"""
    before = ctx.arena.clone()
    ctx.raise_error_flags(2)
    at = int((ctx.arena != before).nonzero()[0])
    return at - 4


@pytest.mark.parametrize("wave", [0, 1237, GROUP_BYTES - 1])
@pytest.mark.parametrize("chain", ["run_chain", "run_chain_graph", "run_chain_persistent"])
def test_inconsistent_grouping_is_reported(wave, chain):
    import paper_2209_13711_amd as lst
    geo, params = G.get("barrel_toy"), PR.make()
    ev = E.generate(1, 4)
    ref = oracle.Oracle(params, geo.f32, geo.i32).run_event(ev)
    ctx = lst.Context(params, geo.f32, geo.i32, device=0)
    print(f"case group fault byte {wave} {chain}", flush=True)
    assert_parity(ctx.run_event(ev), ref)
    byte = counters(ctx) + 4 * GROUP + wave
    assert_parity(ctx.run_event(ev), ref)
    ctx.arena[byte] = 4
    for fn in (lambda: ctx.objects(0, lst.LST_MD), lambda: ctx.objects(0, lst.LST_T5_KEPT),
               lambda: ctx.t5_scores(0)):
        with pytest.raises(lst.LSTError) as ei:
            fn()
        assert ei.value.code == lst.LST_E_FAULT, ei.value
    # every kind of chain starts from clean bytes
    ctx.load_hits(np.array([0, ev.n_hits], np.int32), ev.x, ev.y, ev.z, ev.module, ev.sensor)
    getattr(ctx, chain)()
    assert_parity({k: ctx.objects(0, k) for k in range(5)}, ref)
    assert ctx.counts(0)["error_flags"] == 0
    # and the counts see a byte set before they are first read
    ctx.run_chain()
    ctx.arena[byte] = 4
    c = ctx.counts(0, check=False)
    assert c["rc"] == lst.LST_E_FAULT and c["error_flags"] == 4
