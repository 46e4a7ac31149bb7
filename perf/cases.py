"""Timed workloads of the library: whole events through the chain, batches,
pixel objects, training-set collection, and the scorer's training and scoring
calls, each through the public binding as a program calls it.

A chain pass is what an event loop does with one batch: hand the hits over,
run the chain, read the batch's counts and its kept quintuplets (or track
candidates).  The library returns objects in no fixed order, so a pass sorts
them by first hit, which is unique (kept quintuplets share no hit).

Events are drawn from a pool of simulated helices per detector and spectrum
(the configurations of ``synth.events``): a seed picks the tracks, smears,
drops and shuffles their hits and adds noise, so that making an event takes
milliseconds.
"""
import functools
import math

import numpy as np
import torch

import paper_2209_13711_amd as lst
from paper_2209_13711_amd import scorer
from synth import events as E, geometry as G, params as PR, weights as W

DEVICE = "cuda:0"
POOL = 12000          # helices of a pool; an event takes a part of them
NF, NH = 40, 64       # scorer inputs and hidden units


# ---------------------------------------------------------------- cases
def listed():
    return [
        # one small event (200 helices, barrel detector), per-stage launches:
        # the smallest call of the chain, latency only
        dict(name="event_small", family="chain", config=1, tracks=200, events=1, graph=False),
        # the headline workload: one PU200-like event, full detector, as a graph
        dict(name="event_pu200", family="chain", config=2, tracks=4000, events=1, graph=True),
        # the same with both learned scorers vetoing triplets and quintuplets,
        # windows widened as they are when the scorers are on
        dict(name="event_scored", family="chain", config=2, tracks=4000, events=1, graph=True,
             scored=True, window=1.5),
        # the same through the pixel stage to track candidates
        dict(name="event_pixel", family="pixel", config=2, tracks=4000, events=1),
        # 16 PU200-like events in one launch
        dict(name="batch_pu200", family="chain", config=2, tracks=4000, events=16, graph=True),
        # 24 events of uneven size (pileup 50 to 250) in one launch
        dict(name="batch_uneven", family="chain", config=3, tracks=5000, events=24, graph=True,
             uneven=True),
        # stress events (displaced tracks, noise, widened windows), hits
        # stored in half precision
        dict(name="stress_half", family="chain", config=5, tracks=6000, events=3, graph=True,
             window=1.5, half=True),
        # training set of the triplet scorer: features, labels, canonical order
        dict(name="collect_t3", family="collect", config=4, tracks=2000, events=1, kind=2),
        # training steps at the default batch size, several in one call (few:
        # rounding to BF16 makes longer runs of two correct programs part)
        dict(name="train_4096", family="train", batch=4096, steps=2),
        # one training step by the separate calls, rows that fill no tile
        dict(name="step_5000", family="step", rows=5000),
        # scoring a stored set of candidates: standardise, forward
        dict(name="rows_200003", family="rows", rows=200003),
        # scoring a handful of candidates
        dict(name="rows_16", family="rows", rows=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["event", "event", "batch", "pixel", "collect", "train", "step", "rows"])
    if family == "event":
        config = rng.choice([1, 2, 4, 5])
        c = dict(family="chain", config=config, tracks=_log(rng, 20, 4000), events=1,
                 graph=rng.random() < 0.7)
        if rng.random() < 0.3:
            c.update(scored=True, window=1.5)
        if rng.random() < 0.3:
            c.update(half=True)
        return c
    if family == "batch":
        return dict(family="chain", config=rng.choice([2, 3, 4]), tracks=_log(rng, 100, 3000),
                    events=rng.randint(2, 16), graph=True, uneven=rng.random() < 0.7)
    if family == "pixel":
        return dict(family="pixel", config=rng.choice([2, 5]), tracks=_log(rng, 100, 4000),
                    events=rng.randint(1, 3))
    if family == "collect":
        return dict(family="collect", config=rng.choice([2, 4]), tracks=_log(rng, 100, 2000),
                    events=rng.randint(1, 2), kind=rng.choice([2, 3]))
    if family == "train":
        return dict(family="train", batch=_log(rng, 64, 8192), steps=rng.randint(1, 3))
    if family == "step":
        return dict(family="step", rows=_log(rng, 1, 8192))
    return dict(family="rows", rows=_log(rng, 1, 200003))


# ---------------------------------------------------------------- inputs: events
@functools.lru_cache(maxsize=None)
def _pool(config):
    """exact sensor crossings of the pool's helices, sorted by track, and the helices"""
    cfg = E.CONFIGS[config]
    tracks = E._draw_tracks(cfg, np.random.default_rng(1000 + config), POOL)
    ev = E.simulate(G.get(cfg.geometry), E.Helices(**tracks), None)
    order = np.argsort(ev.truth, kind="stable")
    hits = {k: getattr(ev, k)[order] for k in ("x", "y", "z", "module", "sensor")}
    first = np.searchsorted(ev.truth[order], np.arange(POOL + 1))
    return hits, first, tracks


def _event(config, n, rng):
    """one event of n helices of the pool: smeared, thinned, noise added, shuffled"""
    cfg, geo = E.CONFIGS[config], G.get(E.CONFIGS[config].geometry)
    hits, first, tracks = _pool(config)
    pick = np.sort(rng.choice(POOL, size=n, replace=False))
    cnt = first[pick + 1] - first[pick]
    truth = np.repeat(np.arange(n), cnt)
    at = np.repeat(first[pick] - np.cumsum(cnt) + cnt, cnt) + np.arange(int(cnt.sum()))
    keep = rng.random(len(at)) >= cfg.ineff
    at, truth = at[keep], truth[keep]
    mod, sen = hits["module"][at], hits["sensor"][at]
    du, dv = rng.normal(0, cfg.sigma_u, len(at)), rng.normal(0, cfg.sigma_v, len(at))
    f = geo.f64
    pos = [hits[k][at] + du * f[u, mod] + dv * f[v, mod]
           for k, u, v in zip("xyz", (G.F_UX, G.F_UY, G.F_UZ), (G.F_VX, G.F_VY, G.F_VZ))]
    m = int(round(cfg.noise_frac * len(at)))
    if m:
        area = np.cumsum(f[G.F_HU] * f[G.F_HV])
        nm = np.searchsorted(area, rng.random(m) * area[-1])
        ns = rng.integers(0, 2, m)
        lu, lv = rng.uniform(-1, 1, m) * f[G.F_HU, nm], rng.uniform(-1, 1, m) * f[G.F_HV, nm]
        off = (ns - 0.5) * f[G.F_GAP, nm]
        for i in range(3):
            noise = (f[G.F_CX + i, nm] + off * f[G.F_WX + i, nm] + lu * f[G.F_UX + i, nm]
                     + lv * f[G.F_VX + i, nm])
            pos[i] = np.r_[pos[i], noise]
        mod, sen, truth = np.r_[mod, nm], np.r_[sen, ns], np.r_[truth, np.full(m, -1)]
    p = rng.permutation(len(mod))
    return E.Event(*(a[p].astype(np.float32) for a in pos), mod[p].astype(np.int32),
                   sen[p].astype(np.uint8), truth[p].astype(np.int32),
                   {k: v[pick] for k, v in tracks.items()})


def _events(case, seed):
    rng = np.random.default_rng([seed, case["config"]])
    n = case["tracks"]
    sizes = ([max(1, int(n * rng.uniform(0.2, 1.0))) for _ in range(case["events"])]
             if case.get("uneven") else [n] * case["events"])
    return [_event(case["config"], k, rng) for k in sizes]


def _cat(parts, name):
    return np.ascontiguousarray(np.concatenate([getattr(p, name) for p in parts]))


def _offsets(counts):
    return np.r_[0, np.cumsum(counts)].astype(np.int32)


# ---------------------------------------------------------------- inputs: scorer
# typical centre and spread of the features: five per mini-doublet (radius and
# |z| over 100 cm, bend pull, endcap and 2S flags), then the fit quantities
def _standardisation(n_md):
    mean, istd = np.zeros(NF, np.float32), np.full(NF, 1.0, np.float32)
    for j in range(n_md):
        mean[5 * j:5 * j + 5] = (0.35 + 0.15 * j, 0.0, 0.0, 0.3, 0.3)
        istd[5 * j:5 * j + 5] = (3.0, 1.0, 2.0, 2.0, 2.0)
    return mean, istd


def _network(seed):
    return W.random_params(np.random.default_rng(seed), bias=0.1)


def _context(case):
    cfg = E.CONFIGS[case["config"]]
    geo = G.get(cfg.geometry)
    ctx = lst.Context(PR.make(w=case.get("window", 1.0)), geo.f32, geo.i32, device=0)
    if case.get("half"):
        ctx.set_hit_storage(True)
    if case.get("scored"):
        for kind, n_md in ((lst.LST_T3, 3), (lst.LST_T5, 5)):
            ctx.mlp_load(_network(kind), *_standardisation(n_md), threshold=-0.6, kind=kind)
        ctx.set_mode(lst.LST_MODE_MLP)
    return ctx


def _rows(n, seed):
    """raw features [n, 40] and labels of stored candidates"""
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    mean, istd = (torch.from_numpy(a).to(DEVICE) for a in _standardisation(5))
    f = torch.randn((n, NF), generator=g, device=DEVICE) / istd + mean
    side = (f - mean) * istd
    y = (side[:, 25:33].sum(1) + torch.randn(n, generator=g, device=DEVICE) > 0).to(torch.uint8)
    return f, y, mean, istd


def _prepared(ctx, n, seed):
    """standardised BF16 rows, labels and fresh optimiser state"""
    f, y, mean, istd = _rows(n, seed)
    x = torch.empty((n, 64), dtype=torch.int16, device=DEVICE)
    ctx.mlp_prepare(f, mean, istd, x)
    p0 = torch.from_numpy(_network(7)).to(DEVICE)
    return x, y, p0


def _buffers(ctx, b):
    new = lambda shape, t: torch.empty(shape, dtype=t, device=DEVICE)
    return dict(logits=new(b, torch.float32), h1=new((b, 64), torch.int16),
                h2=new((b, 64), torch.float32), work=new(ctx.mlp_workspace_bytes(b), torch.uint8))


def _scorer_context():
    geo = G.get("barrel_toy")
    return lst.Context(PR.make(), geo.f32, geo.i32, device=0)


# ---------------------------------------------------------------- prepare
def prepare(case, seed):
    family = case["family"]
    if family in ("chain", "pixel", "collect"):
        ctx = _context(case)
        evs = _events(case, seed)
        s = dict(case=case, ctx=ctx, events=evs, offsets=_offsets([e.n_hits for e in evs]),
                 hits=[_cat(evs, k) for k in ("x", "y", "z", "module", "sensor")])
        if family == "collect":
            return s
        caps = lst.default_caps(len(evs), int(s["offsets"][-1]))
        if family == "pixel":
            px = [E.pixel_seeds(e, case["config"], seed % 2**31 + i) for i, e in enumerate(evs)]
            s["pixel"] = (_offsets([p.n_hits for p in px]), _cat(px, "x"), _cat(px, "y"),
                          _cat(px, "z"), _offsets([p.n_seeds for p in px]), _cat(px, "seeds"),
                          PR.make_pixel())
            n_sd = len(s["pixel"][5])
            caps.update(px_hits=max(1, len(s["pixel"][1])), seeds=max(1, n_sd),
                        px_cand=max(4096, 8 * n_sd))
        ctx.reserve(caps)
        # widened windows on dense events can exceed the default capacities:
        # the arena grows to the need here, once
        ctx.run_batch(s["offsets"], *s["hits"])
        return s
    ctx = _scorer_context()
    s = dict(case=case, ctx=ctx)
    if family == "rows":
        n = case["rows"]
        s["features"], _, s["mean"], s["istd"] = _rows(n, seed)
        s["params"] = torch.from_numpy(_network(7)).to(DEVICE)
        s["x"] = torch.empty((n, 64), dtype=torch.int16, device=DEVICE)
        s["logits"] = torch.empty(n, dtype=torch.float32, device=DEVICE)
        return s
    b = case["batch"] if family == "train" else case["rows"]
    n = b * _batches(case)
    s["x"], s["y"], p0 = _prepared(ctx, n, seed)
    s["buffers"] = _buffers(ctx, b)
    s["order"] = np.random.default_rng(seed).permutation(_batches(case)).astype(np.int32)
    # weights and Adam's moments as the training starts, and the trained ones
    s["start"] = torch.stack([p0, torch.zeros_like(p0), torch.zeros_like(p0)])
    s["state"], s["grad"] = torch.empty_like(s["start"]), torch.empty_like(p0)
    s["losses"] = torch.zeros(_batches(case), dtype=torch.float32, device=DEVICE)
    return s


def _batches(case):
    return case.get("steps", 1)


# ---------------------------------------------------------------- run
def _table(rows, n_max):
    """the rows in the program's table of n_max rows (the rest zero)"""
    assert len(rows) <= n_max, (len(rows), n_max)
    out = np.zeros((n_max,) + rows.shape[1:], rows.dtype)
    out[:len(rows)] = rows
    return out


def _kept(ctx, case):
    """counts and kept quintuplets of every event, by event and first hit"""
    counts, kept = [], []
    for e in range(case["events"]):
        c = ctx.counts(e)
        counts.append(np.hstack([v for k, v in c.items() if k != "rc"]))
        t = ctx.objects(e, lst.LST_T5_KEPT)
        kept.append(t[np.argsort(t[:, 0])])
    return dict(counts=np.array(counts, np.int64), sizes=np.array([len(k) for k in kept]),
                kept=_table(np.concatenate(kept), case["events"] * (2 * case["tracks"] + 16)))


def run(state):
    case, ctx = state["case"], state["ctx"]
    family = case["family"]
    if family in ("chain", "pixel"):
        ctx.load_hits(state["offsets"], *state["hits"])
        if family == "pixel" or case["graph"]:
            ctx.run_chain_graph()
        else:
            ctx.run_chain()
        if family == "chain":
            return _kept(ctx, case)
        ctx.load_pixel(*state["pixel"])
        ctx.run_pixel()
        return [_table(ctx.track_candidates(e), 2 * case["tracks"] + 16)
                for e in range(case["events"])]
    if family == "collect":
        features, labels = scorer.collect(ctx, state["events"], kind=case["kind"])
        n_max = case["events"] * (16 * case["tracks"] + 64)
        return dict(features=_table(features, n_max), labels=_table(labels, n_max))
    if family == "rows":
        ctx.mlp_prepare(state["features"], state["mean"], state["istd"], state["x"])
        ctx.mlp_forward(state["params"], state["x"], state["logits"])
        return dict(x=state["x"], logits=state["logits"])
    # every pass trains from the same start
    state["state"].copy_(state["start"])
    (p, m, v), grad = state["state"], state["grad"]
    bf, losses = state["buffers"], state["losses"]
    if family == "train":
        ctx.mlp_train_steps(p, state["x"], state["y"], case["batch"], state["order"], 0,
                            bf["logits"], bf["h1"], bf["h2"], bf["work"], grad, m, v, losses, 2e-3)
        return dict(params=p, m=m, v=v, losses=losses)
    ctx.mlp_forward(p, state["x"], bf["logits"], bf["h1"], bf["h2"])
    ctx.mlp_backward(p, state["x"], state["y"], bf["logits"], bf["h1"], bf["h2"], bf["work"], grad,
                     losses[:1])
    ctx.mlp_adam(p, grad, m, v, 1, 2e-3)
    return dict(params=p, m=m, v=v, grad=grad, losses=losses, logits=bf["logits"])


# ---------------------------------------------------------------- work
def work(case):
    """bytes: inputs read and results written once; flops: the candidate pairs
    of the chain at about 30 operations each (pairs grow with the square of
    the tracks: 1.1 M per PU200-like event, 1.6 M per 3000-track barrel event),
    the multiply-adds of the network"""
    family = case["family"]
    if family in ("chain", "pixel", "collect"):
        full = E.CONFIGS[case["config"]].geometry == "full"
        n = case["tracks"] * (0.6 if case.get("uneven") else 1.0)
        hits, pairs = (13.7 if full else 13.0) * n, (0.07 if full else 0.17) * n * n
        out = {"chain": 0.5 * 40, "pixel": 0.55 * 48 + 0.6 * 80, "collect": 4 * 161}[family] * n
        return {"bytes": case["events"] * (17.0 * hits + out), "flops": case["events"] * 30.0 * pairs}
    n_par = W.N_PARAM
    if family == "rows":
        n = case["rows"]
        return {"bytes": n * (160.0 + 128 + 128 + 4) + 4 * n_par, "flops": n * 13440.0}
    n = case["batch"] * case["steps"] if family == "train" else case["rows"]
    # a row read once, its share of the optimiser state of its step
    steps = _batches(case)
    saved = 0.0 if family == "train" else 2.0 * (4 + 128 + 256)
    return {"bytes": n * (129.0 + saved) + steps * 4.0 * 7 * n_par, "flops": n * 34944.0}


# ---------------------------------------------------------------- exact
def _bf16(t):
    """float64 values rounded to BF16 (ties to even), as float64"""
    return t.to(torch.float32).to(torch.bfloat16).to(torch.float64)


def _split(p):
    o, out = 0, []
    for shape in ((NH, NF), (NH,), (NH, NH), (NH,), (NH,), (1,)):
        n = math.prod(shape)
        out.append(p[o:o + n].reshape(shape))
        o += n
    return out


def _forward(p, x):
    w1, b1, w2, b2, w3, b3 = _split(p)
    h1 = _bf16(torch.relu(x @ _bf16(w1).T + b1))
    h2 = torch.relu(h1 @ _bf16(w2).T + b2)
    return h1, h2, h2 @ w3 + b3


def _gradient(p, x, y):
    """gradient of the mean cross-entropy and its value, weights and first
    hidden layer in BF16 as the products take them"""
    _, _, w2, _, w3, _ = _split(p)
    h1, h2, z = _forward(p, x)
    loss = (torch.relu(z) - z * y + torch.log1p(torch.exp(-z.abs()))).mean()
    g = (torch.sigmoid(z) - y) / len(y)
    d2 = g[:, None] * w3 * (h2 > 0)
    d1 = (d2 @ _bf16(w2)) * (h1 > 0)
    grad = torch.cat([(d1.T @ x).reshape(-1), d1.sum(0), (d2.T @ h1).reshape(-1), d2.sum(0),
                      h2.T @ g, g.sum()[None]])
    return grad, loss, z


def exact(case, seed):
    family = case["family"]
    if family in ("chain", "pixel", "collect"):
        return None   # hit indices and counts; features of whatever objects were found
    n = case["rows"] if family != "train" else case["batch"] * case["steps"]
    f, y, mean, istd = _rows(n, seed)
    # the rows as the network reads them: standardised in FP32, rounded to BF16
    x = ((f - mean) * istd).to(torch.bfloat16).to(torch.float64)
    p = torch.from_numpy(_network(7)).to(DEVICE, torch.float64)
    if family == "rows":
        return dict(x=None, logits=_forward(p, x)[2])
    y = y.to(torch.float64)
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    losses = torch.zeros(_batches(case), dtype=torch.float64, device=DEVICE)
    order = np.random.default_rng(seed).permutation(_batches(case))
    b = n // _batches(case)
    for t, k in enumerate(order.tolist(), 1):
        grad, losses[k], z = _gradient(p, x[k * b:(k + 1) * b], y[k * b:(k + 1) * b])
        m = 0.9 * m + 0.1 * grad
        v = 0.999 * v + 0.001 * grad * grad
        p = p - 2e-3 * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
    out = dict(params=p, m=m, v=v, losses=losses)
    return out if family == "train" else dict(out, grad=grad, logits=z)
