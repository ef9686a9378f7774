"""Workloads of the library's public entry points, small to large.

`listed()` names the cases, `draw(rng)` makes another one of the same ranges,
`prepare(case, seed)` builds what a program holds before the call, `run(state)`
is one pass, `work(case)` the bytes and operations that a pass cannot do
without, and `exact(case, seed)` the computed floating-point outputs in 64 bits
by plain torch.

Inputs are the synthetic traces of the benchmark and the tests: iteration-
structured timelines with lognormal trace lengths, plain traces with
exponential gaps, and integer tensors of gamma-distributed region times.
"""
import functools
import math
import random

import numpy as np
import torch

from paper_2605_03561_amd import gpu_synth, synth, ta

DEV = "cuda:0"
APP_SEED = 77          # one application: its tree, marker and regions
KEPT = 150             # nodes of a pruned tree
N_AE = 24928           # parameters of the pre-screen's network
ROBUST = 1.4826
MEAN_DEV = 1.253314


# ---- cases -------------------------------------------------------------------

def listed():
    return [
        # A job of 16 ranks looked at interactively, call by call: nothing but
        # launches and host work.
        dict(name="eager_16_ranks", kind="eager", ranks=16, events=2000, nodes=200, iters=40,
             regions=16),
        # The plain workload that a CPU can check (64 ranks x 10,000 events),
        # as one graph launch and the rack / chassis summary.
        dict(name="plan_64_ranks", kind="plan", layout="plain", ranks=64, events=10000, nodes=200,
             iters=100, regions=16, ragged=True),
        # The same batch step on a mid-sized job: 10,000 ranks, long traces, a
        # 1,000-node tree, 300 iterations of 32 regions.
        dict(name="plan_10000_ranks", kind="plan", layout="timeline", ranks=10000, events=50000,
             nodes=1000, iters=300, regions=32, ragged=False),
        # The shape of the 100,000-rank batch (5,000 nodes, 500 iterations, 64
        # regions) with 40,000 ranks.
        dict(name="plan_40000_ranks", kind="plan", layout="timeline", ranks=40000, events=20000,
             nodes=5000, iters=500, regions=64, ragged=False),
        # A mixed batch: six requests of one application, 1,000 to 16,000 ranks
        # and 100 to 300 iterations, some ranks ending early.
        dict(name="batch_6_requests", kind="batch", requests=6, ranks_lo=1000, ranks_hi=16000,
             iters_lo=100, iters_hi=300, nodes=5000, regions=64),
        # Statistics of a tensor that a program already holds, odd in every
        # size: imbalance without the pass's totals, plain z scores, the scan
        # of the totals, rack / chassis summary.
        dict(name="stats_3001_ranks", kind="stats", ranks=3001, iters=217, regions=37),
        # Every node of the tree per rank and iteration, in sparse rows.
        dict(name="node_model_1500_ranks", kind="node_model", ranks=1500, events=20000, nodes=5000,
             iters=500, regions=64),
        # Sparse per-rank profiles and time windows over a tree of 97,833 nodes.
        dict(name="window_97833_nodes", kind="window", ranks=3000, events=20000, nodes=97833),
        # Profiles and the dense model on the 150 largest nodes of a pruned tree,
        # and what pruning this run at 1 % would keep.
        dict(name="pruned_4000_ranks", kind="pruned", ranks=4000, events=10000, nodes=5000,
             iters=200, regions=64),
        # Grouping of 100,000 ranks: K-Means on region totals, DBSCAN on the
        # totals, compute nodes shared by the groups.
        dict(name="cluster_100000_ranks", kind="cluster", ranks=100000, regions=64, k=6),
        # Training of the pre-screen's network: one gradient, then five epochs
        # from a checkpoint to a checkpoint.
        dict(name="train_90000_rows", kind="train", ranks=300, iters=300, epochs=5, batch=4096),
        # The pre-screen of a 10,000-rank tensor with a network in hand.
        dict(name="prescreen_10000_ranks", kind="prescreen", ranks=10000, iters=300),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["eager", "plan", "plan", "plan", "batch", "stats", "node_model", "window",
                       "pruned", "cluster", "train", "prescreen"])
    if kind == "eager":
        return dict(kind=kind, ranks=_log(rng, 3, 300), events=_log(rng, 300, 10000), nodes=200,
                    iters=rng.randint(5, 100), regions=rng.randint(2, 24))
    if kind == "plan":
        if rng.random() < 0.3:
            return dict(kind=kind, layout="plain", ranks=_log(rng, 16, 500),
                        events=_log(rng, 1000, 20000), nodes=200, iters=rng.randint(10, 100),
                        regions=rng.randint(2, 24), ragged=True)
        ranks = _log(rng, 300, 40000)
        iters = rng.randint(30, 500)
        regions = rng.randint(5, 64)
        return dict(kind=kind, layout="timeline", ranks=ranks, events=_log(rng, 5000, 20000),
                    nodes=_log(rng, 1000, 5000), iters=iters, regions=regions,
                    ragged=ranks < 12000 and rng.random() < 0.5)
    if kind == "batch":
        lo = _log(rng, 300, 2000)
        it = rng.randint(60, 150)
        return dict(kind=kind, requests=rng.randint(2, 6), ranks_lo=lo,
                    ranks_hi=lo * rng.randint(2, 8) + 1, iters_lo=it,
                    iters_hi=it + rng.randint(1, 150), nodes=_log(rng, 1500, 5000),
                    regions=rng.randint(16, 64))
    if kind == "stats":
        return dict(kind=kind, ranks=_log(rng, 50, 20000), iters=rng.randint(10, 300),
                    regions=rng.randint(3, 64))
    if kind == "node_model":
        return dict(kind=kind, ranks=_log(rng, 50, 1500), events=_log(rng, 3000, 40000),
                    nodes=_log(rng, 1500, 8000), iters=rng.randint(30, 500),
                    regions=rng.randint(8, 64))
    if kind == "window":
        return dict(kind=kind, ranks=_log(rng, 100, 3000), events=_log(rng, 2000, 20000),
                    nodes=_log(rng, 2000, 97833))
    if kind == "pruned":
        return dict(kind=kind, ranks=_log(rng, 100, 4000), events=_log(rng, 3000, 20000),
                    nodes=_log(rng, 1500, 5000), iters=rng.randint(30, 200),
                    regions=rng.randint(8, 64))
    if kind == "cluster":
        return dict(kind=kind, ranks=_log(rng, 1000, 100000), regions=rng.randint(1, 64),
                    k=rng.randint(2, 8))
    if kind == "train":
        return dict(kind=kind, ranks=rng.randint(20, 300), iters=rng.randint(50, 300),
                    epochs=rng.randint(1, 5), batch=rng.choice([1000, 2048, 4096]))
    return dict(kind=kind, ranks=_log(rng, 300, 10000), iters=rng.randint(30, 300))


# ---- inputs ------------------------------------------------------------------

def _gen(seed, *salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(hash((int(seed),) + salt) & 0x7FFFFFFFFFFFFFFF)
    return g


@functools.lru_cache(maxsize=8)
def _plain_app(nodes, regions):
    rng = np.random.default_rng([APP_SEED, nodes, regions])
    while True:  # a tree of `nodes` with room for that many disjoint regions
        parent = synth.make_tree(rng, nodes, 8)
        marker = synth.pick_marker(rng, parent)
        try:
            return parent, marker, synth.pick_regions(rng, parent, marker, regions)
        except ValueError:
            continue


@functools.lru_cache(maxsize=4)
def _deep_tree(nodes):
    return synth.make_tree(np.random.default_rng([APP_SEED, nodes]), nodes, 12)


def _plain_traces(seed, ranks, events, nodes, iters, regions):
    """Traces of unequal lengths (0.6 to 1 times `events`), gaps Exp(2 us), a
    marker about every events / iters events: ranks differ in their number of
    iterations."""
    parent, marker, regs = _plain_app(nodes, regions)
    rng = np.random.default_rng([seed, ranks, events])
    lens = rng.integers(max(1, int(0.6 * events)), events + 1, ranks)
    offsets = np.zeros(ranks + 1, np.int64)
    np.cumsum(lens, out=offsets[1:])
    E = int(offsets[-1])
    off = torch.from_numpy(offsets).to(DEV)
    g = _gen(seed, 1)
    gaps = torch.empty(E, device=DEV, dtype=torch.float64).exponential_(1 / 2000.0, generator=g)
    t = torch.cumsum(gaps.round_().to(torch.int64), 0)
    rank = torch.repeat_interleave(torch.arange(ranks, device=DEV), torch.from_numpy(lens).to(DEV))
    t0 = torch.randint(0, 10**9, (ranks,), device=DEV, generator=g)
    ts = (t - t[off[:-1]][rank] + t0[rank]).contiguous()
    pool = torch.from_numpy(np.delete(np.arange(nodes), marker)).to(DEV)  # the marker is a leaf
    ctx = pool[torch.randint(0, nodes - 1, (E,), device=DEV, generator=g)].to(torch.int32)
    pos = torch.arange(E, device=DEV) - off[:-1][rank]
    ctx[pos % max(1, events // iters) == 0] = marker
    step = max(1, events // iters)
    n_iters = -(-events // step)
    return dict(parent=parent, marker=marker, regions=regs, offsets=off, offsets_host=offsets,
                ts=ts, ctx=ctx.contiguous(), n_iters=n_iters)


def _timeline(seed, ranks, events, nodes, iters, regions, ragged, min_len=None, max_len=None):
    w = gpu_synth.timeline_on_gpu(seed=int(seed) % (1 << 31), n_ranks=ranks, median_len=events,
                                  min_len=min_len or max(iters, events // 20),
                                  max_len=max_len or 10 * events, n_nodes=nodes, depth_max=12,
                                  n_iters=iters, n_regions=regions, inject_frac=0.02,
                                  inject_regions=min(3, regions), device=DEV, app_seed=APP_SEED)
    out = dict(parent=w.parent, marker=w.marker, regions=w.regions, offsets=w.offsets,
               offsets_host=w.offsets_host, ts=w.ts, ctx=w.ctx, n_iters=iters)
    if ragged:  # every eighth rank or so ends early, after whole iterations
        rng = np.random.default_rng([seed, 2])
        have = np.where(rng.random(ranks) < 0.12, rng.integers((iters + 1) // 2, iters + 1, ranks),
                        iters)
        old = w.offsets_host
        lens = np.where(have < iters, have * w.events_per_iter.astype(np.int64), np.diff(old))
        offsets = np.zeros(ranks + 1, np.int64)
        np.cumsum(lens, out=offsets[1:])
        shift = torch.from_numpy(old[:-1] - offsets[:-1]).to(DEV)
        idx = torch.repeat_interleave(shift, torch.from_numpy(lens).to(DEV))
        idx += torch.arange(int(offsets[-1]), device=DEV)
        out.update(offsets=torch.from_numpy(offsets).to(DEV), offsets_host=offsets,
                   ts=w.ts[idx], ctx=w.ctx[idx])
    return out


def _traces(case, seed):
    c = case
    if c["kind"] == "eager" or c.get("layout") == "plain":
        return _plain_traces(seed, c["ranks"], c["events"], c["nodes"], c["iters"], c["regions"])
    return _timeline(seed, c["ranks"], c["events"], c["nodes"], c["iters"], c["regions"],
                     c.get("ragged", True))


def _requests(case):
    """(ranks, iterations) of a mixed batch's requests, geometric in the ranks."""
    n = case["requests"]
    out = []
    for q in range(n):
        f = q / max(1, n - 1)
        out.append((int(round(case["ranks_lo"] * (case["ranks_hi"] / case["ranks_lo"]) ** f)),
                    case["iters_lo"] + (case["iters_hi"] - case["iters_lo"]) * ((q * 5) % n) //
                    max(1, n - 1)))
    return out


def _request_traces(case, seed, q):
    ranks, iters = _requests(case)[q]
    return _timeline(seed * 1000 + q, ranks, 40 * iters, case["nodes"], iters, case["regions"], True,
                     min_len=2 * iters, max_len=400 * iters)


def _tensor(seed, ranks, iters, regions):
    """Region times: gamma with a mean per region and a factor per rank, some
    cells not sampled (0), every eighth rank or so with fewer iterations."""
    g = _gen(seed, 3)
    mu = torch.exp(torch.empty(regions, device=DEV).uniform_(math.log(2e4), math.log(5e5),
                                                             generator=g))
    f = torch.randn(ranks, device=DEV, generator=g).mul_(0.05).add_(1.0).clamp_(min=0.5)
    # the sum of four exponentials is a gamma variable of shape 4
    T = torch.zeros((ranks, iters, regions), device=DEV, dtype=torch.float32)
    for _ in range(4):
        T += torch.empty_like(T).exponential_(1.0, generator=g)
    T *= (mu / 4.0) * f[:, None, None]
    T *= torch.empty_like(T).uniform_(generator=g) > 0.08
    short = torch.rand(ranks, device=DEV, generator=g) < 0.12
    have = torch.randint((iters + 1) // 2, iters + 1, (ranks,), device=DEV, generator=g)
    it = torch.where(short, have, torch.full_like(have, iters)).to(torch.int32)
    T *= torch.arange(iters, device=DEV)[None, :, None] < it[:, None, None]
    return T.round_().to(torch.int64), it


def _placement(seed, ranks):
    node, rack, chassis = synth.topology(int(seed) % (1 << 31), ranks)
    return dict(rank_node=torch.from_numpy(node).to(DEV), node_rack=torch.from_numpy(rack).to(DEV),
                node_chassis=torch.from_numpy(chassis).to(DEV), n_racks=22, n_chassis=22 * 8)


def _wide_traces(case, seed):
    """Traces over a large tree: each rank works in a few hundred contexts that
    neighbouring ranks share."""
    c = case
    rng = np.random.default_rng([c["ranks"], c["events"], 4])
    lens = np.clip(np.rint(rng.lognormal(math.log(c["events"]), 1.0, c["ranks"])),
                   max(1, c["events"] // 20), 10 * c["events"]).astype(np.int64)
    offsets = np.zeros(c["ranks"] + 1, np.int64)
    np.cumsum(lens, out=offsets[1:])
    E = int(offsets[-1])
    off = torch.from_numpy(offsets).to(DEV)
    g = _gen(seed, 5)
    t = torch.cumsum(torch.empty(E, device=DEV).exponential_(1 / 20000.0, generator=g).round_()
                     .to(torch.int64), 0)
    rank = torch.repeat_interleave(torch.arange(c["ranks"], device=DEV),
                                   torch.from_numpy(lens).to(DEV))
    ts = (t - t[off[:-1]][rank]).contiguous()
    width = min(c["nodes"], 1500)
    base = torch.randint(0, c["nodes"], (c["ranks"] // 16 + 1,), device=DEV, generator=g)
    inside = torch.randint(0, width, (E,), device=DEV, generator=g)
    ctx = ((base[rank // 16] + inside * 61) % c["nodes"]).to(torch.int32)
    return dict(offsets=off, ts=ts, ctx=ctx.contiguous(), span=int(ts.max().item()) + 1)


def _groups(case, seed):
    """Region totals of ranks that fall into k overlapping groups."""
    g = _gen(seed, 6)
    R, D, k = case["ranks"], case["regions"], case["k"]
    mu = torch.exp(torch.empty(D, device=DEV, dtype=torch.float64).uniform_(16.0, 19.0, generator=g))
    lift = torch.rand((k, D), device=DEV, dtype=torch.float64, generator=g) * 0.25 + 1.0
    who = torch.randint(0, k, (R,), device=DEV, generator=g)
    X = mu * lift[who] * (1 + 0.08 * torch.randn((R, D), device=DEV, dtype=torch.float64, generator=g))
    X = X.clamp_(min=0).round_().to(torch.int64)
    init = X[torch.sort(torch.randperm(R, device=DEV, generator=g)[:k]).values].to(torch.float64)
    return X, init.contiguous()


def _weights(seed):
    """Xavier-uniform weights, small biases: W1 W2 W3 W4 b1 b2 b3 b4."""
    rng = np.random.default_rng([seed, 7])
    parts = []
    for o, i in ((128, 64), (32, 128), (128, 32), (64, 128)):
        parts.append(rng.uniform(-1, 1, o * i) * math.sqrt(6.0 / (o + i)))
    parts += [rng.uniform(-0.05, 0.05, n) for n in (128, 32, 128, 64)]
    return np.concatenate(parts).astype(np.float32)


def _with_weights(h, seed):
    """A checkpoint of `h`'s network with `_weights(seed)`, no moments."""
    h.ae_init(1)
    blob = bytearray(h.ae_get_state())
    tail = (3 * N_AE + 128) * 4
    blob[-tail:-tail + 4 * N_AE] = _weights(seed).tobytes()
    return bytes(blob)


# ---- one pass ------------------------------------------------------------------

def prepare(case, seed):
    c, kind = case, case["kind"]
    h = ta.Handle(0)
    s = dict(kind=kind)
    if kind in ("eager", "plan", "node_model", "pruned"):
        w = _traces(c, seed)
        h.set_tree(w["parent"])
        h.set_regions(w["marker"], w["regions"])
        tr = ta.DeviceTraces(w["offsets"], w["ts"], w["ctx"], DEV)
        s.update(h=h, tr=tr, iters=w["n_iters"], ragged=c.get("ragged", True))
    if kind == "plan":
        # a fixed launch shape: a tuned one may be another from plan to plan
        s["plan"] = h.plan(tr, w["n_iters"], w["offsets_host"], autotune=0)
        s["place"] = _placement(seed, c["ranks"])
    elif kind == "pruned":
        si = h.summary(h.attribute(tr, incl=False)[0])[1]
        # a node before its descendants, which cost no more and have larger ids
        kept = np.sort(np.argsort(-si.cpu().numpy(), kind="stable")[:KEPT]).astype(np.int32)
        h.set_regions(w["marker"], kept)
        h.set_pruned(kept)
        s["kept"] = (torch.zeros(c["nodes"], dtype=torch.int32, device=DEV),
                     torch.zeros(4, dtype=torch.int32, device=DEV))
    elif kind == "node_model":
        # entry arrays that a program keeps for runs of about this size
        E = _events(c)
        s["out"] = tuple(torch.zeros(int(n * E), dtype=t, device=DEV)
                         for n in (2, 9) for t in (torch.int32, torch.int64))
    elif kind == "batch":
        reqs = []
        for q in range(c["requests"]):
            w = _request_traces(c, seed, q)
            if q == 0:
                h.set_tree(w["parent"])
                h.set_regions(w["marker"], w["regions"])
            reqs.append((ta.DeviceTraces(w["offsets"], w["ts"], w["ctx"], DEV), w["offsets_host"],
                         w["n_iters"]))
        s.update(h=h, plan=h.mixed_batch(reqs, autotune=0))
    elif kind == "stats":
        T, it = _tensor(seed, c["ranks"], c["iters"], c["regions"])
        s.update(h=h, T=T, it=it, place=_placement(seed, c["ranks"]))
    elif kind == "window":
        w = _wide_traces(c, seed)
        h.set_tree(_deep_tree(c["nodes"]))
        tr = ta.DeviceTraces(w["offsets"], w["ts"], w["ctx"], DEV)
        E, span = tr.n_events, w["span"]
        out = (torch.zeros(c["ranks"], dtype=torch.int64, device=DEV),
               torch.zeros(E, dtype=torch.int32, device=DEV),
               torch.zeros(E, dtype=torch.int64, device=DEV))
        some = torch.arange(0, c["ranks"], 7, dtype=torch.int32, device=DEV)
        s.update(h=h, tr=tr, out=out, some=some, window=(span // 10, span // 10 + span // 20),
                 whole=(0, span))
    elif kind == "cluster":
        X, init = _groups(c, seed)
        tot = X.sum(1).contiguous()
        place = _placement(seed, c["ranks"])
        s.update(h=h, X=X, init=init, tot=tot, eps=int(tot.median().item()) // 2000 + 1,
                 rank_node=place["rank_node"], n_nodes=place["node_rack"].numel(), k=c["k"])
    elif kind in ("train", "prescreen"):
        T, it = _tensor(seed, c["ranks"], c["iters"], 64)
        h.ae_init(1)
        h.ae_fit_norm(T, it)
        s.update(h=h, state=_with_weights(h, seed))
        h.ae_set_state(s["state"])
        if kind == "train":
            s.update(rows=h.ae_rows(T, it), epochs=c["epochs"], batch=c["batch"])
        else:
            h.ae_set_score_kind(ta.AE_SCORE_RESIDUAL_Z)
            k = max(1, int(0.385 * c["ranks"]))
            h.ae_calibrate(h.ae_score(T, it), 1.0 - 0.9 * k / c["ranks"])
            s.update(T=T, it=it, k=k)
    h.sync_status()
    return s


def _topology(s, o):
    p = s["place"]
    return s["h"].topology(o["rank_score"], o["rank_flag"], p["rank_node"], p["node_rack"],
                           p["node_chassis"], p["n_racks"], p["n_chassis"])


def run(s):
    h, kind = s.get("h"), s["kind"]
    if kind == "eager":
        seg = h.attribute_segment(s["tr"], s["iters"])
        imb = h.imbalance(seg["tensor"], seg["iters_found"], seg["rank_sum"], seg["rank_sumsq"],
                          seg["span"])
        return dict(seg=seg, imb=imb, out=h.outliers(seg["tensor"], seg["iters_found"]))
    if kind == "plan":
        p = s["plan"]
        p.launch()
        return dict(seg=p.seg, imb=p.imb, out=p.out, topo=_topology(s, p.out))
    if kind == "batch":
        s["plan"].launch()
        return s["plan"].outs
    if kind == "stats":
        T, it = s["T"], s["it"]
        z = h.outliers(T, it, kind=ta.SCORE_Z, region=True)
        return dict(imb=h.imbalance(T, it), z=z, totals=h.outliers(T, it, mode=ta.SCAN_TOTALS),
                    topo=_topology(s, z))
    if kind == "node_model":
        # row starts (counted[0]) are not written for iterations that a rank does not have
        counted = h.node_model_count(s["tr"], s["iters"])
        n_x, n_i = int(counted[2][-1].item()), int(counted[3][-1].item())
        h.node_model_fill(s["tr"], s["iters"], counted, n_x, n_i, out=s["out"])
        return dict(counted=counted[1:], entries=s["out"])
    if kind == "window":
        sp = h.sparse_profiles(s["tr"], out=s["out"])
        return dict(sparse=sp, window=h.window_profile(s["tr"], *s["window"]),
                    some=h.window_profile(s["tr"], *s["whole"], ranks=s["some"]))
    if kind == "pruned":
        excl, _ = h.attribute(s["tr"], incl=False)
        se, si = h.summary(excl)
        kept = h.prune(se, si, 0.01, out=s["kept"])
        pe, pi = h.pruned_profiles(excl)
        T, it, outside = h.segment(s["tr"], s["iters"])
        return dict(sums=(se, si), kept=kept, profiles=(pe, pi), tensor=T, iters_found=it,
                    outside=outside, inclusive=h.tensor_inclusive(T))
    if kind == "cluster":
        labels, cent, counts, n = h.kmeans(s["X"], s["init"], 50)
        db = h.dbscan1d(s["tot"], s["eps"], 100)
        return dict(labels=labels, centroids=cent, counts=counts, n_iter=n, dbscan=db,
                    nodes=h.node_intersections(labels, s["rank_node"], s["n_nodes"], s["k"]))
    if kind == "train":
        h.ae_set_state(s["state"])
        grad, loss = h.ae_grad(s["rows"][:s["batch"]])
        el = h.ae_train(s["rows"], s["epochs"], batch=s["batch"], seed=5, noise=0.5)
        state = np.frombuffer(h.ae_get_state(), np.uint8)[-(3 * N_AE + 128) * 4:]
        return dict(grad=grad, loss=loss, epoch_loss=el, state=state.view(np.float32))
    top, score, fallback = h.prescreen(s["T"], s["it"], s["k"])
    return dict(top=top, score=score, fallback=fallback)


# ---- what a pass cannot do without -----------------------------------------------

def _mean_len(median, lo, hi):
    q = (np.arange(4096) + 0.5) / 4096
    x = torch.special.ndtri(torch.from_numpy(q)).numpy()
    return float(np.clip(np.exp(math.log(median) + x), lo, hi).mean())


def _events(c):
    if c["kind"] == "eager" or c.get("layout") == "plain":
        return 0.8 * c["ranks"] * c["events"]
    return c["ranks"] * _mean_len(c["events"], c["events"] // 20, 10 * c["events"])


def work(case):
    c, kind, R = case, case["kind"], case.get("ranks", 0)
    if kind in ("eager", "plan"):
        E, I, G, N = _events(c), c["iters"], c["regions"], c["nodes"]
        return dict(bytes=12 * E + 8 * R * I * G + 16 * R * N + 24 * R * G + 37 * R + 40 * I * G,
                    flops=0)
    if kind == "batch":
        b = 0
        for r, i in _requests(c):
            b += 12 * r * _mean_len(40 * i, 2 * i, 400 * i) + 8 * r * i * c["regions"]
            b += 24 * r * c["regions"] + 37 * r
        return dict(bytes=b, flops=0)
    if kind == "stats":
        cells = R * c["iters"] * c["regions"]
        return dict(bytes=8 * cells + 8 * R * c["regions"] + 40 * c["iters"] * c["regions"], flops=0)
    if kind == "node_model":
        E = _events(c)
        return dict(bytes=12 * E + 12 * 3.8 * E + 16 * R * c["iters"], flops=0)
    if kind == "window":
        E = _events(c)
        return dict(bytes=12 * E + 12 * min(E, 1500 * R) + 32 * c["nodes"], flops=0)
    if kind == "pruned":
        E, K = _events(c), KEPT
        return dict(bytes=12 * E + 16 * R * c["iters"] * K + 16 * R * K + 16 * c["nodes"], flops=0)
    if kind == "cluster":
        return dict(bytes=8 * R * c["regions"] + 29 * R, flops=3.0 * R * c["regions"] * c["k"])
    rows = R * c["iters"]
    if kind == "train":
        return dict(bytes=256 * rows, flops=147456.0 * (rows * c["epochs"] + c["batch"]))
    return dict(bytes=512 * rows + 8 * R, flops=49152.0 * rows)


# ---- the computed outputs in 64 bits ----------------------------------------------

def _node_regions(parent, regions):
    """The nearest region ancestor-or-self of every node, -1 for none."""
    reg = np.full(len(parent), -1, np.int64)
    reg[np.asarray(regions)] = np.arange(len(regions))
    for v in range(len(parent)):  # a parent's id is smaller than its children's
        if reg[v] < 0 and parent[v] >= 0:
            reg[v] = reg[parent[v]]
    return torch.from_numpy(reg).to(DEV)


def _tensor_of(w):
    """(T, iterations per rank, span) of traces, by one index_add per block of ranks."""
    off, R, I, G = w["offsets_host"], len(w["offsets_host"]) - 1, w["n_iters"], len(w["regions"])
    reg = _node_regions(w["parent"], w["regions"])
    T = torch.zeros(R * I * G, dtype=torch.int64, device=DEV)
    it = torch.zeros(R, dtype=torch.int64, device=DEV)
    a = 0
    while a < R:
        b = min(R, max(a + 1, int(np.searchsorted(off, off[a] + (1 << 26)))))
        e0, e1 = int(off[a]), int(off[b])
        o = w["offsets"][a:b + 1] - e0
        n = o[1:] - o[:-1]
        ts, ctx = w["ts"][e0:e1], w["ctx"][e0:e1].long()
        rank = torch.repeat_interleave(torch.arange(b - a, device=DEV), n)
        d = torch.zeros_like(ts)
        d[:-1] = ts[1:] - ts[:-1]
        d[o[1:][n > 0] - 1] = 0
        m = ctx == w["marker"]
        opens = m.clone()
        opens[1:] &= ~m[:-1] | (rank[1:] != rank[:-1])
        count = torch.cumsum(opens.long(), 0)
        before = torch.zeros(b - a, dtype=torch.int64, device=DEV)
        before[1:] = count[(o[1:-1] - 1).clamp(min=0)]
        i = count - before[rank] - 1
        g = reg[ctx]
        ok = (g >= 0) & (i >= 0) & (i < I)
        T.index_add_(0, (((a + rank) * I + i) * G + g)[ok], d[ok])
        it[a:b].index_add_(0, rank, opens.long())
        a = b
    span = w["ts"][w["offsets"][1:] - 1] - w["ts"][w["offsets"][:-1]]
    return T.view(R, I, G), it, span


def _mean(x, n):
    return x.sum(0) / n


def _exact_imbalance(T, it, span):
    R, I, G = T.shape
    it = it.long()
    cols = {k: torch.full((I, G), math.nan, dtype=torch.float64, device=DEV)
            for k in ("mean", "std", "max_minus_mean")}
    mx = torch.zeros((I, G), dtype=torch.float64, device=DEV)
    n = (it[:, None] > torch.arange(I, device=DEV)[None, :]).sum(0).double()
    step = max(1, (1 << 27) // (R * G))
    S = torch.zeros((R, G), dtype=torch.float64, device=DEV)
    for a in range(0, I, step):
        x = T[:, a:a + step].double()
        ok = (it[:, None] > torch.arange(a, min(I, a + step), device=DEV)[None, :])[:, :, None]
        S += (x * ok).sum(1)
        k = n[a:a + step, None]
        m = (x * ok).sum(0) / k
        cols["mean"][a:a + step] = m
        cols["std"][a:a + step] = ((((x - m) * ok) ** 2).sum(0) / (k - 1)).sqrt()
        mx[a:a + step] = torch.where(ok, x, -math.inf).amax(0)
        cols["max_minus_mean"][a:a + step] = mx[a:a + step] - m
    cols["std"][n <= 1] = math.nan
    has = n > 0
    o = dict(cols)
    o["avg_mean"] = cols["mean"][has].mean(0)
    o["avg_max"] = mx[has].mean(0)
    o["savings_per_iter"] = cols["max_minus_mean"][has].mean(0)
    o["total_savings"] = o["savings_per_iter"] * has.sum()
    o["balance_ratio"] = S.sum(0) / R / S.amax(0)
    good = has[:, None] & (n > 1)[:, None] & (cols["mean"] > 0)
    cv = torch.where(good, cols["std"] / cols["mean"], 0.0)
    o["cv_across"] = cv.sum(0) / good.sum(0)
    V = torch.zeros((R, G), dtype=torch.float64, device=DEV)
    nr = it.double()[:, None]
    for a in range(0, I, step):
        ok = (it[:, None] > torch.arange(a, min(I, a + step), device=DEV)[None, :])[:, :, None]
        V += (((T[:, a:a + step].double() - (S / nr)[:, None, :]) * ok) ** 2).sum(1)
    good = (nr > 1) & (S > 0)
    within = torch.where(good, (V / (nr - 1)).sqrt() / (S / nr), 0.0)
    o["cv_within"] = within.sum(0) / good.sum(0)
    o["share"] = S.sum(0) / S.sum()
    if span is not None:
        o["potential_speedup"] = (o["total_savings"].sum() / span.max().double()).reshape(1)
    else:
        o["potential_speedup"] = torch.full((1,), math.nan, dtype=torch.float64, device=DEV)
    return {k: o.get(k) for k in ta.IMB_FIELDS}


def _middle(sorted_rows, n):
    """Mean of the two middle values of each row's first n (n > 0)."""
    lo = sorted_rows.gather(1, ((n - 1) // 2)[:, None])[:, 0]
    hi = sorted_rows.gather(1, (n // 2)[:, None])[:, 0]
    return (lo + hi) / 2


def _robust(x, ok):
    """Robust z of each row's entries marked ok, 0 elsewhere."""
    n = ok.sum(1)
    x = torch.where(ok, x, math.inf)
    med = _middle(torch.sort(x, 1).values, n.clamp(min=1))
    dev = torch.where(ok, (x - med[:, None]).abs(), math.inf)
    mad = _middle(torch.sort(dev, 1).values, n.clamp(min=1))
    mean_dev = torch.where(ok, dev, 0.0).sum(1) / n
    scale = torch.where(mad > 0, ROBUST * mad, MEAN_DEV * mean_dev)
    z = torch.where(ok, x - med[:, None], 0.0) / scale[:, None]
    return torch.where((scale > 0)[:, None], z, torch.zeros_like(z))


def _plain_z(x, ok):
    n = ok.sum(1, keepdim=True)
    m = torch.where(ok, x, 0.0).sum(1, keepdim=True) / n
    v = torch.where(ok, (x - m) ** 2, 0.0).sum(1, keepdim=True) / (n - 1)
    z = torch.where(ok, (x - m) / v.sqrt(), 0.0)
    return torch.where(v > 0, z, torch.zeros_like(z))


def _exact_scores(T, it, z=_robust):
    R, I, G = T.shape
    m = torch.zeros((G, R), dtype=torch.float64, device=DEV)
    for i in range(I):
        ok = (it > i)[None, :].expand(G, R)
        m += z(T[:, i].double().t().contiguous(), ok)
    m /= it.clamp(min=1)
    z2 = z(m, (it > 0)[None, :].expand(G, R))
    return z2.abs().amax(0), z2.t().contiguous()


def _exact_topology(p, score):
    out = {}
    for name, place, k in (("rack", p["node_rack"], p["n_racks"]),
                           ("chassis", p["node_chassis"], p["n_chassis"])):
        at = place.long()[p["rank_node"].long()]
        n = torch.bincount(at, minlength=k).double()
        s = torch.zeros(k, dtype=torch.float64, device=DEV).index_add_(0, at, score)
        mx = torch.full((k,), -math.inf, dtype=torch.float64, device=DEV)
        mx.scatter_reduce_(0, at, score, "amax")
        out["flagged_" + name] = None
        out["max_" + name] = torch.where(n > 0, mx, math.nan)
        out["mean_" + name] = s / n
    return out


SEG = ("tensor", "iters_found", "outside", "span", "rank_sum", "rank_sumsq", "excl", "incl")


def _exact_out(score, region=None):
    return dict(rank_score=score, rank_flag=None, n_flagged=None, region_score=region)


def _forward(W, x):
    w1, w2, w3, w4 = W[:8192].view(128, 64), W[8192:12288].view(32, 128), \
        W[12288:16384].view(128, 32), W[16384:24576].view(64, 128)
    b1, b2, b3, b4 = W[24576:24704], W[24704:24736], W[24736:24864], W[24864:]
    y = torch.relu(x @ w1.t() + b1)
    y = torch.relu(y @ w2.t() + b2)
    y = torch.relu(y @ w3.t() + b3)
    return y @ w4.t() + b4


def _normalised(T, it):
    """Valid profile rows and the mask of the valid (rank, iteration) pairs."""
    ok = torch.arange(T.shape[1], device=DEV)[None, :] < it[:, None]
    x = T[ok].double()
    mu = x.mean(0)
    sd = ((x - mu) ** 2).mean(0).sqrt()
    return (x - mu) / sd, ok


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("eager", "plan"):
        w = _traces(c, seed)
        T, it, span = _tensor_of(w)
        del w
        # sorting the columns of the largest batches takes too long
        score = _exact_scores(T, it)[0] if T.numel() < 300_000_000 else None
        o = dict(seg=dict.fromkeys(SEG), imb=_exact_imbalance(T, it, span), out=_exact_out(score))
        if kind == "plan" and score is not None:
            o["topo"] = _exact_topology(_placement(seed, c["ranks"]), score)
        return o
    if kind == "batch":
        outs = []
        for q in range(c["requests"]):
            T, it, _ = _tensor_of(_request_traces(c, seed, q))
            outs.append(dict(rank_score=_exact_scores(T, it)[0]))
        return outs
    if kind == "stats":
        T, it = _tensor(seed, c["ranks"], c["iters"], c["regions"])
        score, region = _exact_scores(T, it, _plain_z)
        ok = torch.arange(c["iters"], device=DEV)[None, :, None] < it[:, None, None]
        S = (T * ok).sum(1).double().t().contiguous()
        totals = _robust(S, (it > 0)[None, :].expand_as(S)).abs().amax(0)
        return dict(imb=_exact_imbalance(T, it, None), z=_exact_out(score, region),
                    totals=_exact_out(totals),
                    topo=_exact_topology(_placement(seed, c["ranks"]), score))
    if kind == "cluster":
        X, cent = _groups(c, seed)
        x, old = X.double(), None
        for _ in range(50):
            d = torch.stack([((x - cent[j]) ** 2).sum(1) for j in range(c["k"])], 1)
            lab = d.argmin(1)
            n = torch.bincount(lab, minlength=c["k"])
            s = torch.zeros((c["k"], x.shape[1]), dtype=torch.int64, device=DEV).index_add_(0, lab, X)
            cent = torch.where((n > 0)[:, None], s.double() / n[:, None], cent)
            if old is not None and bool((lab == old).all()):
                break
            old = lab
        return dict(centroids=cent)
    if kind == "train":
        T, it = _tensor(seed, c["ranks"], c["iters"], 64)
        x = _normalised(T, it)[0][:c["batch"]]
        W = torch.from_numpy(_weights(seed)).to(DEV).double().requires_grad_()
        loss = ((_forward(W, x) - x) ** 2).mean()
        loss.backward()
        return dict(grad=W.grad, loss=loss.detach().reshape(1))
    if kind == "prescreen":
        T, it = _tensor(seed, c["ranks"], c["iters"], 64)
        x, ok = _normalised(T, it)
        W = torch.from_numpy(_weights(seed)).to(DEV).double()
        r = torch.cat([_forward(W, b) - b for b in x.split(1 << 18)])
        rank = torch.nonzero(ok)[:, 0]
        m = torch.zeros((c["ranks"], 64), dtype=torch.float64, device=DEV).index_add_(0, rank, r)
        m = (m / it.clamp(min=1)[:, None]).t().contiguous()
        return dict(score=_robust(m, (it > 0)[None, :].expand_as(m)).abs().amax(0))
    return None
