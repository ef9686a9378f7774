"""Time windows over the range of events per rank: the forms that the division
of the work takes, against the oracle, and a short window's cost."""
import numpy as np
import pytest

from paper_2605_03561_amd import synth

pytestmark = pytest.mark.gpu


def traces(rng, lens, nodes, width=1500):
    """Ranks of the given lengths; 16 neighbouring ones share `width` nodes."""
    lens = np.asarray(lens, np.int64)
    off = np.concatenate([[0], np.cumsum(lens)])
    E = int(off[-1])
    ts = np.cumsum(rng.integers(0, 2000, E))
    rank = np.repeat(np.arange(len(lens)), lens)
    ts -= ts[off[:-1].clip(max=E - 1)][rank]
    base = rng.integers(0, nodes, len(lens) // 16 + 1)
    ctx = (base[rank // 16] + rng.integers(0, min(width, nodes), E) * 61) % nodes
    return off, ts, ctx.astype(np.int32)


LENGTHS = {
    "two events": [2] * 9000,                         # a wave per rank
    "500": [500] * 40, "513": [513] * 40,             # around a wave per rank
    "short and long": [30] * 3000 + [70000],          # split, no table
    "table": [2100] * 260, "below it": [2000] * 260,  # around the table
    "table, many ranks": [2100] * 8193,
    "skew": [0] * 4000 + [40000] * 20 + [3] * 4000 + [200000],
}


@pytest.mark.parametrize("nodes", [5000, 8192, 97833])
@pytest.mark.parametrize("lens", LENGTHS.values(), ids=LENGTHS.keys())
def test_division_of_the_events(oracle, nodes, lens):
    """Whole traces, one moment, and a part; all ranks, and repeated ones."""
    import torch

    from paper_2605_03561_amd import ta
    rng = np.random.default_rng([nodes, len(lens)])
    if nodes == 5000 and len(lens) == 8193:
        lens = lens[:8193:3]
    off, ts, ctx = traces(rng, lens, nodes, nodes if nodes > 8192 and len(lens) == 260 else 1500)
    parent = synth.make_tree(rng, nodes, 12)
    h = ta.Handle(0)
    h.set_tree(parent)
    tr = ta.DeviceTraces(off, ts, ctx)
    sel = rng.integers(0, len(lens), 50).astype(np.int32)
    hi = int(ts.max())
    for a, b in [(-1, hi + 1), (hi // 3, hi // 3 + 1), (100, hi // 2)]:
        for ids in (None, sel):
            st, ex, inc = oracle.window_profile(off, ts, ctx, parent, a, b, ranks=ids)
            assert st == 0
            d = None if ids is None else torch.from_numpy(ids).cuda()
            ge, gi = h.window_profile(tr, a, b, ranks=d)
            assert np.array_equal(ge.cpu().numpy(), ex)
            assert np.array_equal(gi.cpu().numpy(), inc)
    h.sync_status()
    h.close()


def best_time(f, n=7):
    import torch
    f()
    t = []
    for _ in range(n):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        torch.cuda.synchronize()
        t.append(a.elapsed_time(b))
    return min(t)


@pytest.mark.parametrize("nodes", [5000, 97833])
def test_short_window_costs_less_than_the_whole(nodes):
    """Two events of each of 8,000 ranks against all 2,000 of them: a thousandth
    of the work."""
    from paper_2605_03561_amd import ta
    rng = np.random.default_rng(nodes)
    off, ts, ctx = traces(rng, [2000] * 8000, nodes)
    h = ta.Handle(0)
    h.set_tree(synth.make_tree(rng, nodes, 12))
    tr = ta.DeviceTraces(off, ts, ctx)
    whole = best_time(lambda: h.window_profile(tr, -1, 10**9))
    short = best_time(lambda: h.window_profile(tr, 10**6, 10**6 + 2000))
    print(f"whole {whole * 1e3:.0f} us, short {short * 1e3:.0f} us")
    assert short < whole
    h.close()


@pytest.mark.parametrize("nodes", [5000, 97833, 131073])
@pytest.mark.parametrize("reach", [300, 4096, 5000, 97833])
def test_sparse_profiles_by_reach(oracle, nodes, reach):
    """Sparse profiles of ranks that reach few nodes, the most that one pass
    holds and more, with ranks above and below a workgroup's step on average."""
    from paper_2605_03561_amd import ta
    rng = np.random.default_rng([nodes, reach])
    parent = synth.make_tree(rng, nodes, 12)
    for lens in ([20000, 3, 0, 12000, 4097], [30, 4000, 0, 1, 700] * 8):
        off, ts, ctx = traces(rng, lens, nodes, reach)
        h = ta.Handle(0)
        h.set_tree(parent)
        tr = ta.DeviceTraces(off, ts, ctx)
        st, cnt, ids, ex = oracle.sparse_profiles(off, ts, ctx, nodes)
        assert st == 0
        g = [x.cpu().numpy() for x in h.sparse_profiles(tr)]
        assert np.array_equal(g[0][:len(lens)], cnt)
        for r in range(len(lens)):
            s = slice(off[r], off[r] + cnt[r])
            assert np.array_equal(g[1][s], ids[s]) and np.array_equal(g[2][s], ex[s])
        h.sync_status()
        h.close()


def test_many_nodes_cost_no_second_attempt():
    """Ranks of 20,000 events that reach up to 4,000 nodes (which one pass holds)
    against 300: the same passes over the events, so well below twice the time."""
    import torch

    from paper_2605_03561_amd import ta
    nodes, R, n = 97833, 300, 20000
    rng = np.random.default_rng(1)
    parent = synth.make_tree(rng, nodes, 12)
    t = []
    for width in (300, 4000):
        off, ts, ctx = traces(rng, [n] * R, nodes, width)
        h = ta.Handle(0)
        h.set_tree(parent)
        tr = ta.DeviceTraces(off, ts, ctx)
        out = (torch.zeros(R, dtype=torch.int64, device="cuda"),
               torch.zeros(R * n, dtype=torch.int32, device="cuda"),
               torch.zeros(R * n, dtype=torch.int64, device="cuda"))
        t.append(best_time(lambda: h.sparse_profiles(tr, out=out)))
        h.close()
    print(f"300 nodes {t[0] * 1e3:.0f} us, 4,000 nodes {t[1] * 1e3:.0f} us")
    assert t[1] < 2 * t[0]
