"""The fused pass at the edges of its tiles, waves and ring windows, against
the oracle (bit for bit)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("every", [1, 3, 64, 256, 1000])
@pytest.mark.parametrize("gap", [3, 2**31])
def test_tile_and_window_edges(oracle, every, gap):
    """Ranks of 0, 1, 2 and around one, two and three tiles of 2,048 events,
    placed one after the other so that tiles start inside ranks; a marker every
    `every` events (so a tile holds from 2,048 iterations, many ring windows, to
    two), also as the first event, the last one and on both sides of a wave's and
    a tile's edge; gaps that make cells below and above 2^32; repeated timestamps."""
    import torch

    from paper_2605_03561_amd import synth, ta
    rng = np.random.default_rng([every, gap])
    N, G = 60, 5
    parent = synth.make_tree(rng, N, 6)
    marker = synth.pick_marker(rng, parent)
    regions = synth.pick_regions(rng, parent, marker, G)
    lens = np.array([0, 1, 2, 255, 256, 257, 2047, 2048, 2049, 1, 4095, 4097, 6144, 0, 6145, 300])
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ts, ctx = [], []
    for k, n in enumerate(lens):
        d = rng.integers(0, gap, n) * (rng.random(n) < 0.8)
        ts.append(10**6 + np.cumsum(d))
        c = rng.integers(0, N, n)
        c[c == marker] = (marker + 1) % N
        c[np.arange(n) % every == (k % 2) * (every // 2)] = marker
        if n > 2 and k % 3 == 0:
            c[-1] = marker
        ctx.append(c)
    ts = np.concatenate(ts).astype(np.int64)
    ctx = np.concatenate(ctx).astype(np.int32)
    I = 3100
    st, T, it, outside, span = oracle.segment(off, ts, ctx, parent, marker, regions, I)
    assert st == 0
    st, ex, inc = oracle.attribute(off, ts, ctx, parent)
    assert st == 0
    h = ta.Handle(0)
    h.set_tree(parent)
    h.set_regions(marker, regions)
    tr = ta.DeviceTraces(off, ts, ctx)
    p = h.plan(tr, I, off, imbalance=False, outliers=False, autotune=0)
    p.launch()
    T2, it2, out2 = h.segment(tr, I)
    for g in (h.attribute_segment(tr, I), p.seg):
        h.sync_status()
        g = {k: v.cpu().numpy() for k, v in g.items()}
        assert np.array_equal(g["iters_found"], it)
        assert np.array_equal(g["tensor"], T)
        assert np.array_equal(g["outside"], outside)
        assert np.array_equal(g["span"], span)
        assert np.array_equal(g["excl"], ex)
        assert np.array_equal(g["incl"], inc)
        assert np.array_equal(g["rank_sum"], T.sum(1))
        q = g["rank_sumsq"].astype(np.uint64).astype(object)
        assert np.array_equal(q[..., 0] + q[..., 1] * 2**64, (T.astype(object) ** 2).sum(1))
    assert np.array_equal(T2.cpu().numpy(), T) and np.array_equal(it2.cpu().numpy(), it)
    assert np.array_equal(out2.cpu().numpy(), outside)
    p.close()
    h.close()
