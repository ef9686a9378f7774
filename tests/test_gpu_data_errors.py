"""The fused pass's outputs when the traces hold a data error: what a rank
still gets beside the sticky status."""
import numpy as np
import pytest

from paper_2605_03561_amd import synth

pytestmark = pytest.mark.gpu


def _traces(rng, N, G, lens, every):
    parent = synth.make_tree(rng, N, 6)
    marker = synth.pick_marker(rng, parent)
    regions = synth.pick_regions(rng, parent, marker, G)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ts, ctx = [], []
    for n in lens:
        ts.append(10**6 + np.cumsum(rng.integers(0, 5000, n)))
        c = rng.integers(0, N, n)
        c[c == marker] = (marker + 1) % N
        c[np.arange(n) % every == every // 2] = marker
        ctx.append(c)
    return (parent, marker, regions, off, np.concatenate(ts).astype(np.int64),
            np.concatenate(ctx).astype(np.int32))


@pytest.mark.parametrize("every", [2, 7, 300])
def test_outside_when_iterations_overflow(oracle, every):
    """Ranks with more iterations than the tensor holds, and others without:
    time in a region of an iteration that is not stored is neither in a cell nor
    outside (as in the oracle), eager, in segmentation alone and in a plan, on
    two calls (nothing is left over from one to the next)."""
    from paper_2605_03561_amd import ta
    rng = np.random.default_rng(every)
    lens = [5, 9000, 0, 1, 2 * every, 20000, 2048, 6145, 30]
    parent, marker, regions, off, ts, ctx = _traces(rng, 60, 5, lens, every)
    I = 3
    st, T, it, outside, span = oracle.segment(off, ts, ctx, parent, marker, regions, I)
    assert st != 0 and (it > I).any() and (it <= I).any()
    h = ta.Handle(0)
    h.set_tree(parent)
    h.set_regions(marker, regions)
    tr = ta.DeviceTraces(off, ts, ctx)
    p = h.plan(tr, I, off, imbalance=False, outliers=False, autotune=0)
    for _ in range(2):
        p.launch()
        T2, it2, out2 = h.segment(tr, I)
        g = h.attribute_segment(tr, I)
        for o in (p.seg, g, dict(tensor=T2, iters_found=it2, outside=out2)):
            assert np.array_equal(o["tensor"].cpu().numpy(), T)
            assert np.array_equal(o["iters_found"].cpu().numpy(), it)
            assert np.array_equal(o["outside"].cpu().numpy(), outside)
        with pytest.raises(ta.TAError) as ei:
            h.sync_status()
        assert ei.value.status == ta.ITER_OVERFLOW
    p.close()
    h.close()


@pytest.mark.parametrize("bad", [60, 2**31 - 1, -1])
def test_context_out_of_range(oracle, bad):
    """A context outside [0, N), also in tiles that lie inside a rank, on both
    sides of a boundary and as the last event of a tile: the event is in no
    region and not in the marker's subtree, as if it were in the tree's root,
    which is neither here."""
    from paper_2605_03561_amd import ta
    rng = np.random.default_rng([3, bad & 0xffff])
    N, lens, every = 60, [5, 9000, 0, 1, 20000, 2048, 6145], 50
    parent, marker, regions, off, ts, ctx = _traces(rng, N, 5, lens, every)
    assert parent[0] == -1 and marker != 0 and 0 not in regions
    at = rng.random(len(ctx)) < 0.02
    at[off[1] + every // 2 - 1::every * 7] = True
    at[off[1] + every // 2 + 1::every * 11] = True
    at[4095] = at[8191] = at[8192] = True
    fixed, ctx = np.where(at, 0, ctx).astype(np.int32), np.where(at, bad, ctx).astype(np.int32)
    I = 500
    st, T, it, outside, span = oracle.segment(off, ts, fixed, parent, marker, regions, I)
    assert st == 0
    st, ex, inc = oracle.attribute(off, ts, fixed, parent)
    assert st == 0
    h = ta.Handle(0)
    h.set_tree(parent)
    h.set_regions(marker, regions)
    tr = ta.DeviceTraces(off, ts, ctx)
    p = h.plan(tr, I, off, imbalance=False, outliers=False, autotune=0)
    p.launch()
    for o in (p.seg, h.attribute_segment(tr, I)):
        for k, ref in (("tensor", T), ("iters_found", it), ("outside", outside), ("span", span),
                       ("excl", ex), ("incl", inc)):
            assert np.array_equal(o[k].cpu().numpy(), ref), k
    with pytest.raises(ta.TAError) as ei:
        h.sync_status()
    assert ei.value.status == ta.CTX_RANGE
    p.close()
    h.close()
