"""The node model at the edges of its row classes, of the row batches that a
wave takes, of its staging and of the boundary pass, against the oracle (bit
for bit)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nodes,deep", [(31, False), (32, True), (300, True), (8192, False),
                                        (8193, False), (131073, False)])
def test_row_and_rank_edges(oracle, nodes, deep):
    """Rows of 1, 2 and around 64, 128 and 512 events mixed in one rank (so a
    batch of rows holds every class), ranks of 0 and 1 events and around one and
    two steps of the boundary pass, starting at odd events; `deep` trees are one
    chain with leaves, whose rows have many more inclusive entries than are
    staged at once; every fourth event of some ranks lasts 0."""
    from paper_2605_03561_amd import synth, ta
    rng = np.random.default_rng([nodes, deep])
    if deep:
        chain = max(nodes * 3 // 4, 2)
        parent = np.empty(nodes, dtype=np.int32)
        parent[:chain] = np.arange(-1, chain - 1)
        parent[chain:] = rng.integers(chain // 2, chain, nodes - chain)
        marker = 1
    else:
        parent = synth.make_tree(rng, nodes, 8)
        marker = synth.pick_marker(rng, parent)
    inside = np.zeros(nodes, dtype=bool)
    for v in range(nodes):
        inside[v] = v == marker or (parent[v] >= 0 and inside[parent[v]])
    outs = np.flatnonzero(~inside)
    lens = [1, 2, 63, 64, 65, 127, 128, 129, 511, 512, 513, 700, 64, 1, 3]
    ranks = [lens, [], [1], [2, 1], lens[::-1], [8191], [8193, 5], [5, 8192, 4], [16384, 64],
             [1] * 40, [64] * 17 + [65] * 16 + [2]]
    off, ctx, ts = [0], [], []
    I = 48
    for k, rows in enumerate(ranks):
        for n in rows:  # a row ends with an event outside the marker's subtree
            c = rng.integers(0, nodes, n).astype(np.int32)
            c[inside[c]] = marker
            if n > 2:  # inside nodes without leaving: one boundary per row
                m = n // 2
                c[:m] = rng.choice(np.flatnonzero(inside), m)
                c[m:] = rng.choice(outs, n - m)
            c[0] = marker
            if n > 1:
                c[-1] = outs[rng.integers(len(outs))]
            ctx.append(c)
        n = sum(rows)
        d = rng.integers(1, 10**7, n)
        if k % 2:
            d[::4] = 0
        ts.append(10**9 + np.cumsum(d))
        off.append(off[-1] + n)
    off = np.array(off, dtype=np.int64)
    ctx = np.concatenate(ctx).astype(np.int32)
    ts = np.concatenate(ts).astype(np.int64)
    st, m = oracle.node_model(off, ts, ctx, parent, marker, I)
    assert st == 0
    h = ta.Handle(0)
    h.set_tree(parent)
    h.set_regions(marker, np.array([marker], dtype=np.int32))
    for _ in range(2):
        g = h.node_model(ta.DeviceTraces(off, ts, ctx), I)
        h.sync_status()
        for k in ("row_off_x", "row_off_i", "node_x", "val_x", "node_i", "val_i"):
            assert np.array_equal(g[k].cpu().numpy(), m[k]), k
    h.close()
