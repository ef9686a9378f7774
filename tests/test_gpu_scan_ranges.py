"""The exact scan and the column statistics over ranges of cells and ranks that
the other tests do not reach, against the oracle."""
import numpy as np
import pytest

from paper_2605_03561_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ta():
    from paper_2605_03561_amd import ta as T
    return T


@pytest.fixture(scope="module")
def h(ta):
    hh = ta.Handle(0)
    yield hh
    hh.close()


def cells_as_traces(cells, parent, marker, region):
    """Traces whose tensor is `cells` [R, I] of one region: per iteration the
    marker for 10 ns and the region for the cell's time."""
    R, I = cells.shape
    d = np.zeros((R, I, 2), np.int64)
    d[..., 0], d[..., 1] = 10, cells
    t = np.zeros((R, 2 * I + 1), np.int64)
    np.cumsum(d.reshape(R, -1), axis=1, out=t[:, 1:])
    c = np.empty((R, 2 * I + 1), np.int32)
    c[:, 0:-1:2], c[:, 1::2], c[:, -1] = marker, region, region
    off = np.arange(R + 1, dtype=np.int64) * (2 * I + 1)
    return off, t.reshape(-1), c.reshape(-1)


def same_imbalance(got, ref):
    for k in ("min", "max"):
        assert np.array_equal(got[k].cpu().numpy(), ref[k]), k
    for k in ("mean", "std", "max_minus_mean"):
        np.testing.assert_allclose(got[k].cpu().numpy(), ref[k], rtol=1e-12, atol=0)


@pytest.mark.parametrize("R", [1500, 2305])
def test_column_offsets_at_the_limits(ta, h, oracle, R):
    """A plan's column sums from 32-bit offsets (up to 2^29 from the first rank's
    cell; beyond, cell by cell): columns whose offsets reach 2^29 and 2^31 from
    below, at and from above, to either side.  Exact sums: one rounding each."""
    parent = np.array([-1, 0, 0, 0], np.int32)
    marker, region = 1, 2
    lims = [2**29 - 1, 2**29, 2**29 + 1, 2**30, 2**31 - 2, 2**31 - 1, 2**31, 2**31 + 1, 2**33]
    rng = np.random.default_rng(R)
    cells = np.empty((R, 2 * len(lims)), np.int64)
    for i, x in enumerate(lims):
        cells[:, 2 * i] = rng.integers(0, x + 1, R)
        cells[:, 2 * i + 1] = x - rng.integers(0, x + 1, R)
        cells[0, 2 * i], cells[R // 2, 2 * i] = 0, x
        cells[0, 2 * i + 1], cells[R - 1, 2 * i + 1] = x, 0
    off, ts, ctx = cells_as_traces(cells, parent, marker, region)
    h.set_tree(parent)
    h.set_regions(marker, [region])
    p = h.plan(ta.DeviceTraces(off, ts, ctx), cells.shape[1], off, autotune=0, region=True)
    p.launch()
    h.sync_status()
    T = p.seg["tensor"].cpu().numpy()
    assert np.array_equal(T[..., 0], cells)
    it = np.full(R, cells.shape[1], np.int32)
    same_imbalance(p.imb, oracle.imbalance(T, it)[1])
    st, score, flag, nf, reg = oracle.outliers(T, it)
    assert st == 0
    assert np.array_equal(p.out["region_score"].cpu().numpy(), reg)
    assert np.array_equal(p.out["rank_score"].cpu().numpy(), score)
    p.close()


def far_columns(rng, R):
    """Columns with cells 2^31 and further from the first rank's: none, one, and
    shares around a half, above, below and on both sides; the first rank itself
    far; keys spread over nearly 2^31, so that the MAD comes near the far cells;
    mostly equal cells (a MAD of 0); cells spread over 2^33 and 2^45."""
    cols = []
    def col(x, share, up):
        x = x.copy()
        m = rng.random(R) < share
        m[0] = False
        if share < 0:
            m[:] = False
            m[R // 3] = True
        x[m] += np.where(up if np.ndim(up) else np.full(R, up), 1, -1)[m] * (
            2**31 + rng.integers(0, 2**40, R)[m])
        cols.append(x)
    base = 3 * 10**12 + rng.integers(0, 10**6, R)
    both = rng.random(R) < 0.5
    for share in (0.0, -1, 0.02, 0.24, 0.26, 0.49, 0.5, 0.51, 0.9):
        for up in (True, False, both):
            col(base, share, up)
    edge = 3 * 10**12 + rng.integers(-2**30 + 2, 2**30, R)
    edge[0] = 3 * 10**12
    for share in (0.0, -1, 0.1, 0.4):
        for up in (True, False, both):
            col(edge, share, up)
    flat = np.where(rng.random(R) < 0.8, 3 * 10**12, base)
    flat[0] = 3 * 10**12
    for share in (-1, 0.1, 0.3):
        col(flat, share, both)
    x = base.copy()
    x[0] += 2**40
    cols.append(x)
    cols.append(3 * 10**12 + rng.integers(0, 2**33, R))
    cols.append(rng.integers(-2**44, 2**44, R))
    # offsets of exactly the limits
    lim = np.array([0, 1, -1, 2**31 - 2, 2**31 - 1, 2**31, -2**31 + 2, -2**31 + 1, -2**31])
    x = 3 * 10**12 + lim[rng.integers(0, len(lim), R)]
    x[0] = 3 * 10**12
    cols.append(x)
    return np.stack(cols, axis=1)


@pytest.mark.parametrize("R", [1025, 1026, 2049, 3073, 4100, 5121, 6200, 9999, 13000, 17001, 21000, 33001, 41000])
def test_far_cells(ta, h, oracle, R):
    """The robust scan over columns with far cells, at every launch shape of the
    column selection, an odd and an even row length, ranks that end early:
    medians, deviations and scores as the oracle's, bit for bit."""
    import torch
    rng = np.random.default_rng(R)
    cells = far_columns(rng, R)
    n = cells.shape[1]
    I = n + n % 2 + R % 2
    T = np.zeros((R, I, 1), np.int64)
    T[:, :n, 0] = cells
    it = np.where(rng.random(R) < 0.15, rng.integers(0, I + 1, R), I).astype(np.int32)
    for have in (it, np.full(R, I, np.int32)):
        o = h.outliers(torch.from_numpy(T).cuda(), torch.from_numpy(have).cuda(), region=True)
        st, score, flag, nf, reg = oracle.outliers(T, have)
        assert st == 0
        assert np.array_equal(o["region_score"].cpu().numpy(), reg)
        assert np.array_equal(o["rank_score"].cpu().numpy(), score)
        assert np.array_equal(o["rank_flag"].cpu().numpy(), flag)


@pytest.mark.parametrize("R", [1025, 2050, 4100, 9999, 17001, 33001, 41000])
def test_far_cells_of_larger_tensors(ta, h, oracle, R):
    """The same columns in as many regions as make 2^23 cells, from where on wide
    columns are copied in two halves; ranks that end early."""
    import torch
    rng = np.random.default_rng([R, 2])
    cells = far_columns(rng, R)
    I = cells.shape[1]
    G = 2**23 // (R * I) + 2
    T = np.repeat(cells[:, :, None], G, axis=2) + rng.integers(0, 1000, (1, I, G))
    it = np.where(rng.random(R) < 0.15, rng.integers(0, I + 1, R), I).astype(np.int32)
    it[0] = I
    o = h.outliers(torch.from_numpy(T).cuda(), torch.from_numpy(it).cuda(), region=True)
    st, score, flag, nf, reg = oracle.outliers(T, it)
    assert st == 0
    assert np.array_equal(o["region_score"].cpu().numpy(), reg)
    assert np.array_equal(o["rank_score"].cpu().numpy(), score)
    assert np.array_equal(o["rank_flag"].cpu().numpy(), flag)


def best_time(f, n=9):
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


@pytest.mark.parametrize("R,I,G", [(4000, 100, 32), (16000, 60, 64), (40000, 40, 64)])
def test_far_cells_cost(ta, h, R, I, G):
    """The same scan with one rank far off in every cell, one region spread over
    2^33 and every cell spread: at most 2, 2.5 and 4 times the time of near cells
    (8-byte cells by the line would be 16 times the bytes)."""
    import torch
    rng = np.random.default_rng(R)
    T = torch.from_numpy(rng.integers(0, 2 * 10**5, (R, I, G))).cuda()
    t = []
    for case in ("near", "rank", "region", "spread"):
        x = T.clone()
        if case == "rank":
            x[R // 3] += 5 * 10**9
        elif case == "region":
            x[:, :, G // 3] *= 50000
        elif case == "spread":
            x *= 50000
        t.append(best_time(lambda: h.outliers(x)) * 1e3)
    print(R, " ".join(f"{v:.0f}" for v in t), "us")
    assert t[1] < 2 * t[0] and t[2] < 2.5 * t[0] and t[3] < 4 * t[0]


def test_wide_columns_of_a_large_tensor(ta, h, oracle):
    """Beyond 2^33 cells there are no high words for wide columns: they are read
    from the tensor.  3,300 equal iterations of 64 regions, one of them wide and one
    with far cells: a mean over equal scores, so the score of one iteration up to
    the rounding of 3,300 additions (3,300 * 2^-53 relative, below 1e-12)."""
    import torch
    R, I, G = 41000, 3300, 64
    if torch.cuda.mem_get_info()[0] < 140 << 30:
        pytest.skip("needs 140 GB of device memory")
    rng = np.random.default_rng(9)
    one = rng.integers(0, 10**6, (R, 1, G))
    one[:, 0, 5] = rng.integers(0, 2**34, R)
    one[rng.choice(R, 40, replace=False), 0, 7] += 2**35
    h2 = ta.Handle(0)
    T = torch.empty((R, I, G), dtype=torch.int64, device="cuda")
    T[:] = torch.from_numpy(one).cuda()
    o = h2.outliers(T, region=True)
    torch.cuda.synchronize()
    reg, score = o["region_score"].cpu().numpy(), o["rank_score"].cpu().numpy()
    del T, o
    h2.close()
    torch.cuda.empty_cache()
    st, ref, flag, nf, rref = oracle.outliers(one, np.full(R, 1, np.int32))
    assert st == 0
    np.testing.assert_allclose(reg, rref, rtol=1e-12, atol=1e-12)
    np.testing.assert_allclose(score, ref, rtol=1e-12, atol=1e-12)
