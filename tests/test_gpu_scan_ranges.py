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
