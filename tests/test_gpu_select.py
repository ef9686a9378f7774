"""Exact selections held in registers, at the edges of their launch shapes,
against the oracle (bit for bit: exact order statistics, then the same FP64
operations in the same order)."""
import numpy as np
import pytest

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


def tensor(rng, R, I, G):
    """Columns of every kind: spread, wide, signed, mostly zero, constant, and
    few distinct values; ranks without iterations and with fewer of them."""
    T = rng.integers(0, 10**6, (R, I, G)).astype(np.int64)
    T[..., 1 % G] = rng.integers(-2**59, 2**59, (R, I))
    T[..., 2 % G] *= rng.random((R, I)) < 0.3
    T[..., 3 % G] = 12345
    T[..., 4 % G] = rng.integers(0, 3, (R, I)) * 10**9
    it = np.where(rng.random(R) < 0.1, rng.integers(0, I + 1, R), I).astype(np.int32)
    it[0] = I
    return T, it


@pytest.mark.parametrize("R", [1, 2, 64, 65, 256, 257, 1024, 1025, 2047, 4096, 4097, 8192, 8193,
                               16384, 16385, 32768, 32769])
def test_region_selection_edges(ta, h, oracle, R):
    """Both modes at the rank counts where the number of waves or keys per lane
    changes, and on both sides of the passes over memory."""
    import torch
    T, it = tensor(np.random.default_rng([R, 1]), R, 3, 5)
    for mode in (ta.SCAN_TOTALS, ta.SCAN_FULL):
        o = h.outliers(torch.from_numpy(T).cuda(), torch.from_numpy(it).cuda(), mode=mode, region=True)
        st, score, flag, nf, reg = oracle.outliers(T, it, mode=mode)
        assert st == 0
        assert np.array_equal(o["region_score"].cpu().numpy(), reg)
        assert np.array_equal(o["rank_score"].cpu().numpy(), score)
        assert np.array_equal(o["rank_flag"].cpu().numpy(), flag)
        assert int(o["n_flagged"].item()) == nf
