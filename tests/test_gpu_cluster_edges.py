"""K-Means at the edges of its launch paths, against the oracle (bit for bit)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,K", [(1, 1), (64, 8), (64, 9), (63, 8), (128, 8), (129, 8), (32, 32), (33, 32), (176, 32)])
@pytest.mark.parametrize("R", [0, 1, 257, 5000])
def test_kmeans_update_paths(oracle, D, K, R):
    """Numbers of sums up to and above the one where each workgroup takes the
    centroids itself; one iteration, two, three (each array of sums is reused
    from the fourth on), enough to converge and far more; clusters that stay
    empty (a far centroid) and ones that lose their rows; several calls on one
    handle."""
    import torch

    from paper_2605_03561_amd import ta
    rng = np.random.default_rng([R, D, K])
    X = (rng.integers(0, 6, (max(R, 1), 1)) * 10**5 + rng.integers(0, 10**5, (max(R, 1), D))).astype(np.int64)[:R]
    C0 = rng.integers(0, 7 * 10**5, (K, D)).astype(np.float64)
    if K > 2:
        C0[1] = 1e12
    h = ta.Handle(0)
    dX = torch.from_numpy(X).cuda()
    for max_iter in (1, 2, 3, 4, 5, 60, 60):
        st, lab, Cc, cnt, it = oracle.kmeans(X, C0, max_iter)
        assert st == 0
        gl, gc, gn, gi = h.kmeans(dX, torch.from_numpy(C0).cuda(), max_iter)
        assert np.array_equal(gl.cpu().numpy(), lab)
        assert np.array_equal(gc.cpu().numpy(), Cc)
        assert np.array_equal(gn.cpu().numpy(), cnt)
        assert int(gi.item()) == it
    h.close()
