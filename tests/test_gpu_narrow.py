"""Statistics of tensors with few cells per rank: the forms that a thread per
region, a wave and a workgroup per rank take, against the oracle, and their cost."""
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


def tensor(rng, R, I, G):
    T = rng.integers(0, 10**6, (R, I, G))
    T[:, :, 1 % G] = rng.integers(-2**42, 2**42, (R, I))  # sums of deviations below 2^62
    T[:, I // 2] *= rng.random((R, G)) < 0.5
    it = np.where(rng.random(R) < 0.2, rng.integers(0, I + 1, R), I).astype(np.int32)
    return T.astype(np.int64), it


SHAPES = [(1, 1), (1, 63), (1, 64), (2, 5), (4, 63), (7, 3), (8, 32), (9, 29), (16, 16), (31, 8),
          (32, 8), (32, 9), (33, 7), (33, 1), (3, 128), (1, 129), (2, 100)]


@pytest.mark.parametrize("R", [1, 3, 255, 4097, 20001])
@pytest.mark.parametrize("I,G", SHAPES)
def test_rank_sums(ta, h, oracle, R, I, G):
    """Totals and imbalance where the number of threads per rank changes; sums of
    integers, so the totals' scan is the oracle's bit for bit."""
    import torch
    T, it = tensor(np.random.default_rng([R, I, G]), R, I, G)
    dT, dit = torch.from_numpy(T).cuda(), torch.from_numpy(it).cuda()
    o = h.outliers(dT, dit, mode=ta.SCAN_TOTALS, region=True)
    st, score, flag, nf, reg = oracle.outliers(T, it, mode=1)
    assert st == 0
    assert np.array_equal(o["region_score"].cpu().numpy(), reg)
    assert np.array_equal(o["rank_flag"].cpu().numpy(), flag)
    g = h.imbalance(dT, dit)
    _, ref = oracle.imbalance(T, it)
    for k in ("min", "max"):
        assert np.array_equal(g[k].cpu().numpy(), ref[k])
    for k in ("mean", "std", "max_minus_mean", "cv_across", "cv_within"):
        np.testing.assert_allclose(g[k].cpu().numpy(), ref[k], rtol=1e-12, atol=1e-9)


def test_sums_of_single_cells_cost(ta, h):
    """Rank sums of 2,000,000 ranks of one cell: an imbalance without them against
    one with the sums in hand.  The sums read 16 MB and write 48; a wave per rank
    made the call more than half as long again as it is with a thread."""
    import torch
    R = 2_000_000
    T = torch.randint(0, 10**6, (R, 1, 1), device="cuda")
    s = T.sum(1)
    q = torch.zeros((R, 1, 2), dtype=torch.int64, device="cuda")
    q[..., 0] = (T * T).sum(1)
    without = best_time(lambda: h.imbalance(T)) * 1e3
    given = best_time(lambda: h.imbalance(T, rank_sum=s, rank_sumsq=q)) * 1e3
    print(f"without {without:.0f} us, given {given:.0f} us")
    assert without < 1.5 * given


@pytest.mark.parametrize("R", [1, 2, 63, 64, 4099, 20001])
@pytest.mark.parametrize("I,G", SHAPES + [(128, 1), (129, 1), (25, 5), (43, 3)])
def test_plain_scores(ta, h, oracle, R, I, G):
    """The plain scan where its column sums take several ranks' rows side by side
    and its scores a thread per region.  Column sums are exact; a region's second
    stage adds R scores in another order than the oracle: within R * 2^-53 of the
    largest of them."""
    import torch
    T, it = tensor(np.random.default_rng([R, I, G, 1]), R, I, G)
    dT, dit = torch.from_numpy(T).cuda(), torch.from_numpy(it).cuda()
    for have, dh in ((it, dit), (np.full(R, I, np.int32), None)):
        o = h.outliers(dT, dh, kind=ta.SCORE_Z, region=True)
        st, score, flag, nf, reg = oracle.outliers(T, have, kind=1)
        assert st == 0
        tol = max(R, 64) * 2.0**-53 * max(1.0, float(np.abs(reg).max()))
        np.testing.assert_allclose(o["region_score"].cpu().numpy(), reg, rtol=1e-12, atol=tol)
        np.testing.assert_allclose(o["rank_score"].cpu().numpy(), score, rtol=1e-12, atol=tol)
        near = np.abs(score - 3.5) < 1e-9
        assert np.array_equal(o["rank_flag"].cpu().numpy()[~near], flag[~near])
        assert abs(int(o["n_flagged"].item()) - nf) <= near.sum()


@pytest.mark.parametrize("R,I,G", [(300, 40, 5), (20000, 3, 7), (5000, 30, 16), (70000, 2, 3)])
def test_plain_plan(ta, h, oracle, R, I, G):
    """A plan's plain scan, whose column sums the imbalance shares."""
    from paper_2605_03561_amd import synth
    w = synth.plain_workload(seed=R, n_ranks=R, events=4 * I, n_nodes=60, n_iters=I, n_regions=G,
                             mean_gap_ns=3000.0)
    h.set_tree(w.parent)
    h.set_regions(w.marker, w.regions)
    p = h.plan(ta.DeviceTraces(w.offsets, w.ts, w.ctx), I, w.offsets, autotune=0, region=True,
               kind=ta.SCORE_Z)
    for _ in range(2):
        p.launch()
    h.sync_status()
    T, it = p.seg["tensor"].cpu().numpy(), p.seg["iters_found"].cpu().numpy()
    st, score, flag, nf, reg = oracle.outliers(T, it, kind=1)
    assert st == 0
    tol = R * 2.0**-53 * max(1.0, float(np.abs(reg).max()))
    np.testing.assert_allclose(p.out["region_score"].cpu().numpy(), reg, rtol=1e-12, atol=tol)
    _, ref = oracle.imbalance(T, it, span=p.seg["span"].cpu().numpy())
    for k in ("min", "max"):
        assert np.array_equal(p.imb[k].cpu().numpy(), ref[k])
    for k in ("mean", "std", "max_minus_mean"):
        np.testing.assert_allclose(p.imb[k].cpu().numpy(), ref[k], rtol=1e-12, atol=1e-9)
    p.close()


def test_more_ranks_than_waves_fit_a_launch(ta, h):
    """70,000,000 ranks of 40 cells: 64 threads per rank would be more than a launch
    can have.  Totals and plain scores against torch in FP64 (sums of 70,000,000
    terms, so within 1e-6), the imbalance's mean and rank sums."""
    import torch
    R, I = 70_000_000, 40
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GB of device memory")
    T = torch.randint(0, 1000, (R, I, 1), device="cuda")
    S = T.sum(1)[:, 0].double()
    z = (S - S.mean()) / S.std()
    o = h.outliers(T, mode=ta.SCAN_TOTALS, kind=ta.SCORE_Z)
    torch.testing.assert_close(o["rank_score"], z.abs(), rtol=1e-6, atol=1e-6)
    cols = T[:, :, 0]
    m = torch.zeros(R, dtype=torch.float64, device="cuda")
    for i in range(I):
        c = cols[:, i].double()
        m += (c - c.mean()) / c.std()
    m /= I
    z = (m - m.mean()) / m.std()
    o = h.outliers(T, kind=ta.SCORE_Z)
    torch.testing.assert_close(o["rank_score"], z.abs(), rtol=1e-6, atol=1e-6)
    g = h.imbalance(T)
    torch.testing.assert_close(g["mean"][:, 0], cols.sum(0).double() / R, rtol=1e-12, atol=0)
    h.sync_status()
    del T, S, z, m, cols, o, g
    torch.cuda.empty_cache()
