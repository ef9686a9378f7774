"""The exact scan's paths by rank count, beyond those that other tests reach:
the row-major passes (more than 49,152 ranks) in a plan and with over-full bracket
slots, the regions' selection by passes over memory (more than 32,768 ranks) with
a missed bracket and with few active ranks, the scores of four ranks per lane,
and more than 256 regions.  Against the oracle, bit for bit."""
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


def same_scan(o, ref):
    st, score, flag, nf, reg = ref
    assert st == 0
    assert np.array_equal(o["region_score"].cpu().numpy(), reg)
    assert np.array_equal(o["rank_score"].cpu().numpy(), score)
    assert np.array_equal(o["rank_flag"].cpu().numpy(), flag)
    assert int(o["n_flagged"][0]) == nf


@pytest.mark.parametrize("I", [10, 7])
def test_row_major_scan_in_a_plan(ta, h, oracle, I):
    """50,001 ranks, 5 regions, an even and an odd row length, ranks that end at
    different iterations: two column halves on two streams, and the imbalance
    from the same pass, on every replay, and equal to the eager calls."""
    import torch
    w = synth.timeline_workload(seed=15, n_ranks=50001, median_len=160, min_len=40, max_len=1500,
                                n_nodes=60, depth_max=5, n_iters=I, n_regions=5, inject_frac=0.02)
    rng = np.random.default_rng(16)
    off = np.asarray(w.offsets, np.int64)
    lens = np.diff(off)
    cut = np.arange(0, len(lens), 3)
    lens[cut] = (lens[cut] * rng.random(len(cut))).astype(np.int64)
    new = np.concatenate([[0], np.cumsum(lens)])
    keep = np.repeat(off[:-1] - new[:-1], lens) + np.arange(new[-1])
    ts, ctx = np.asarray(w.ts)[keep], np.asarray(w.ctx)[keep]
    h.set_tree(w.parent)
    h.set_regions(w.marker, w.regions)
    tr = ta.DeviceTraces(new, ts, ctx)
    st, T, it, out, span = oracle.segment(new, ts, ctx, w.parent, w.marker, w.regions, I)
    assert st == 0 and len(np.unique(it)) > 2
    ref = oracle.outliers(T, it)
    p = h.plan(tr, I, new, autotune=0, region=True)
    eager = h.attribute_segment(tr, I)
    imb = h.imbalance(eager["tensor"], eager["iters_found"], eager["rank_sum"],
                      eager["rank_sumsq"], eager["span"])
    same_scan(h.outliers(eager["tensor"], eager["iters_found"], region=True), ref)
    for rep in range(3):
        p.out["rank_score"].fill_(-7)
        p.out["region_score"].fill_(-7)
        for k in p.imb:
            p.imb[k].fill_(-7)
        torch.cuda.synchronize()
        p.launch()
        h.sync_status()
        assert np.array_equal(p.seg["tensor"].cpu().numpy(), T)
        same_scan(p.out, ref)
        for k in p.imb:
            a, b = p.imb[k], imb[k]
            assert torch.equal(torch.nan_to_num(a, nan=1.5), torch.nan_to_num(b, nan=1.5)), (rep, k)
    p.close()


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("I,G", [(2, 3), (3, 4)])
def test_row_major_slot_overflow(ta, h, oracle, wide, I, G):
    """Columns of 60,000 ranks built against the 2,048 sample ranks (pairs of
    consecutive ranks, evenly spaced), so that the median's interior (region 0)
    or the MAD's (region 1) is more than the 256 cells that a chunk of 1,024 ranks
    keeps; with `wide` another region does not fit the 32-bit copy.  Eager, both
    modes; and the scan in a plan by traces with those cells."""
    import torch
    R = 60000
    rng = np.random.default_rng([60, wide, I])
    Rp = (R + 63) // 64 * 64
    j = np.arange(2048, dtype=np.int64)
    samp = (((j >> 1) * Rp // 1024) & ~1) + (j & 1)
    is_s = np.zeros(R, bool)
    is_s[samp[samp < R]] = True
    T = rng.integers(0, 10**7, (R, I, G))
    for i in range(I):
        spread = rng.integers(0, 10**6, R)
        T[:, i, 0] = np.where(is_s, spread, 499_000 + rng.integers(0, 2_000, R))
        two = np.where(rng.random(R) < 0.5, 250_000, 750_000) + rng.integers(-10_000, 10_000, R)
        T[:, i, 1] = np.where(is_s, spread, two)
        if wide:
            T[:, i, 2] = rng.integers(0, 1 << 40, R)
    it = np.full(R, I, np.int32)
    it[rng.choice(R, 3000, replace=False)] = 1
    dT, dit = torch.from_numpy(T).cuda(), torch.from_numpy(it).cuda()
    for mode in (0, 1):
        same_scan(h.outliers(dT, dit, mode=mode, region=True), oracle.outliers(T, it, mode=mode))
    # the same cells as traces: per iteration the marker, then each region for its time
    parent = np.array([-1] + [0] * (G + 1), np.int32)
    d = np.zeros((R, I, G + 1), np.int64)
    d[..., 0], d[..., 1:] = 10, T
    t = np.zeros((R, I * (G + 1) + 1), np.int64)
    np.cumsum(d.reshape(R, -1), axis=1, out=t[:, 1:])
    c = np.empty((R, I * (G + 1) + 1), np.int32)
    c[:, :-1] = np.tile(np.arange(1, G + 2), I)
    c[:, -1] = 0
    off = np.arange(R + 1, dtype=np.int64) * c.shape[1]
    h.set_tree(parent)
    h.set_regions(1, np.arange(2, G + 2, dtype=np.int32))
    p = h.plan(ta.DeviceTraces(off, t.reshape(-1), c.reshape(-1)), I, off, autotune=0, region=True)
    for _ in range(2):
        p.launch()
    h.sync_status()
    assert np.array_equal(p.seg["tensor"].cpu().numpy(), T)
    same_scan(p.out, oracle.outliers(T, np.full(R, I, np.int32)))
    p.close()


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("case", ["miss", "few", "few and ties"])
def test_region_selection_over_memory(ta, h, oracle, case, mode):
    """More than 32,768 ranks, whose regions are selected by passes over memory: the
    4,096 sample ranks far above the rest, so that the bracket misses the median;
    fewer than 16,384 ranks with iterations, where there is no bracket; and those
    with few distinct values."""
    import torch
    R, I, G = 40000, 1, 3
    rng = np.random.default_rng([len(case), mode])
    r = np.arange(R, dtype=np.int64)
    it = np.full(R, I, np.int32)
    if case == "miss":
        is_s = np.zeros(R, bool)
        is_s[((2 * np.arange(4096, dtype=np.int64) + 1) * R) // (2 * 4096)] = True
        x = np.where(is_s, 10**9 + r, r)
        T = np.stack([x, x[::-1] + rng.integers(0, 3, R), rng.integers(0, 10**6, R)], axis=1)
    else:
        T = rng.integers(0, 10**6, (R, G))
        if case == "few and ties":
            T[:, 0] = 5 + (rng.random(R) < 0.3)
            T[:, 1] = 7
        it[rng.permutation(R)[16000:]] = 0
    T = T.reshape(R, I, G).astype(np.int64)
    o = h.outliers(torch.from_numpy(T).cuda(), torch.from_numpy(it).cuda(), mode=mode, region=True)
    same_scan(o, oracle.outliers(T, it, mode=mode))


@pytest.mark.parametrize("R,I,G", [(16387, 2, 64), (17001, 3, 61), (4099, 2, 257), (40001, 1, 27),
                                   (65, 3, 257), (1000, 2, 257), (65, 2, 300), (1000, 3, 300),
                                   (1024, 1, 513), (1, 2, 300)])
def test_scores_of_many_ranks_and_regions(ta, h, oracle, R, I, G):
    """The column copy's scores with one and four ranks per lane (from 1,024 workgroups
    on; rank counts that are no multiple of four), and up to 1,024 ranks with more
    than 256 regions; some ranks end early, one column spread over 2^34 and one with
    a far cell."""
    import torch
    rng = np.random.default_rng([R, I, G])
    T = rng.integers(0, 10**6, (R, I, G))
    T[:, 0, 1] = rng.integers(0, 2**34, R)
    T[R // 2, I - 1, 2] += 2**33
    T[:, :, 3] *= rng.random((R, I)) < 0.4
    it = np.where(rng.random(R) < 0.1, rng.integers(0, I + 1, R), I).astype(np.int32)
    o = h.outliers(torch.from_numpy(T).cuda(), torch.from_numpy(it).cuda(), region=True)
    same_scan(o, oracle.outliers(T, it))


@pytest.mark.parametrize("R", [8193, 12288, 12289, 16385, 24576, 24577, 32768])
def test_keys_per_lane(ta, h, oracle, R):
    """The regions' selection on both sides of 12 and 24 keys per lane, both modes,
    with equal, spread and negative values and ranks without iterations; the
    pre-screen's second stage and top-k against its own scores."""
    import torch
    rng = np.random.default_rng([R, 12])
    I, G = 2, 5
    T = rng.integers(0, 10**6, (R, I, G))
    T[..., 1] = rng.integers(-2**50, 2**50, (R, I))
    T[..., 2] = 777
    T[..., 3] = rng.integers(0, 2, (R, I))
    it = np.where(rng.random(R) < 0.1, rng.integers(0, I + 1, R), I).astype(np.int32)
    dT, dit = torch.from_numpy(T).cuda(), torch.from_numpy(it).cuda()
    for mode in (0, 1):
        same_scan(h.outliers(dT, dit, mode=mode, region=True), oracle.outliers(T, it, mode=mode))
    X = torch.from_numpy(rng.integers(0, 10**6, (R, 3, 64))).cuda()
    X[R // 3: R // 3 + 50] = X[R // 3]
    h.ae_init(2)
    h.ae_fit_norm(X, None)
    h.ae_set_score_kind(ta.AE_SCORE_RESIDUAL_Z)
    for k in (1, R // 2, R):
        top, sc, fb = h.prescreen(X, None, k)
        s = sc.cpu().numpy()
        assert not fb and np.isfinite(s).all()
        assert np.array_equal(top.cpu().numpy(), np.sort(np.lexsort((np.arange(R), -s))[:k]))
    assert len(np.unique(s[R // 3: R // 3 + 50])) == 1
