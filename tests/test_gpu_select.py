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


@pytest.mark.parametrize("R", [65, 300, 700, 1025, 2049, 3073, 4097, 5121, 6145, 8193, 10241, 12289, 16385,
                               20481, 24577, 32769, 40961, 49153])
@pytest.mark.parametrize("gap", [2000.0, 3e9])
def test_column_selection_in_a_plan(ta, h, oracle, R, gap):
    """The scan's first pass in a plan, which also takes the imbalance columns,
    at every launch shape of the column selection and past the last, with cells
    of microseconds and with columns too spread for 32-bit offsets.  Odd row
    lengths."""
    from paper_2605_03561_amd import synth
    w = synth.plain_workload(seed=R, n_ranks=R, events=30, n_nodes=60, n_iters=3, n_regions=5,
                             mean_gap_ns=gap)
    h.set_tree(w.parent)
    h.set_regions(w.marker, w.regions)
    p = h.plan(ta.DeviceTraces(w.offsets, w.ts, w.ctx), 3, w.offsets, autotune=0, region=True)
    for _ in range(2):
        p.launch()
    h.sync_status()
    T, it = p.seg["tensor"].cpu().numpy(), p.seg["iters_found"].cpu().numpy()
    st, score, flag, nf, reg = oracle.outliers(T, it)
    assert st == 0
    assert np.array_equal(p.out["region_score"].cpu().numpy(), reg)
    assert np.array_equal(p.out["rank_score"].cpu().numpy(), score)
    assert np.array_equal(p.out["rank_flag"].cpu().numpy(), flag)
    _, ref = oracle.imbalance(T, it, span=p.seg["span"].cpu().numpy())
    for k in ("min", "max"):
        assert np.array_equal(p.imb[k].cpu().numpy(), ref[k])
    for k in ("mean", "std", "max_minus_mean", "savings_per_iter", "balance_ratio", "cv_across",
              "cv_within"):
        np.testing.assert_allclose(p.imb[k].cpu().numpy(), ref[k], rtol=1e-12, atol=0)
    p.close()


@pytest.mark.parametrize("R", [1024, 1025, 4096, 4097, 8193, 16384, 16385, 32768, 32769])
def test_prescreen_selection_edges(ta, h, R):
    """Second stage of the pre-screen's score and its top-k at the rank counts
    where the keys per lane change, with a network of zero weights and output
    biases c: the residual is c - x up to one FP32 rounding per row, so the mean
    residual is off by about 1e-7 of max(|x|, |c|) <= 10, i.e. 1e-6, and the
    score by that over a scale of at least 0.1 -- or a relative 1e-6 of the MAD
    times the score, below 1e-4 of it."""
    import torch

    from oracle import ae
    rng = np.random.default_rng([R, 2])
    I = 5
    T = np.rint(rng.gamma(4.0, 2.5e4, (R, I, 64))).astype(np.int64)
    T[:, :, 3] = 12345                         # constant region: z = 0
    T[: (5 * R) // 7 + 1, :, 4] = 777          # MAD 0, mean AD > 0
    T[R // 2: R // 2 + 40] = T[R // 2]         # ranks with equal scores
    it = np.where(rng.random(R) < 0.05, rng.integers(0, I, R), I).astype(np.int32)
    it[R // 2: R // 2 + 40] = I
    dT, dit = torch.from_numpy(T).cuda(), torch.from_numpy(it).cuda()
    h.ae_init(3)
    h.ae_fit_norm(dT, dit)
    state = bytearray(h.ae_get_state())
    NP = h.AE_NP
    tail = 4 * (3 * NP + 128)
    w = np.zeros(NP, np.float32)
    w[NP - 64:] = np.linspace(-0.5, 0.5, 64)
    state[-tail:-tail + 4 * NP] = w.tobytes()
    mu, isd = np.frombuffer(bytes(state[-512:]), np.float32).reshape(2, 64)
    h2 = ta.Handle(0)
    h2.ae_set_state(bytes(state))
    h2.ae_set_score_kind(ta.AE_SCORE_RESIDUAL_Z)
    shapes = dict(W1=(128, 64), W2=(32, 128), W3=(128, 32), W4=(64, 128), b1=(128,), b2=(32,),
                  b3=(128,), b4=(64,))
    params, at = {}, 0
    for name, shape in shapes.items():
        n = int(np.prod(shape))
        params[name] = w[at:at + n].astype(np.float64).reshape(shape)
        at += n
    ref = ae.rank_scores(params, T, it, mu, (np.float32(1) / isd), kind=2)
    for k in (1, R // 3, R):
        top, sc, fb = h2.prescreen(dT, dit, k)
        s = sc.cpu().numpy()
        assert not fb
        assert np.array_equal(top.cpu().numpy(), np.sort(np.lexsort((np.arange(R), -s))[:k]))
    np.testing.assert_allclose(s, ref, rtol=1e-4, atol=1e-5)
    h2.close()


@pytest.mark.parametrize("R", [1, 2, 63, 65, 257, 2047, 2048, 2051])
@pytest.mark.parametrize("I,G", [(3, 5), (27, 37), (5, 257), (1, 300), (2, 1), (17, 64), (9, 127)])
def test_plain_scores_and_rank_sums(ta, h, oracle, R, I, G):
    """Plain z-scores, totals and imbalance from a tensor, with rows above and
    below 1,024 cells, regions below, at and above a wave and a workgroup, and
    rank counts around the chunks of the column sums and the ranks per
    workgroup.  Selections, sums and totals bit for bit; the plain z-score's
    second stage sums R values in another order than the oracle: R * 2^-53
    relative on the mean and deviation, and as much of the largest value on the
    score."""
    import torch
    if R > 300 and I * G > 1000:
        I = max(1, 1000 // G + 1)
    T, it = tensor(np.random.default_rng([R, I, G]), R, I, G)
    dT, dit = torch.from_numpy(T).cuda(), torch.from_numpy(it).cuda()
    o = h.outliers(dT, dit, kind=ta.SCORE_Z, region=True)
    st, score, flag, nf, reg = oracle.outliers(T, it, kind=1)
    assert st == 0
    np.testing.assert_allclose(o["region_score"].cpu().numpy(), reg, rtol=1e-9, atol=1e-9)
    np.testing.assert_allclose(o["rank_score"].cpu().numpy(), score, rtol=1e-9, atol=1e-9)
    o = h.outliers(dT, dit, mode=ta.SCAN_TOTALS, region=True)
    st, score, flag, nf, reg = oracle.outliers(T, it, mode=1)
    assert st == 0
    assert np.array_equal(o["region_score"].cpu().numpy(), reg)
    assert np.array_equal(o["rank_flag"].cpu().numpy(), flag)
    g = h.imbalance(dT, dit)
    _, ref = oracle.imbalance(T, it)
    for k in ("min", "max"):
        assert np.array_equal(g[k].cpu().numpy(), ref[k])
    for k in ("mean", "std", "max_minus_mean", "savings_per_iter", "cv_across", "cv_within"):
        np.testing.assert_allclose(g[k].cpu().numpy(), ref[k], rtol=1e-9, atol=1e-9)


@pytest.mark.parametrize("R", [0, 1, 255, 256, 257, 40000])
@pytest.mark.parametrize("mode", [0, 1])
def test_flag_count(ta, h, R, mode):
    """The number of flags from none to all but a few, on several calls and
    without any rank."""
    import torch
    rng = np.random.default_rng([R, mode])
    T, it = rng.integers(0, 10**6, (R, 3, 5)).astype(np.int64), np.full(R, 3, np.int32)
    for tau in (1e9, 0.5, 0.0):
        for kind in (ta.SCORE_MAD, ta.SCORE_Z):
            o = h.outliers(torch.from_numpy(T).cuda(), torch.from_numpy(it).cuda(), mode=mode, kind=kind, tau=tau)
            flag = o["rank_flag"].cpu().numpy()
            assert np.array_equal(flag, o["rank_score"].cpu().numpy() > tau)
            assert int(o["n_flagged"].item()) == int(flag.sum())
