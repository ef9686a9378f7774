"""The training kernels at the edges of their 16-row tiles (fewer rows than a
tile, one more than a tile, more tiles than workgroups), on weights that came
from a saved state, from the initialisation and from an optimiser step: the
backward pass reads transposed copies of the weights that each of them writes.
Against oracle/ae.py; relative L2 per matrix at most 1e-2 (bfloat16 operands
rounded alike, sums in FP32 instead of FP64)."""
import numpy as np
import pytest

from oracle import ae
from test_gpu_ae import NP, flat, to_params, unpack

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 4096, 4113, 8209])
@pytest.mark.parametrize("origin", ["state", "init", "step"])
def test_gradient_tiles(n, origin):
    import torch

    from paper_2605_03561_amd import ta
    rng = np.random.default_rng([n, len(origin)])
    X = rng.normal(0, 1, (n, 64)).astype(np.float32)
    rows = torch.from_numpy(X).cuda()
    h = ta.Handle(0)
    h.ae_init(n)
    if origin == "state":
        st = bytearray(h.ae_get_state())
        w = unpack(bytes(st))[0].copy()
        w += rng.normal(0, 0.05, NP).astype(np.float32)
        st[len(st) - (3 * NP + 128) * 4:len(st) - (2 * NP + 128) * 4] = w.tobytes()
        h.ae_set_state(bytes(st))
    elif origin == "step":
        h.ae_train(rows, epochs=1, batch=n, lr=0.02, seed=9)
    torch.cuda.synchronize()
    p = to_params(unpack(h.ae_get_state())[0])
    for _ in range(2):
        g, loss = h.ae_grad(rows)
        g = g.cpu().numpy().astype(np.float64)
        l_ref, g_ref = ae.loss_and_grads(p, X.astype(np.float64), bf16=True)
        assert abs(loss.item() - l_ref) / l_ref < 1e-3
        rg = flat(g_ref)
        cuts = np.cumsum([ae.DIMS[l] * ae.DIMS[l + 1] for l in range(4)])
        for a, b in zip(np.split(g, cuts), np.split(rg, cuts)):
            assert np.linalg.norm(a - b) <= 1e-2 * np.linalg.norm(b)
    h.close()


@pytest.mark.parametrize("R", [12288, 12289])
def test_prescreen_twelve_keys(R):
    """The pre-screen's selections on both sides of twelve keys per lane."""
    from paper_2605_03561_amd import ta
    from test_gpu_select import test_prescreen_selection_edges as check
    h = ta.Handle(0)
    check(ta, h, R)
    h.close()
