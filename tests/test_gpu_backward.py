"""Backward pass of the PIFA layer (pifa_layer_backward) against the fp64
oracle's chain rule, through the C ABI.

The oracle evaluates the gradients on the same bf16 bits the GPU consumes
(X, dY, W_p, C); Y_p for dC comes from the GPU forward's output Y[:, I], whose
bf16 rounding is inside the bar.  Bar: rel_F <= 5e-3 for dX (bf16 out), dW_p
and dC (fp32 out).  At the benchmark size the oracle checks sampled rows of
dX and sampled pivot slots of dW_p and dC (a reduced problem that yields
exactly those gradient entries).
"""
import numpy as np
import pytest

import oracle
from paper_2501_19090_amd import inputs

from gpu_util import (DeviceLayer, activations, config_layer, from_dev, gaussian_layer, rel_fro, sample_rows,
                      to_dev, torch_mod)

pytestmark = pytest.mark.gpu
TOL = 5e-3


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    if not torch_mod().cuda.is_available():
        pytest.skip("no GPU")


def _grads(lay, x_dev, g_dev, M):
    from paper_2501_19090_amd import pifa
    torch = torch_mod()
    y = lay.forward(x_dev, M)
    dX = torch.full((max(M, 1), lay.d_in), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    dWp = torch.full((lay.r, lay.d_in), float("nan"), dtype=torch.float32, device="cuda:0")
    dC = torch.full((max(lay.d_out - lay.r, 1), lay.r), float("nan"), dtype=torch.float32, device="cuda:0")
    pifa.pifa_layer_backward(lay.handle, x_dev, y, g_dev, dX, dWp, dC if lay.d_out > lay.r else None, M)
    torch.cuda.synchronize()
    return dX, dWp, dC


def _check_small(lay, M, seed):
    x_dev, x64 = activations(M, lay.d_in, seed, "bf16")
    g_dev, g64 = activations(M, lay.d_out, seed + 1000, "bf16")
    dX, dWp, dC = _grads(lay, x_dev, g_dev, M)
    rX, rW, rC = oracle.pifa_backward(x64, g64, lay.piv, lay.npiv, lay.Wp, lay.C)
    assert rel_fro(from_dev(dX), rX) <= TOL, ("dX", M)
    assert rel_fro(from_dev(dWp), rW) <= TOL, ("dWp", M)
    if rC.size:
        assert rel_fro(from_dev(dC), rC) <= TOL, ("dC", M)


@pytest.mark.parametrize("d_in,d_out,r", [(256, 320, 96), (136, 203, 72), (512, 1024, 300), (128, 96, 96)])
def test_backward_small_shapes(d_in, d_out, r):
    """Ragged r (not a multiple of 64), n_np not a multiple of 8, r = d_out."""
    piv, npiv, Wp, C, *_ = gaussian_layer(d_in, d_out, r, 50 + r)
    lay = DeviceLayer(piv, npiv, Wp, C, "bf16")
    try:
        for M in (1, 5, 17, 100, 300):
            _check_small(lay, M, seed=M)
    finally:
        lay.close()


def test_backward_full_size_sampled():
    """The LLaMA-7B attention shape (4096 x 4096, r = 2048) at M = 4096."""
    piv, npiv, Wp, C, *_ = config_layer("B_attn_4096")
    lay = DeviceLayer(piv, npiv, Wp, C, "bf16")
    try:
        M = 4096
        x_dev, x64 = activations(M, lay.d_in, 21, "bf16")
        g_dev, g64 = activations(M, lay.d_out, 22, "bf16")
        dX, dWp, dC = _grads(lay, x_dev, g_dev, M)
        # dX rows depend only on their own rows of X and G: the first, the
        # last and 510 seeded rows (the oracle's backward of all 4096 rows
        # takes minutes)
        rows = sample_rows(M, k=510)
        rX, _, _ = oracle.pifa_backward(x64[rows], g64[rows], lay.piv, lay.npiv, lay.Wp, lay.C)
        assert rel_fro(from_dev(dX)[rows], rX) <= TOL
        # dW_p[S, :] and dC[:, S] for a few pivot slots S: the same gradients
        # of the reduced layer whose pivot set is I[S] (outputs re-indexed)
        S = np.array([0, 1, 517, 1024, 2046, 2047])
        Gs = np.concatenate([g64[:, lay.piv[S]], g64[:, lay.npiv]], axis=1)
        piv_s = np.arange(S.size, dtype=np.int32)
        npiv_s = np.arange(S.size, S.size + lay.npiv.size, dtype=np.int32)
        _, rW, rC = oracle.pifa_backward(x64, Gs, piv_s, npiv_s, lay.Wp[S], lay.C[:, S])
        assert rel_fro(from_dev(dWp)[S], rW) <= TOL
        assert rel_fro(from_dev(dC)[:, S], rC) <= TOL
        assert torch_mod().isfinite(dWp).all() and torch_mod().isfinite(dC).all()
    finally:
        lay.close()


@pytest.mark.parametrize("M,r,tile", [
    (4096, 4041, (256, 256)),   # r_pad = 4096
    (4096, 2560, (256, 192)),   # r_pad = 2560: the last 64 of 192 columns
    (4090, 2750, (256, 192)),   # r_pad = 2752, the same; the last two are padding
    (4096, 2810, (256, 192)),   # r_pad = 2816: the last 128 of 192 columns, six of them padding
    (4096, 2304, (256, 192)),   # r_pad = 2304: whole tiles
    (4001, 2000, (256, 128)),
    (2041, 1990, (128, 128)),
    (1855, 4100, (128, 128)),   # 495 tiles, two to a CU
])
def test_backward_pivot_gradient_tiles(M, r, tile):
    """G_p on every output tile that it can take, at ranks whose last tile is
    cut at different columns, with large values of an earlier, longer call
    still in the workspace.  The last pivot columns are compared on their own
    too: a few wrong columns are little of the whole gradient."""
    from paper_2501_19090_amd import pifa
    torch = torch_mod()
    n_np = 44
    d_in, d_out = (r + 7) // 8 * 8, r + n_np
    assert pifa.pifa_gemm_plan(M, -(-r // 64) * 64, -(-n_np // 8) * 8)[:2] == tile
    rng = np.random.default_rng(r)
    piv, npiv = inputs.random_partition(d_out, r, 3)
    lay = DeviceLayer(piv, npiv, rng.standard_normal((r, d_in)) * r ** -0.5,
                      rng.standard_normal((n_np, r)) * r ** -0.5, "bf16")
    try:
        x_dev, _ = activations(M + 256, d_in, 5, "bf16")
        g_dev, _ = activations(M + 256, d_out, 6, "bf16")
        _grads(lay, x_dev, g_dev * 4096, M + 256)
        x_dev, x64 = activations(M, d_in, 7, "bf16")
        g_dev, g64 = activations(M, d_out, 8, "bf16")
        dX, dWp, dC = _grads(lay, x_dev, g_dev, M)
        # dX row by row, dW_p and dC by pivot slots (as in the full-size test)
        rows = sample_rows(M, k=254)
        rX, _, _ = oracle.pifa_backward(x64[rows], g64[rows], lay.piv, lay.npiv, lay.Wp, lay.C)
        assert rel_fro(from_dev(dX)[rows], rX) <= TOL
        S = np.unique(np.concatenate([np.arange(0, r, 97), np.arange(r - 32, r)]))
        Gs = np.concatenate([g64[:, lay.piv[S]], g64[:, lay.npiv]], axis=1)
        piv_s = np.arange(S.size, dtype=np.int32)
        npiv_s = np.arange(S.size, S.size + n_np, dtype=np.int32)
        _, rW, rC = oracle.pifa_backward(x64, Gs, piv_s, npiv_s, lay.Wp[S], lay.C[:, S])
        for part in (slice(None), slice(-8, None), slice(-32, None)):
            assert rel_fro(from_dev(dWp)[S][part], rW[part]) <= TOL
            assert rel_fro(from_dev(dC)[:, S][:, part], rC[:, part]) <= TOL
        assert torch.isfinite(dX).all() and torch.isfinite(dWp).all() and torch.isfinite(dC).all()
    finally:
        lay.close()


@pytest.mark.parametrize("M,r", [(3, 1), (300, 40), (4096, 1000)])
def test_backward_infinite_gradient(M, r):
    """An infinity in a non-pivot gradient reaches dX with its sign: the rank's
    padding adds nothing to the row."""
    n_np, d_in = 3, (r + 7) // 8 * 8
    piv, npiv = inputs.random_partition(r + n_np, r, 3)
    lay = DeviceLayer(piv, npiv, np.ones((r, d_in)), np.ones((n_np, r)), "bf16")
    try:
        x_dev, _ = activations(M, d_in, 7, "bf16")
        g_dev, g64 = activations(M, r + n_np, 8, "bf16")
        inf = np.arange(1, M, 97)
        g_dev[inf, int(npiv[1])] = float("inf")
        dX = from_dev(_grads(lay, x_dev, g_dev, M)[0])
        assert np.all(dX[inf] == np.inf)
        rows = np.setdiff1d(np.arange(M), inf)
        Gp = g64[rows][:, piv] + g64[rows][:, npiv].sum(1, keepdims=True)
        assert rel_fro(dX[rows], np.repeat(Gp.sum(1, keepdims=True), d_in, 1)) <= TOL
    finally:
        lay.close()


def test_backward_deterministic_and_optional_outputs():
    from paper_2501_19090_amd import pifa
    torch = torch_mod()
    piv, npiv, Wp, C, *_ = gaussian_layer(256, 320, 96, 146)
    lay = DeviceLayer(piv, npiv, Wp, C, "bf16")
    try:
        M = 77
        x_dev, _ = activations(M, 256, 3, "bf16")
        g_dev, _ = activations(M, 320, 4, "bf16")
        a = _grads(lay, x_dev, g_dev, M)
        b = _grads(lay, x_dev, g_dev, M)
        for u, v in zip(a, b):
            assert torch.equal(u, v)
        # outputs may be skipped one by one
        y = lay.forward(x_dev, M)
        dWp = torch.zeros((96, 256), dtype=torch.float32, device="cuda:0")
        pifa.pifa_layer_backward(lay.handle, x_dev, y, g_dev, None, dWp, None, M)
        torch.cuda.synchronize()
        assert torch.equal(dWp, a[1])
        # M = 0 is the zero gradient
        pifa.pifa_layer_backward(lay.handle, x_dev, y, g_dev, None, dWp, None, 0)
        torch.cuda.synchronize()
        assert not dWp.any()
    finally:
        lay.close()


def test_backward_rejects_f32_layer():
    from paper_2501_19090_amd import pifa
    piv, npiv, Wp, C, *_ = gaussian_layer(64, 80, 32, 7)
    lay = DeviceLayer(piv, npiv, Wp, C, "f32")
    try:
        x_dev, _ = activations(4, 64, 1, "f32")
        # the binding refuses fp32 activations for the (bf16-only) backward ...
        with pytest.raises(TypeError):
            pifa.pifa_layer_backward(lay.handle, x_dev, x_dev, x_dev, None, None, None, 4)
        # ... and the library itself refuses the fp32 layer
        st = pifa.lib().pifa_layer_backward(lay.handle, x_dev.data_ptr(), x_dev.data_ptr(), x_dev.data_ptr(), 4,
                                            None, None, None, None)
        assert st == pifa.PIFA_ERR_UNSUPPORTED
    finally:
        lay.close()
