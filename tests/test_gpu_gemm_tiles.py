"""The prefill products at the edges of their tiles: ragged rows, columns and
K for every output tile, row-major and packed weights, contiguous and
unaligned outputs, and K-major operands (calibration sums), against fp64.

The bound per output is the fp32 accumulation error K u sum_k |a_k b_k|
(u = 2^-24, any summation order) plus, for a bf16 output, its rounding
(2^-8 of the value: half a unit in the last place of 8 significant bits is
2^-9)."""
import numpy as np
import pytest

from gpu_util import from_dev, torch_mod

pytestmark = pytest.mark.gpu
U32 = 2.0 ** -24


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    if not torch_mod().cuda.is_available():
        pytest.skip("no GPU")


def _bf16(shape, seed):
    torch = torch_mod()
    g = torch.Generator().manual_seed(seed)
    return torch.randn(*shape, generator=g).to(torch.bfloat16)


@pytest.mark.parametrize("M,N,K,tile", [
    (4095, 4040, 72, (256, 256)),   # K past one tile by 8, contiguous rows
    (4095, 4041, 200, (256, 256)),  # odd row length: the scatter's stores
    (4090, 2500, 136, (256, 192)),
    (4001, 2041, 264, (256, 128)),
    (4033, 2040, 8, (256, 128)),    # a single 8-deep K chunk
    (2041, 2040, 200, (128, 128)),
    (1921, 2047, 328, (128, 128)),
    # scattered outputs past the depth up to which the 256 x 256, 256 x 192 and
    # 128 x 128 tiles go through registers (768; 1280 up to one tile per CU),
    # and rows of X that start inside a line on 256 x 192 tiles and with few rows
    (4095, 4041, 776, (256, 256)),
    (4090, 2500, 832, (256, 192)),
    (4090, 2500, 776, (256, 192)),
    (1921, 2047, 1288, (128, 128)),
    (1021, 3847, 1288, (128, 128)),
    # more 128 x 128 tiles than CUs, two to a CU
    (1855, 4120, 136, (128, 128)),
    (1855, 4115, 328, (128, 128)),
    (1855, 4115, 776, (128, 128)),
])
@pytest.mark.parametrize("packed", [True, False])
def test_tile_edges(M, N, K, tile, packed):
    torch = torch_mod()
    from paper_2501_19090_amd import pifa
    assert pifa.pifa_gemm_plan(M, N, K) == tile + (1,)
    X, W = _bf16((M, K), 1), _bf16((N, K), 2)
    # rows next to ordinary ones hold infinities: nothing of a row may reach
    # another, also where the last K tile reads past the end of the row
    X[5::97] = float("inf")
    x, w = X.to("cuda:0"), W.to("cuda:0")
    y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    if packed:
        h = pifa.dense_layer_create(w)
        try:
            pifa.dense_layer_forward(h, x, y)
            torch.cuda.synchronize()
        finally:
            pifa.dense_layer_destroy(h)
    else:
        pifa.dense_forward(w, x, y)
        torch.cuda.synchronize()
    rows = np.setdiff1d(np.arange(M), np.arange(5, M, 97))
    a, b = X.double().numpy()[rows], W.double().numpy()
    ref = a @ b.T
    bound = 2.0 ** -8 * np.abs(ref) + K * U32 * (np.abs(a) @ np.abs(b).T)
    got = from_dev(y)
    assert np.all(np.abs(got[rows] - ref) <= bound)
    assert not np.any(np.isfinite(got[5::97]))


@pytest.mark.parametrize("n,tokens,tile", [
    (4000, 77, (256, 256)),
    (2008, 130, (128, 128)),
    (2400, 64, (256, 128)),
])
def test_k_major_tile_edges(n, tokens, tile):
    from paper_2501_19090_amd import pifa
    assert pifa.pifa_gemm_plan(n, n, tokens, wide_epilogue=2) == tile + (1,)
    _check_sums(n, tokens)


@pytest.mark.parametrize("n,tokens,tile", [
    (3, 600, (64, 64)), (2001, 72, (128, 128)), (2052, 64, (256, 128)), (2399, 77, (256, 128)),
    (3333, 130, (256, 192)), (4001, 72, (256, 256)),
])
def test_calibration_sums_of_unaligned_rows(n, tokens, tile):
    """Activation rows that are not whole 16-byte units, and sums with rows of
    any length: the products run on transposed copies."""
    from paper_2501_19090_amd import pifa
    assert pifa.pifa_gemm_plan(n, n, -(-tokens // 8) * 8)[:2] == tile
    _check_sums(n, tokens)


def _check_sums(n, tokens):
    torch = torch_mod()
    from paper_2501_19090_amd import pifa
    xo, xu = _bf16((tokens, n), 3), _bf16((tokens, n), 4)
    h = pifa.pifa_calib_create(n)
    S = torch.empty((n, n), dtype=torch.float64, device="cuda:0")
    P = torch.empty_like(S)
    try:
        pifa.pifa_calib_accumulate(h, xo.to("cuda:0"), xu.to("cuda:0"))
        pifa.pifa_calib_accumulate(h, xo.to("cuda:0"), xu.to("cuda:0"))
        pifa.pifa_calib_read(h, S, P)
        torch.cuda.synchronize()
    finally:
        pifa.pifa_calib_destroy(h)
    a, b = xo.double().numpy(), xu.double().numpy()
    for got, left in ((S, b), (P, a)):
        bound = 2 * tokens * U32 * (np.abs(left).T @ np.abs(b)) + 1e-12
        assert np.all(np.abs(got.cpu().numpy() - 2 * (left.T @ b)) <= bound)


@pytest.mark.parametrize("d_out,r,M", [(96, 33, 5), (4100, 2050, 3), (16392, 40, 3), (33000, 24, 2), (257, 257, 4),
                                       # either side of the depth at which the gradient products' kernel
                                       # changes (512 rows)
                                       (4100, 2050, 511), (4100, 2050, 513), (1500, 700, 1023), (1500, 700, 1025),
                                       # through LDS: whole 16-byte units, and rows that start inside one
                                       (4104, 40, 4097), (4101, 40, 4098),
                                       # dC of 128 x 128 tiles two to a CU, and shallow on one round of 256 x 256
                                       (5970, 4115, 520), (7075, 4000, 200)])
@pytest.mark.parametrize("offset", [0, 1])
def test_backward_column_split(d_out, r, M, offset):
    """The gather of a gradient's pivot and non-pivot columns: few and many
    rows, long rows, odd row lengths, no non-pivot; offset: gradients and
    outputs that start inside a 16-byte unit."""
    torch = torch_mod()
    from paper_2501_19090_amd import inputs, pifa
    d_in = 264 if r <= 264 else max(2056, (r + 7) // 8 * 8)
    piv, npiv = inputs.random_partition(d_out, r, 9)
    Wp, C = _bf16((r, d_in), 5), _bf16((d_out - r, r), 6)
    X, G = _bf16((M, d_in), 7), _bf16((M, d_out), 8)
    Wd, Cd, Xd, Gd = (t.double().numpy() for t in (Wp, C, X, G))
    Y = np.zeros((M, d_out))
    Y[:, piv] = Xd @ Wd.T
    Y[:, npiv] = Y[:, piv] @ Cd.T
    Yb = torch.from_numpy(Y).to(torch.bfloat16)
    lay = pifa.PifaLayer(Wp.to("cuda:0"), C.to("cuda:0"), piv, npiv, d_out)
    dX = torch.empty((M, d_in), dtype=torch.bfloat16, device="cuda:0")
    dWp = torch.empty((r, d_in), dtype=torch.float32, device="cuda:0")
    dC = torch.empty((d_out - r, r), dtype=torch.float32, device="cuda:0")

    def at_offset(t):
        buf = torch.full((t.numel() + offset,), float("nan"), dtype=t.dtype, device="cuda:0")
        buf[offset:] = t.flatten().to("cuda:0")
        return buf[offset:].view(t.shape)

    pifa.pifa_layer_backward(lay.handle, X.to("cuda:0"), at_offset(Yb), at_offset(G), dX, dWp, dC)
    torch.cuda.synchronize()
    lay.close()
    Gp = Gd[:, piv] + Gd[:, npiv] @ Cd
    # bf16(G_p) feeds dW_p, 2^-9 of each of its terms, and dX is rounded to
    # bf16, 2^-9 of each value: the errors of the terms are independent, so of
    # the whole gradient no more than twice that is left (test_gpu_backward.py)
    for got, ref in ((dWp.cpu().numpy(), Gp.T @ Xd), (from_dev(dX), Gp @ Wd)):
        assert np.linalg.norm(got - ref) <= 5e-3 * np.linalg.norm(ref)
    ref = Gd[:, npiv].T @ Yb.double().numpy()[:, piv]
    bound = (M + 2) * U32 * (np.abs(Gd[:, npiv]).T @ np.abs(Yb.double().numpy()[:, piv]))
    assert np.all(np.abs(dC.cpu().numpy() - ref) <= bound + 1e-30)


@pytest.mark.parametrize("M,N,K", [
    (1, 17, 1), (31, 33, 5), (64, 64, 32), (33, 31, 100),  # 32 x 32 tiles, rows of any alignment
    (1025, 1023, 36), (1031, 1017, 61),                    # 64 x 64 tiles, 16-byte and 4-byte loads
])
def test_f32_tile_edges(M, N, K):
    torch = torch_mod()
    from paper_2501_19090_amd import pifa
    g = torch.Generator().manual_seed(11)
    X, W = torch.randn(M, K, generator=g), torch.randn(N, K, generator=g)
    X[5::97] = float("inf")
    y = torch.full((M, N), float("nan"), device="cuda:0")
    pifa.dense_forward(W.to("cuda:0"), X.to("cuda:0"), y)
    torch.cuda.synchronize()
    rows = np.setdiff1d(np.arange(M), np.arange(5, M, 97))
    a, b = X.double().numpy()[rows], W.double().numpy()
    bound = (K + 1) * U32 * (np.abs(a) @ np.abs(b).T)
    got = from_dev(y)
    assert np.all(np.abs(got[rows] - a @ b.T) <= bound)
    assert not np.any(np.isfinite(got[5::97]))
