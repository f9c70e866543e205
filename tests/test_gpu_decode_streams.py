"""Long decode weight streams with more than four activation rows: dense,
pair-operand and grouped products whose 16-row groups are walked by one
workgroup per CU, at two to four passes over K, ragged rows and columns, and
a change of problem inside a workgroup's range; and the long streams of one
pass or few rows that are not walked.  Bounds per output: bf16
rounding (2^-8 of the value, twice what it needs) plus fp32 accumulation
(K u sum |a b|) and, behind the fp16 pair, 2^-20 of its terms."""
import numpy as np
import pytest

from gpu_util import from_dev, torch_mod

pytestmark = pytest.mark.gpu
U32 = 2.0 ** -24


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    if not torch_mod().cuda.is_available():
        pytest.skip("no GPU")


def _bf16(shape, seed, scale=1.0):
    torch = torch_mod()
    g = torch.Generator().manual_seed(seed)
    return (torch.randn(*shape, generator=g) * scale).to(torch.bfloat16)


def _check(got, ref, bound):
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + bound)


@pytest.mark.parametrize("M,N,K", [(5, 98305, 128), (16, 98305, 128), (16, 8325, 1600), (6, 12289, 4096),
                                   # 8192 blocks: 9 rows are too few, 11 enough
                                   (9, 8192, 2040), (11, 8192, 2040)])
def test_dense_streams(M, N, K):
    from paper_2501_19090_amd import pifa
    torch = torch_mod()
    X, W = _bf16((M, K), 1), _bf16((N, K), 2, K ** -0.5)
    y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    h = pifa.dense_layer_create(W.to("cuda:0"))
    try:
        pifa.dense_layer_forward(h, X.to("cuda:0"), y)
        torch.cuda.synchronize()
    finally:
        pifa.dense_layer_destroy(h)
    a, b = X.double().numpy(), W.double().numpy()
    _check(from_dev(y), a @ b.T, K * U32 * (np.abs(a) @ np.abs(b).T))


def _member(d_in, d_out, r, seed):
    from paper_2501_19090_amd import inputs
    piv, npiv = inputs.random_partition(d_out, r, seed)
    return _bf16((r, d_in), seed + 1, r ** -0.5), _bf16((d_out - r, r), seed + 2, r ** -0.5), piv, npiv


def _reference(X, Wp, C, piv, npiv, d_out):
    x, w, c = (t.double().numpy() for t in (X, Wp, C))
    ref, bound = np.zeros((x.shape[0], d_out)), np.zeros((x.shape[0], d_out))
    yp = x @ w.T
    ep = x.shape[1] * U32 * (np.abs(x) @ np.abs(w).T)
    ref[:, piv], bound[:, piv] = yp, ep
    ref[:, npiv] = yp @ c.T
    bound[:, npiv] = (ep + (w.shape[0] * U32 + 2.0 ** -20) * np.abs(yp)) @ np.abs(c).T
    return ref, bound


@pytest.mark.parametrize("M", [5, 8, 16])
def test_grouped_streams(M):
    """Members of 12, 24 and 3 K blocks; the middle one alone is long enough too."""
    from paper_2501_19090_amd import pifa
    torch = torch_mod()
    shapes = [(9001, 1500), (11400, 3000), (4003, 264)]
    d_in = 3008
    members = [_member(d_in, d, r, 10 * i) for i, (d, r) in enumerate(shapes)]
    X = _bf16((M, d_in), 77)
    specs = [(Wp.to("cuda:0"), C.to("cuda:0"), p, n, (d_in, d, r))
             for (Wp, C, p, n), (d, r) in zip(members, shapes)]
    total = sum(d for d, _ in shapes)
    y = torch.full((M, total), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    g = pifa.pifa_group_create(specs)
    try:
        pifa.pifa_group_forward(g, X.to("cuda:0"), y)
        torch.cuda.synchronize()
    finally:
        pifa.pifa_group_destroy(g)
    got, o = from_dev(y), 0
    for (Wp, C, p, n), (d, r), spec in zip(members, shapes, specs):
        ref, bound = _reference(X, Wp, C, p, n, d)
        _check(got[:, o:o + d], ref, bound)
        lay = pifa.PifaLayer(spec[0], spec[1], p, n, d)
        one = lay(X.to("cuda:0")).view(torch.int16).cpu()
        lay.close()
        assert torch.equal(one, y[:, o:o + d].contiguous().view(torch.int16).cpu())
        o += d
