"""The pivot steps of the GPU build at the edges of their split: rows just
below, at and past one workgroup's 512 and all sixteen workgroups' 8192;
panels of one step, one short of, at and past 16; square, wide and tall;
every row a pivot; and equal rows, whose ties go to the lowest index."""
import numpy as np
import pytest

import oracle
from gpu_util import rel_fro, torch_mod
from paper_2501_19090_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _cuda():
    if not torch_mod().cuda.is_available():
        pytest.skip("no GPU")


def _check(W, r):
    from paper_2501_19090_amd import pifa
    ref = oracle.build_pifa(W, r)
    Wd = torch_mod().from_numpy(np.ascontiguousarray(W)).to("cuda:0")
    piv, npiv, Wp, C, report = pifa.pifa_build_f64(Wd, r)
    assert np.array_equal(piv, ref["pivot_idx"]) and np.array_equal(npiv, ref["nonpivot_idx"])
    assert np.array_equal(Wp.cpu().numpy(), W[ref["pivot_idx"]])
    # fp64 rounding (2^-53) times the pivoted factor's growth and the depth of
    # its sums, at most a few thousand here
    if C.numel():
        assert rel_fro(C.cpu().numpy(), ref["C"]) <= 1e-10
    assert report[3] == 1.0


@pytest.mark.parametrize("d_out,d_in,r", [
    (70, 511, 1), (70, 512, 15), (70, 513, 16), (4200, 40, 17), (33, 1025, 33),
    (17, 16, 16), (1, 8, 1), (50, 8192, 20), (50, 16385, 18), (30, 8200, 24),
])
def test_step_edges(d_out, d_in, r):
    U, V = inputs.lowrank_factors(d_out, d_in, r, seed=3 * d_out + r)
    _check(U @ V, r)


@pytest.mark.parametrize("d_out,d_in,r", [(90, 600, 30), (5000, 64, 20)])
def test_equal_rows(d_out, d_in, r):
    """Every row twice, the halves swapped in order: the first copy is picked."""
    U, V = inputs.lowrank_factors(d_out // 2, d_in, r, seed=5)
    W = U @ V
    W = np.concatenate([W, W[::-1]])
    _check(W, r)
