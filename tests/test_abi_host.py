"""C-ABI checks that need no GPU: the library loads, exports every symbol the
header declares, and rejects bad arguments before touching the device."""
import ctypes

import numpy as np
import pytest

from paper_2501_19090_amd import pifa

FAKE = ctypes.c_void_p(0x1000)  # never dereferenced: validation fails first


def test_library_exports_every_declared_symbol():
    declared = pifa.declared_symbols()
    assert "pifa_layer_create" in declared and "pifa_forward" in declared
    assert "dense_forward" in declared and "lowrank_uv_forward" in declared
    lib = pifa.lib()
    missing = [s for s in declared if not hasattr(lib, s)]
    assert not missing, missing
    # the binding wraps every declared entry point under the same name
    assert not [s for s in declared if not hasattr(pifa, s)]


def test_status_strings():
    for code, name in [(0, "PIFA_OK"), (-1, "PIFA_ERR_INVALID_ARG"), (-2, "PIFA_ERR_BAD_INDEX"),
                       (-3, "PIFA_ERR_UNSUPPORTED"), (-4, "PIFA_ERR_HIP"), (-5, "PIFA_ERR_OOM")]:
        assert pifa.pifa_status_string(code) == name
    assert pifa.pifa_status_string(7) == "PIFA_ERR_UNKNOWN"


def _perm_split(d_out, r, seed=0):
    perm = np.random.default_rng(seed).permutation(d_out).astype(np.int32)
    return perm[:r], perm[r:]


def test_validate_partition_accepts_any_order():
    piv, npiv = _perm_split(50, 20)
    assert pifa.pifa_validate_partition(piv, npiv, (30, 50, 20)) == pifa.PIFA_OK
    assert pifa.pifa_validate_partition(np.sort(piv), np.sort(npiv), (30, 50, 20)) == pifa.PIFA_OK
    # r = d_out: empty complement
    assert pifa.pifa_validate_partition(np.arange(8), None, (8, 8, 8)) == pifa.PIFA_OK


@pytest.mark.parametrize("mutate", ["dup", "range_hi", "range_lo", "overlap"])
def test_validate_partition_rejects_bad_indices(mutate):
    piv, npiv = _perm_split(40, 15, 3)
    piv, npiv = piv.copy(), npiv.copy()
    if mutate == "dup":
        piv[1] = piv[0]
    elif mutate == "range_hi":
        npiv[0] = 40
    elif mutate == "range_lo":
        piv[2] = -1
    elif mutate == "overlap":
        npiv[0] = piv[0]
    assert pifa.pifa_validate_partition(piv, npiv, (16, 40, 15)) == pifa.PIFA_ERR_BAD_INDEX


@pytest.mark.parametrize("dims", [(0, 10, 1), (10, 0, 1), (10, 10, 0), (10, 10, 11), (5, 10, 6),
                                  (10, 5, 6), (-1, 4, 1)])
def test_validate_partition_rejects_bad_dims(dims):
    piv = np.arange(max(dims[2], 1), dtype=np.int32)
    assert pifa.pifa_validate_partition(piv, piv, dims) == pifa.PIFA_ERR_INVALID_ARG


def test_validate_partition_null_pointers():
    lib = pifa.lib()
    assert lib.pifa_validate_partition(None, None, pifa.pifa_dims(4, 4, 2)) == pifa.PIFA_ERR_INVALID_ARG
    piv = np.arange(4, dtype=np.int32)
    # r = d_out needs no complement
    assert lib.pifa_validate_partition(piv.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)), None,
                                       pifa.pifa_dims(4, 4, 4)) == pifa.PIFA_OK


def _create(Wp, C, piv, npiv, dims, dtype):
    out = ctypes.c_void_p()
    pp = None if piv is None else np.ascontiguousarray(piv, np.int32).ctypes.data_as(
        ctypes.POINTER(ctypes.c_int32))
    npp = None if npiv is None else np.ascontiguousarray(npiv, np.int32).ctypes.data_as(
        ctypes.POINTER(ctypes.c_int32))
    st = pifa.lib().pifa_layer_create(Wp, C, pp, npp, pifa.pifa_dims(*dims), dtype, ctypes.byref(out))
    return st, out.value


def test_create_rejects_before_device_work():
    piv, npiv = _perm_split(64, 16)
    ok_dims = (64, 64, 16)
    # null output handle pointer
    assert pifa.lib().pifa_layer_create(FAKE, FAKE, None, None, pifa.pifa_dims(*ok_dims),
                                        pifa.PIFA_BF16, None) == pifa.PIFA_ERR_INVALID_ARG
    # bad dtype
    assert _create(FAKE, FAKE, piv, npiv, ok_dims, 7)[0] == pifa.PIFA_ERR_INVALID_ARG
    # null weights / missing C with r < d_out
    assert _create(None, FAKE, piv, npiv, ok_dims, pifa.PIFA_BF16)[0] == pifa.PIFA_ERR_INVALID_ARG
    assert _create(FAKE, None, piv, npiv, ok_dims, pifa.PIFA_BF16)[0] == pifa.PIFA_ERR_INVALID_ARG
    # bf16 rows must be 16-byte multiples
    assert _create(FAKE, FAKE, piv, npiv, (60, 64, 16), pifa.PIFA_BF16)[0] == pifa.PIFA_ERR_UNSUPPORTED
    # bad partition
    bad = npiv.copy(); bad[0] = piv[0]
    st, h = _create(FAKE, FAKE, piv, bad, ok_dims, pifa.PIFA_BF16)
    assert st == pifa.PIFA_ERR_BAD_INDEX and h is None
    # rank larger than a dimension
    assert _create(FAKE, FAKE, piv, npiv, (8, 64, 16), pifa.PIFA_F32)[0] == pifa.PIFA_ERR_INVALID_ARG


def test_forward_and_baselines_reject_bad_args():
    lib = pifa.lib()
    assert lib.pifa_forward(None, FAKE, FAKE, 4, None) == pifa.PIFA_ERR_INVALID_ARG
    assert lib.pifa_layer_destroy(None) == pifa.PIFA_OK
    assert lib.pifa_layer_weight_bytes(None) == 0
    assert lib.dense_forward(FAKE, FAKE, FAKE, -1, 8, 8, pifa.PIFA_BF16, None) == pifa.PIFA_ERR_INVALID_ARG
    assert lib.dense_forward(FAKE, FAKE, FAKE, 4, 8, 8, 9, None) == pifa.PIFA_ERR_INVALID_ARG
    assert lib.dense_forward(None, FAKE, FAKE, 4, 8, 8, pifa.PIFA_BF16, None) == pifa.PIFA_ERR_INVALID_ARG
    assert lib.dense_forward(FAKE, FAKE, FAKE, 4, 12, 8, pifa.PIFA_BF16, None) == pifa.PIFA_ERR_UNSUPPORTED
    # M = 0 is a no-op that succeeds without a device
    assert lib.dense_forward(FAKE, FAKE, FAKE, 0, 8, 8, pifa.PIFA_BF16, None) == pifa.PIFA_OK
    assert lib.lowrank_uv_forward(FAKE, FAKE, FAKE, FAKE, 0, pifa.pifa_dims(8, 8, 4), pifa.PIFA_BF16,
                                  None) == pifa.PIFA_OK
    assert lib.lowrank_uv_forward(FAKE, FAKE, FAKE, FAKE, 4, pifa.pifa_dims(8, 8, 9), pifa.PIFA_BF16,
                                  None) == pifa.PIFA_ERR_INVALID_ARG
    assert lib.lowrank_uv_forward(FAKE, FAKE, FAKE, FAKE, 4, pifa.pifa_dims(16, 16, 4), pifa.PIFA_BF16,
                                  None) == pifa.PIFA_ERR_UNSUPPORTED
    assert lib.lowrank_layer_forward(None, FAKE, FAKE, 4, None) == pifa.PIFA_ERR_INVALID_ARG
    assert lib.lowrank_layer_destroy(None) == pifa.PIFA_OK
    assert lib.pifa_layer_set_intermediate_scale(None, 0) == pifa.PIFA_ERR_INVALID_ARG
    assert lib.pifa_layer_overflow_count(None, None) == pifa.PIFA_ERR_INVALID_ARG


def test_status_strings_of_build_and_reconstruction():
    assert pifa.pifa_status_string(pifa.PIFA_ERR_NOT_RANK_R) == "PIFA_ERR_NOT_RANK_R"
    assert pifa.pifa_status_string(pifa.PIFA_ERR_NOT_SPD) == "PIFA_ERR_NOT_SPD"
    assert pifa.pifa_status_string(pifa.PIFA_ERR_WRONG_DEVICE) == "PIFA_ERR_WRONG_DEVICE"


def test_group_backward_and_calibration_reject_bad_args_on_host():
    """Argument errors of the grouped, backward and reconstruction entry points
    are found before any device work."""
    lib = pifa.lib()
    out = ctypes.c_void_p()
    dims = (pifa.pifa_dims * 2)(pifa.pifa_dims(64, 96, 32), pifa.pifa_dims(32, 96, 32))
    ptrs = (ctypes.c_void_p * 2)(FAKE.value, FAKE.value)
    piv, npiv = np.arange(32, dtype=np.int32), np.arange(32, 96, dtype=np.int32)  # a valid partition
    pp = (pifa._i32p * 2)(piv.ctypes.data_as(pifa._i32p), piv.ctypes.data_as(pifa._i32p))
    npp = (pifa._i32p * 2)(npiv.ctypes.data_as(pifa._i32p), npiv.ctypes.data_as(pifa._i32p))
    inval = pifa.PIFA_ERR_INVALID_ARG
    # group: no layers, too many layers, null handle slot, differing d_in, fp32
    assert lib.pifa_group_create(0, ptrs, ptrs, pp, npp, dims, pifa.PIFA_BF16, ctypes.byref(out)) == inval
    assert lib.pifa_group_create(9, ptrs, ptrs, pp, npp, dims, pifa.PIFA_BF16, ctypes.byref(out)) == inval
    assert lib.pifa_group_create(1, ptrs, ptrs, pp, npp, dims, pifa.PIFA_BF16, None) == inval
    assert lib.pifa_group_create(2, ptrs, ptrs, pp, npp, dims, pifa.PIFA_BF16, ctypes.byref(out)) == inval
    assert lib.pifa_group_create(1, ptrs, ptrs, pp, npp, dims, pifa.PIFA_F32,
                                 ctypes.byref(out)) == pifa.PIFA_ERR_UNSUPPORTED
    assert lib.pifa_group_forward(None, FAKE, FAKE, 4, None) == inval
    assert lib.pifa_group_reserve(None, 4) == inval
    assert lib.pifa_group_destroy(None) == pifa.PIFA_OK
    # backward and calibration
    assert lib.pifa_layer_backward(None, FAKE, FAKE, FAKE, 4, FAKE, FAKE, FAKE, None) == inval
    assert lib.pifa_calib_create(0, ctypes.byref(out)) == inval
    assert lib.pifa_calib_create(64, None) == inval
    assert lib.pifa_calib_accumulate(None, FAKE, FAKE, 8, None) == inval
    assert lib.pifa_calib_reconstruct(None, FAKE, 8, FAKE, 4, 0.25, 1e-3, FAKE, FAKE, None) == inval
    assert lib.pifa_calib_read(None, None, None, None) == inval
    assert lib.pifa_calib_destroy(None) == pifa.PIFA_OK


@pytest.mark.parametrize("shape,wide,plan", [
    ((4096, 2048, 4096), True, (256, 128, 1)),    # attention layer, both products
    ((4096, 2496, 4096), True, (256, 192, 1)),    # r = 60% pivot product: one round of 256 x 192
    ((4096, 8960, 2048), True, (256, 192, 1)),    # MLP up projection's non-pivot product
    ((4096, 4096, 8192), True, (256, 256, 1)),    # 70B square layer's pivot product
    ((4096, 4096, 8192), False, (256, 128, 1)),   # epilogue with per-output state: no wide tile
    ((4096, 448, 4096), True, (128, 64, 1)),      # r = 10% pivot product: 224 tiles of 128 x 64, no split
    ((4096, 832, 4096), True, (128, 128, 1)),     # 13.6 MB per split: no split, 224 tiles
    ((2048, 2048, 4096), True, (128, 128, 1)),    # 256 tiles fill the chip
])
def test_gemm_plan_of_measured_shapes(shape, wide, plan):
    """The prefill tile and K split chosen for shapes whose choice was measured."""
    assert pifa.pifa_gemm_plan(*shape, wide_epilogue=wide) == plan


def test_gemm_plan_of_k_major_products():
    """K-major operands have no 256 x 192 tile; where that is not the tile
    chosen, both plans agree, K splits (which size the partial sums) included."""
    assert pifa.pifa_gemm_plan(4096, 2496, 4096, wide_epilogue=2) == (256, 256, 1)
    for M in (17, 100, 128, 640, 1000, 2048, 4096, 11008):
        for N in (64, 200, 410, 832, 2048, 2496, 4096, 8960):
            for K in (64, 512, 4096, 16384):
                all_tiles = pifa.pifa_gemm_plan(M, N, K)
                square = pifa.pifa_gemm_plan(M, N, K, wide_epilogue=2)
                assert square[2] == all_tiles[2] and square[:2] != (256, 192)
                assert square == all_tiles or all_tiles[:2] == (256, 192)


def test_gemm_plan_splits_small_batches():
    """Few rows: K is split, over 64 x 64 tiles up to 128 rows and over
    128 x 64 tiles above (half the splits 128 x 128 tiles would need for as
    many workgroups), with at most 16 splits and partials no larger than the
    operands; a product at most 2048 deep whose 64 x 64 tiles fill half the
    chip or more is not split."""
    for M in (17, 64, 128, 256):
        tm, tn, s = pifa.pifa_gemm_plan(M, 2048, 4096)
        assert (tm, tn) == ((64, 64) if M <= 128 else (128, 64)) and 1 < s <= 16
        assert s * M * 2048 * 4 <= (M + 2048) * 4096 * 2
        assert -(-M // tm) * (2048 // tn) * s <= 512
    assert pifa.pifa_gemm_plan(32, 2048, 4096) == (64, 64, 8)
    assert pifa.pifa_gemm_plan(128, 2048, 4096) == (64, 64, 4)
    assert pifa.pifa_gemm_plan(128, 2048, 2048) == (64, 64, 4)
    assert pifa.pifa_gemm_plan(256, 2048, 4096) == (128, 64, 4)
    # at most 2048 deep, with 64 x 64 tiles filling half the chip or more: no split
    assert pifa.pifa_gemm_plan(256, 2048, 2048) == (64, 64, 1)
    assert pifa.pifa_gemm_plan(512, 2048, 2048) == (64, 64, 1)
    assert pifa.pifa_gemm_plan(256, 4096, 2048) == (64, 64, 1)
    assert pifa.pifa_gemm_plan(192, 2048, 2048)[2] > 1
    # 64 x 64 tiles only while a split stays at most 1024 deep: the dense
    # 4096^2 product at M = 128 keeps 128 x 64 tiles
    assert pifa.pifa_gemm_plan(128, 4096, 4096) == (128, 64, 4)
    assert pifa.pifa_gemm_plan(64, 4096, 4096) == (64, 64, 4)
    with pytest.raises(pifa.PifaError):
        pifa.pifa_gemm_plan(0, 2048, 4096)
