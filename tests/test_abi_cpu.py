"""C-ABI checks that need no GPU: the library loads, exports every function the header
declares, and every argument error is reported before any HIP call is made."""
import ctypes as C
import os
import re

import numpy as np
import pytest

from paper_2503_06564_amd import trdq

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = 0x10000          # a non-null, 64 KiB aligned address that is never dereferenced


def header_functions():
    text = open(os.path.join(ROOT, "include", "trdq.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(trdq_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    L = trdq.lib()
    names = header_functions()
    assert len(names) >= 20
    for name in names:
        assert hasattr(L, name), name
    assert sorted(trdq.SYMBOLS) == names          # the binding covers the whole header
    assert L.trdq_abi_version() == 100
    assert trdq.status_str(trdq.OK) == "ok"
    assert "unsupported" in trdq.status_str(trdq.ERR_UNSUPPORTED)


def test_table_default_and_explicit():
    t = trdq.Table(20, 5)
    assert [t.lookup(s) for s in range(20)] == [s // 4 for s in range(20)]
    assert t.sizes() == (20, 5)
    t2 = trdq.Table(50, 10)
    assert [t2.lookup(s) for s in range(50)] == [s // 5 for s in range(50)]
    t3 = trdq.Table(7, 3)
    sizes = np.bincount([t3.lookup(s) for s in range(7)])
    assert sizes.max() - sizes.min() <= 1
    t4 = trdq.Table(4, 2, [1, 0, 1, 0])
    assert [t4.lookup(s) for s in range(4)] == [1, 0, 1, 0]


@pytest.mark.parametrize("args", [(0, 1), (5, 0), (3, 5), (-1, 1)])
def test_table_bad_sizes(args):
    with pytest.raises(trdq.TrdqError) as e:
        trdq.Table(*args)
    assert e.value.status == trdq.ERR_RANGE


def test_table_errors():
    with pytest.raises(trdq.TrdqError) as e:
        trdq.Table(4, 2, [0, 1, 2, 0])
    assert e.value.status == trdq.ERR_RANGE
    t = trdq.Table(4, 2)
    for step in (-1, 4):
        with pytest.raises(trdq.TrdqError) as e:
            t.lookup(step)
        assert e.value.status == trdq.ERR_RANGE
    L = trdq.lib()
    assert L.trdq_table_create(4, 2, None, None) == trdq.ERR_NULL
    g = C.c_int()
    assert L.trdq_table_lookup(None, 0, C.byref(g)) == trdq.ERR_NULL
    L.trdq_table_destroy(None)                     # no-op


def test_prepare_weights_argument_errors():
    L = trdq.lib()
    h = C.c_void_p()
    call = lambda W, K, N, block, wbits, out: L.trdq_prepare_weights(W, K, N, None, block, wbits, None, out)
    assert call(FAKE, 128, 16, 128, 8, None) == trdq.ERR_NULL
    assert call(None, 128, 16, 128, 8, C.byref(h)) == trdq.ERR_NULL
    assert call(FAKE, 128, 16, 64, 8, C.byref(h)) == trdq.ERR_UNSUPPORTED
    assert call(FAKE, 128, 16, 128, 5, C.byref(h)) == trdq.ERR_UNSUPPORTED
    assert call(FAKE, 100, 16, 128, 8, C.byref(h)) == trdq.ERR_SHAPE
    assert call(FAKE, 0, 16, 128, 8, C.byref(h)) == trdq.ERR_SHAPE
    assert call(FAKE, 128, 0, 128, 8, C.byref(h)) == trdq.ERR_SHAPE
    assert call(FAKE, 128, 24, 128, 4, C.byref(h)) == trdq.ERR_SHAPE
    assert h.value is None


def test_rotate_quant_argument_errors():
    L = trdq.lib()
    rq = L.trdq_rotate_quant
    assert rq(None, 4, 128, 128, None, 128, FAKE, FAKE, None) == trdq.ERR_NULL
    assert rq(FAKE, 4, 128, 128, None, 128, None, FAKE, None) == trdq.ERR_NULL
    assert rq(FAKE, 4, 128, 128, None, 128, FAKE, None, None) == trdq.ERR_NULL
    assert rq(FAKE, 4, 128, 128, None, 64, FAKE, FAKE, None) == trdq.ERR_UNSUPPORTED
    assert rq(FAKE, -1, 128, 128, None, 128, FAKE, FAKE, None) == trdq.ERR_SHAPE
    assert rq(FAKE, 4, 120, 128, None, 128, FAKE, FAKE, None) == trdq.ERR_SHAPE
    assert rq(FAKE, 4, 256, 128, None, 128, FAKE, FAKE, None) == trdq.ERR_SHAPE      # ldx < K
    assert rq(FAKE, 4, 128, 132, None, 128, FAKE, FAKE, None) == trdq.ERR_SHAPE      # ldx % 8
    assert rq(FAKE + 2, 4, 128, 128, None, 128, FAKE, FAKE, None) == trdq.ERR_SHAPE  # alignment
    assert rq(FAKE, 4, 128, 128, FAKE + 4, 128, FAKE, FAKE, None) == trdq.ERR_SHAPE
    assert rq(FAKE, 4, 128 * 65, 128 * 65, None, 128, FAKE, FAKE, None) == trdq.ERR_UNSUPPORTED
    assert rq(FAKE, 0, 128, 128, None, 128, FAKE, FAKE, None) == trdq.OK             # empty input


def test_qgemm_and_fused_argument_errors():
    L = trdq.lib()
    assert L.trdq_qgemm(None, FAKE, FAKE, 4, None, FAKE, 16, None, None) == trdq.ERR_NULL
    assert L.trdq_linear_fused(FAKE, 4, 128, None, None, None, FAKE, 16, None) == trdq.ERR_NULL
    assert L.trdq_qgemm_set_variant(10_000) == trdq.ERR_RANGE
    assert L.trdq_qgemm_set_variant(-1) == trdq.OK
    assert L.trdq_qgemm_num_variants() >= 1
    assert L.trdq_weights_info(None, None, None, None) == trdq.ERR_NULL
    assert L.trdq_weights_export(None, None, None) == trdq.ERR_NULL
    assert L.trdq_weights_export_packed(None, FAKE) == trdq.ERR_NULL
    L.trdq_weights_destroy(None)


def test_layer_argument_errors():
    L = trdq.lib()
    t = trdq.Table(10, 5)
    h = C.c_void_p()
    assert L.trdq_layer_create(None, 128, 16, 8, C.byref(h)) == trdq.ERR_NULL
    assert L.trdq_layer_create(t.handle, 128, 16, 8, None) == trdq.ERR_NULL
    assert L.trdq_layer_create(t.handle, 128, 16, 5, C.byref(h)) == trdq.ERR_UNSUPPORTED
    assert L.trdq_layer_create(t.handle, 130, 16, 8, C.byref(h)) == trdq.ERR_SHAPE
    layer = trdq.Layer(t, 256, 32, 8)
    assert L.trdq_layer_set_group(layer.handle, 5, None, FAKE, None) == trdq.ERR_RANGE
    assert L.trdq_layer_set_group(layer.handle, -1, None, FAKE, None) == trdq.ERR_RANGE
    assert L.trdq_layer_set_group(layer.handle, 0, None, None, None) == trdq.ERR_NULL
    fwd = L.trdq_layer_forward
    assert fwd(layer.handle, 10, FAKE, 4, None, FAKE, 0, FAKE, FAKE, None) == trdq.ERR_RANGE
    assert fwd(layer.handle, -1, FAKE, 4, None, FAKE, 1, None, None, None) == trdq.ERR_RANGE
    assert fwd(layer.handle, 3, FAKE, 4, None, FAKE, 1, None, None, None) == trdq.ERR_MISMATCH   # group not set
    w = C.c_void_p()
    assert L.trdq_layer_weights(layer.handle, 0, C.byref(w)) == trdq.ERR_MISMATCH
    assert L.trdq_layer_weights(layer.handle, 7, C.byref(w)) == trdq.ERR_RANGE
    layer.close()
    L.trdq_layer_destroy(None)


# ---- zigzag permutation (host-side entry point: checked here against the oracle) ----------

@pytest.mark.parametrize("K", [128, 1152, 4608])
def test_zigzag_matches_oracle(oracle, K):
    rng = np.random.default_rng(K)
    mag = np.abs(rng.standard_normal(K)).astype(np.float32)
    mag[rng.choice(K, size=max(1, K // 144), replace=False)] *= 40.0
    mag[5 % K] = mag[17 % K]                                     # a tie: channel order decides
    got = trdq.zigzag_permutation(mag)
    want = oracle.zigzag(mag.astype(np.float64), 128)
    assert np.array_equal(got, want)


def test_zigzag_argument_errors():
    L = trdq.lib()
    mag = np.ones(256, dtype=np.float32)
    perm = np.empty(256, dtype=np.int32)
    assert L.trdq_zigzag_permutation(None, 256, 128, perm.ctypes.data) == trdq.ERR_NULL
    assert L.trdq_zigzag_permutation(mag.ctypes.data, 256, 128, None) == trdq.ERR_NULL
    assert L.trdq_zigzag_permutation(mag.ctypes.data, 200, 128, perm.ctypes.data) == trdq.ERR_SHAPE
    assert L.trdq_zigzag_permutation(mag.ctypes.data, 0, 128, perm.ctypes.data) == trdq.ERR_SHAPE
    assert L.trdq_zigzag_permutation(mag.ctypes.data, 256, 0, perm.ctypes.data) == trdq.ERR_SHAPE
    for bad in (np.nan, np.inf, -np.inf):              # a magnitude that cannot be ordered
        m2 = mag.copy(); m2[17] = bad
        assert L.trdq_zigzag_permutation(m2.ctypes.data, 256, 128, perm.ctypes.data) == trdq.ERR_RANGE


def test_rpr_argument_errors_before_any_gpu_call():
    L = trdq.lib()
    out = C.c_void_p()
    # NULL permutation, then the same checks as the one-rotation entry points
    assert L.trdq_prepare_weights_rpr(0x1000, 256, 64, None, None, 128, 8, None, C.byref(out)) == trdq.ERR_NULL
    assert L.trdq_prepare_weights_rpr(0x1000, 200, 64, None, 0x2000, 128, 8, None, C.byref(out)) == trdq.ERR_SHAPE
    assert L.trdq_prepare_weights_rpr(0x1000, 256, 64, None, 0x2000, 128, 5, None, C.byref(out)) == trdq.ERR_UNSUPPORTED
    assert L.trdq_rotate_quant_rpr(0x1000, 4, 256, 256, None, None, 128, 0x2000, 0x3000, None, None) == trdq.ERR_NULL
    assert L.trdq_rotate_quant_rpr(0x1000, 4, 256, 256, None, 0x4000, 64, 0x2000, 0x3000, None, None) == trdq.ERR_UNSUPPORTED
    assert L.trdq_rotate_quant_rpr(0x1000, 4, 200, 256, None, 0x4000, 128, 0x2000, 0x3000, None, None) == trdq.ERR_SHAPE
    assert L.trdq_rotate_quant_rpr(0x1000, 4, 256, 256, None, 0x4004, 128, 0x2000, 0x3000, None, None) == trdq.ERR_SHAPE
    assert L.trdq_rotate_quant_rpr(0x1000, 4, 128 * 37, 128 * 37, None, 0x4000, 128, 0x2000, 0x3000, None, None) == trdq.ERR_UNSUPPORTED
    assert L.trdq_rotate_quant_rpr(0x1000, 0, 256, 256, None, 0x4000, 128, None, None, None, None) == trdq.OK


def test_calibration_argument_errors_before_any_gpu_call():
    L = trdq.lib()
    assert L.trdq_channel_absmax(0x1000, 4, 256, 256, None, 1, 128, None, None) == trdq.ERR_NULL
    assert L.trdq_channel_absmax(None, 4, 256, 256, None, 1, 128, 0x2000, None) == trdq.ERR_NULL
    assert L.trdq_channel_absmax(0x1000, 4, 200, 256, None, 1, 128, 0x2000, None) == trdq.ERR_SHAPE
    assert L.trdq_channel_absmax(0x1000, 4, 256, 256, None, 1, 64, 0x2000, None) == trdq.ERR_UNSUPPORTED
    assert L.trdq_weight_row_absmax(None, 256, 64, 0x2000, None) == trdq.ERR_NULL
    assert L.trdq_weight_row_absmax(0x1000, 0, 64, 0x2000, None) == trdq.ERR_SHAPE
    assert L.trdq_smooth_diag(None, 0x1000, 256, 0.5, 0x2000, None) == trdq.ERR_NULL
    assert L.trdq_smooth_diag(0x1000, 0x1000, 0, 0.5, 0x2000, None) == trdq.ERR_SHAPE
    assert L.trdq_smooth_diag(0x1000, 0x1000, 256, 1.5, 0x2000, None) == trdq.ERR_RANGE
    assert L.trdq_smooth_diag(0x1000, 0x1000, 256, float("nan"), 0x2000, None) == trdq.ERR_RANGE


def test_asym_argument_errors_before_any_gpu_call():
    L = trdq.lib()
    assert L.trdq_rotate_quant_asym(0x1000, 4, 256, 256, None, 128, 0x2000, 0x3000, None, None, None) == trdq.ERR_NULL
    assert L.trdq_rotate_quant_asym(0x1000, 4, 200, 256, None, 128, 0x2000, 0x3000, 0x4000, None, None) == trdq.ERR_SHAPE
    assert L.trdq_rotate_quant_asym(0x1000, 4, 128 * 37, 128 * 37, None, 128, 0x2000, 0x3000, 0x4000, None, None) == trdq.ERR_UNSUPPORTED
    assert L.trdq_rotate_quant_asym(0x1000, 0, 256, 256, None, 128, None, None, None, None, None) == trdq.OK
    assert L.trdq_qgemm_asym(None, 0x1000, 0x2000, 0x3000, 4, None, 0x4000, 64, None, None) == trdq.ERR_NULL


def test_bits_argument_errors_before_any_gpu_call():
    L = trdq.lib()
    assert L.trdq_rotate_quant_bits(0x1000, 4, 256, 256, None, 128, 6, None, 0x3000, None, None) == trdq.ERR_NULL
    assert L.trdq_rotate_quant_bits(0x1000, 4, 256, 256, None, 128, 9, 0x2000, 0x3000, None, None) == trdq.ERR_RANGE
    assert L.trdq_rotate_quant_bits(0x1000, 4, 256, 256, None, 128, 1, 0x2000, 0x3000, None, None) == trdq.ERR_RANGE
    assert L.trdq_rotate_quant_bits(0x1000, 4, 128 * 37, 128 * 37, None, 128, 6, 0x2000, 0x3000, None, None) == trdq.ERR_UNSUPPORTED
    assert L.trdq_rotate_quant_bits(0x1000, 0, 256, 256, None, 128, 6, None, None, None, None) == trdq.OK
    out = trdq.C.c_void_p()
    assert L.trdq_prepare_weights(0x1000, 256, 64, None, 128, 5, None, trdq.C.byref(out)) == trdq.ERR_UNSUPPORTED


def test_attention_share_host_side(oracle):
    L = trdq.lib()
    assert L.trdq_cosine_similarity(None, 0x1000, 1, 64, 64, 64, 0x2000, 0x3000, None) == trdq.ERR_NULL
    assert L.trdq_cosine_similarity(0x1000, 0x2000, 0, 64, 64, 64, 0x3000, 0x4000, None) == trdq.ERR_SHAPE
    assert L.trdq_cosine_similarity(0x1000, 0x2000, 2, 64, 60, 64, 0x3000, 0x4000, None) == trdq.ERR_SHAPE
    assert L.trdq_cosine_similarity(0x1000, 0x2000, 2, 60, 68, 64, 0x3000, 0x4000, None) == trdq.ERR_SHAPE
    assert L.trdq_cosine_similarity(0x1008, 0x2000, 1, 64, 64, 64, 0x3000, 0x4000, None) == trdq.ERR_SHAPE
    # the variant that allocates nothing: the same checks, and its fixed maximum, before any device work
    assert L.trdq_cosine_similarity_static(None, 0x1000, 1, 64, 64, 64, 0x3000, None) == trdq.ERR_NULL
    assert L.trdq_cosine_similarity_static(0x1000, 0x2000, 0, 64, 64, 64, 0x4000, None) == trdq.ERR_SHAPE
    assert L.trdq_cosine_similarity_static(0x1000, 0x2000, 2, 64, 60, 64, 0x4000, None) == trdq.ERR_SHAPE
    assert L.trdq_cosine_similarity_static(0x1008, 0x2000, 1, 64, 64, 64, 0x4000, None) == trdq.ERR_SHAPE
    assert L.trdq_cosine_similarity_static(0x1000, 0x2000, trdq.COSINE_STATIC_MAX_SEG + 1, 64, 64, 64, 0x4000,
                                           None) == trdq.ERR_RANGE
    rng = np.random.default_rng(3)
    sim = rng.uniform(0.8, 1.0, (20, 28)).astype(np.float32)
    sim[:, 0] = 0.99; sim[:, 27] = 0.97; sim[7, 5] = np.nan
    for thr in (0.9, 0.95, 0.97, 0.999):
        got = trdq.share_plan(sim, thr)
        want = oracle.share_plan(np.nan_to_num(sim, nan=-2.0), np.float32(thr))
        assert np.array_equal(got, want)
    assert trdq.share_plan(sim, 0.95)[0] == 1 and trdq.share_plan(sim, 0.95)[5] == 0
    with pytest.raises(trdq.TrdqError):
        trdq.share_plan(sim, 1.5)


def test_yardstick_argument_errors_before_any_gpu_call():
    L = trdq.lib()
    assert L.trdq_peak_mfma_i8(None, 256, 4, 10, None, None) == trdq.ERR_NULL
    assert L.trdq_peak_mfma_i8(0x1000, 0, 4, 10, None, None) == trdq.ERR_RANGE
    assert L.trdq_peak_mfma_i8(0x1000, 256, 9, 10, None, None) == trdq.ERR_RANGE
    assert L.trdq_peak_mfma_i8(0x1000, 256, 4, 0, None, None) == trdq.ERR_RANGE
    assert L.trdq_peak_mfma_i8(0x1000, 256, 4, (1 << 20) + 1, None, None) == trdq.ERR_RANGE
    assert L.trdq_peak_mfma_i8(0x1002, 256, 4, 10, None, None) == trdq.ERR_SHAPE
    assert L.trdq_peak_mfma_i8_data(None, 256, 4, 10, None, None) == trdq.ERR_NULL
    assert L.trdq_peak_mfma_i8_data(0x1000, 256, 9, 10, None, None) == trdq.ERR_RANGE
    assert L.trdq_peak_stream(0x1000, 0x2000, 12, None) == trdq.ERR_SHAPE
    assert L.trdq_peak_stream(0x1000, 0x2000, -8, None) == trdq.ERR_SHAPE
    assert L.trdq_peak_stream(None, 0x2000, 8, None) == trdq.ERR_NULL
    assert L.trdq_peak_stream(0x1008, 0x2000, 8, None) == trdq.ERR_SHAPE
    assert L.trdq_peak_stream(0x1000, 0x2004, 8, None) == trdq.ERR_SHAPE
    assert L.trdq_peak_stream(None, None, 0, None) == trdq.OK


def test_dense_rotation_argument_errors_before_any_gpu_call():
    L = trdq.lib()
    out = C.c_void_p()
    assert L.trdq_rotation_create(None, None, 256, 128, None, C.byref(out)) == trdq.ERR_NULL
    assert L.trdq_rotation_create(0x1000, None, 256, 128, None, None) == trdq.ERR_NULL
    assert L.trdq_rotation_create(0x1000, None, 200, 128, None, C.byref(out)) == trdq.ERR_SHAPE
    assert L.trdq_rotation_create(0x1000, None, 256, 64, None, C.byref(out)) == trdq.ERR_UNSUPPORTED
    assert L.trdq_rotation_create(0x1000, None, 128 * 37, 128, None, C.byref(out)) == trdq.ERR_UNSUPPORTED
    assert L.trdq_rotate_quant_dense(0x1000, 4, 256, None, 0x2000, 0x3000, None) == trdq.ERR_NULL
    assert L.trdq_prepare_weights_dense(0x1000, 256, 64, None, 8, None, C.byref(out)) == trdq.ERR_NULL
    L.trdq_rotation_destroy(None)


def test_greedy_rotation_argument_errors_before_any_gpu_call():
    L = trdq.lib()
    call = L.trdq_greedy_rotation
    assert call(0x1000, 16, 256, 256, None, 128, None, 4, 0x3000, None, None) == trdq.ERR_NULL
    assert call(0x1000, 16, 256, 256, None, 128, 0x2000, 4, None, None, None) == trdq.ERR_NULL
    assert call(0x1000, 16, 200, 256, None, 128, 0x2000, 4, 0x3000, None, None) == trdq.ERR_SHAPE
    assert call(0x1000, 0, 256, 256, None, 128, 0x2000, 4, 0x3000, None, None) == trdq.ERR_SHAPE
    assert call(0x1000, 16, 256, 256, None, 128, 0x2000, 0, 0x3000, None, None) == trdq.ERR_SHAPE
    assert call(0x1000, 16, 256, 256, None, 128, 0x2000, 5000, 0x3000, None, None) == trdq.ERR_UNSUPPORTED


def test_dense_calibration_argument_errors_before_any_gpu_call():
    L = trdq.lib()
    assert L.trdq_channel_absmax_dense(0x1000, 4, 256, None, 0x2000, None) == trdq.ERR_NULL
    assert L.trdq_greedy_rotation_second(0x1000, 4, 256, None, 0x2000, 0x3000, 4, 0x4000, None, None) == trdq.ERR_NULL
    out = C.c_void_p()
    assert L.trdq_prepare_weights_dense_rpr(0x1000, 256, 64, None, 0x2000, None, 8, None, C.byref(out)) == trdq.ERR_NULL
    assert L.trdq_rotate_quant_dense_rpr(0x1000, 4, 256, None, 0x2000, None, 0x3000, 0x4000, None) == trdq.ERR_NULL
    assert L.trdq_rotate_quant_dense_rpr_ws(0x1000, 4, 256, None, 0x2000, None, 0x3000, 0x4000, 0x5000, 64, None) == trdq.ERR_NULL


def test_dense_rpr_workspace_size():
    n = trdq.rotate_quant_dense_rpr_ws_nbytes
    assert n(4096, 4608) == 4 * 4609 * 4096          # K rows of once-rotated values and one of maxima
    assert n(33, 2304) == 4 * 2305 * 64              # tokens rounded up to 32
    assert n(1, 1664) == 4 * 1665 * 32
    assert n(100, 1536) == 0 and n(16383, 128) == 0  # up to 12 blocks: no workspace below 16384 tokens
    assert n(16384, 1152) == 4 * 1153 * 16384 and n(16385, 128) == 4 * 129 * 16416
    assert n(0, 4608) == 0 and n(-3, 4608) == 0 and n(8, 4600) == 0 and n(8, 0) == 0


def test_asym_weight_calls_check_arguments_before_any_gpu_call():
    L = trdq.lib()
    import ctypes as C
    h = C.c_void_p()
    assert L.trdq_prepare_weights_asym(None, 256, 16, None, 128, 8, None, C.byref(h)) == trdq.ERR_NULL
    assert L.trdq_prepare_weights_asym(0x1000, 256, 16, None, 128, 4, None, C.byref(h)) == trdq.ERR_UNSUPPORTED
    assert L.trdq_prepare_weights_asym(0x1000, 200, 16, None, 128, 8, None, C.byref(h)) == trdq.ERR_SHAPE
    assert L.trdq_prepare_weights_asym(0x1000, 256, 16, None, 128, 8, None, None) == trdq.ERR_NULL
    assert L.trdq_weights_export_zero_points(None, 0x1000) == trdq.ERR_NULL
    assert L.trdq_qgemm_asym_weights(None, 0x1000, 0x2000, None, 0x3000, 4, None, 0x4000, 16, None, None) == trdq.ERR_NULL


def test_fused_asym_checks_arguments_before_any_gpu_call():
    L = trdq.lib()
    assert L.trdq_linear_fused_asym(0x1000, 4, 256, None, None, None, 0x2000, 16, None) == trdq.ERR_NULL


def test_current_stream_without_the_private_lookup(monkeypatch):
    """A torch without its private raw-stream function: the public one answers, for the stream that is current then."""
    import types

    import torch
    streams = iter([5, 77, 78])
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=next(streams)))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch, "_C", types.SimpleNamespace())
    monkeypatch.setattr(trdq, "_raw_stream", None)
    assert trdq._stream(None) == 77 and trdq._stream(None) == 78
    assert trdq._stream(9) == 9 and trdq._stream(types.SimpleNamespace(cuda_stream=11)) == 11


def test_phase_probe_asks_for_kernels_that_record():
    """int4 products of more than two 128 x 128 tiles for each of 256 compute units go to a kernel without time stamps."""
    from paper_2503_06564_amd import probe_phases
    int4 = [c for c in probe_phases.CASES if c[0] == 4]
    assert int4 and all(M * N <= 512 * 128 * 128 for _, M, K, N in int4)
