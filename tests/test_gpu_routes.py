"""Kernels that the library's choice takes for shapes which most other tests leave to the kernels for few tokens or tiles.
Each test asserts first that the rule sends its shape there."""
import numpy as np
import pytest
import torch

import gpu_util as gu
from paper_2503_06564_amd import trdq, workloads as wl
from test_gpu_parity import _linear_case

pytestmark = pytest.mark.gpu


def _direct(M, K, N, asym=False):
    return gu.library_rule("_ZN4trdq4gemm18qgemm8_direct_tileEliib", M, K, N, asym)


def _rows(M, K, N, asym=False):
    return gu.library_rule("_ZN4trdq4gemm15tiled_rows_paysEliib", M, K, N, asym) & 1


def _rows4(M, K, N):
    return not gu.library_rule("_ZN4trdq4gemm18qgemm4_direct_tileElii", M, K, N) >= 0 and gu.library_rule("_ZN4trdq4gemm16tiled4_rows_paysElii", M, K, N) & 1


# whole panels and the remaining rows in two launches: rows of Y that are 8-byte aligned only (M % 256 below and above 128), and
# many ragged tokens at a width that is no multiple of 144 (heads of 256- and of 128-token panels; 16 and 112 rows left)
@pytest.mark.parametrize("M,K,N,pad", [(1500, 1152, 1136, 4), (2100, 640, 1040, 12), (14096, 384, 400, 0), (14192, 256, 528, 0)])
def test_ragged_tokens_in_two_launches(oracle, M, K, N, pad):
    assert _direct(M, K, N) == -1 and (pad % 8 != 0 or not _rows(M, K, N))
    _linear_case(oracle, 15, M, K, N, 8, -1, ldy=N + pad)


# whole 128 x 144 tiles, more than one per compute unit: one round of tall and short row-major tiles, unless three tiles per unit take
# more tall ones than there are units (6144 x 2304: 264) or all of them are short and K is long
@pytest.mark.parametrize("M,K,N,rows", [(4096, 1152, 3456, True), (6144, 768, 2160, True), (6144, 768, 2304, False), (12288, 1152, 1152, False),
                                        (8192, 768, 2304, True), (8192, 1664, 1152, True), (8192, 1792, 1152, False), (4096, 2176, 2304, False)])
def test_whole_tiles_in_one_round(M, K, N, rows):
    assert bool(_rows(M, K, N)) == rows
    g = torch.Generator(device="cuda").manual_seed(N)
    w = trdq.prepare_weights(0.02 * torch.randn(K, N, generator=g, device="cuda"), None)
    Xq = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    acc, Y = torch.empty((M, N), dtype=torch.int32, device="cuda"), torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    trdq.qgemm(w, Xq, torch.ones(M, device="cuda"), Y, acc_debug=acc)
    want = Xq.double() @ torch.from_numpy(w.export()[0].astype(np.float64)).cuda()
    assert torch.equal(acc, want.int())


# int4, 64-token tiles of row-major codes: widened codes with few channel tiles side by side, packed ones beyond (the last tile of
# either kind ragged both ways)
@pytest.mark.parametrize("M,K,N,wide", [(1000, 1664, 1296, True), (2010, 384, 1168, True), (700, 512, 2320, True), (448, 512, 4608, False),
                                        (1000, 384, 3440, False), (3000, 640, 2000, False)])
def test_int4_copy_of_the_codes(M, K, N, wide):
    assert _rows4(M, K, N)
    assert bool(gu.library_rule("_ZN4trdq4gemm22tiled4_rows_reads_wideEli", M, N, 0) & 1) == wide
    g = torch.Generator(device="cuda").manual_seed(N)
    w = trdq.prepare_weights(0.02 * torch.randn(K, N, generator=g, device="cuda"), None, wbits=4)
    Xq = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    sx, bias = torch.rand(M, generator=g, device="cuda"), torch.randn(N, generator=g, device="cuda")
    acc = torch.empty((K // 128, M, N), dtype=torch.int32, device="cuda")
    Y, ring = (torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    trdq.qgemm(w, Xq, sx, Y, bias=bias, acc_debug=acc)
    codes = torch.from_numpy(w.export()[0].astype(np.float64)).cuda()
    want = torch.stack([Xq[:, k:k + 128].double() @ codes[k:k + 128] for k in range(0, K, 128)])
    assert torch.equal(acc, want.int())
    trdq.qgemm(w, Xq, sx, Y.fill_(7.0), bias=bias)
    try:
        trdq.qgemm_set_variant(6)                     # the ring kernel; the folds keep its order
        trdq.qgemm(w, Xq, sx, ring, bias=bias)
    finally:
        trdq.qgemm_set_variant(-1)
    assert torch.equal(Y, ring)


def test_int4_many_channel_tiles_are_no_slower_than_the_ring_kernel():
    """... which the widened codes made them: 62 us against 45 at 1344 x 4608 -> 4608, packed 44.  1.2 leaves room for a busy device."""
    M, K, N = 1344, 4608, 4608
    assert _rows4(M, K, N)
    w = trdq.prepare_weights(0.02 * torch.randn(K, N, device="cuda"), None, wbits=4)
    Xq = torch.randint(-127, 128, (M, K), device="cuda", dtype=torch.int8)
    sx, Y = torch.ones(M, device="cuda"), torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = {}
    try:
        for rep in range(8):
            for variant in (-1, 6):
                trdq.qgemm_set_variant(variant)
                start.record()
                for _ in range(20):
                    trdq.qgemm(w, Xq, sx, Y)
                end.record()
                torch.cuda.synchronize()
                best[variant] = min(best.get(variant, 1e9), start.elapsed_time(end))
    finally:
        trdq.qgemm_set_variant(-1)
    assert best[-1] < 1.2 * best[6], best


# the general fused kernel: panels of 64, 32 and 16 tokens (up to 12, 24 and 48 blocks) in each register form (3, 6, 9, 12 blocks per
# lane row), last panel and last channel tile incomplete
@pytest.mark.parametrize("M,K,N", [(1000, 384, 1168), (1001, 768, 1168), (1001, 1152, 1168), (1010, 1536, 1168), (1000, 1664, 400),
                                   (999, 3072, 272), (1000, 3200, 400), (100, 4736, 272), (37, 6144, 144)])
@pytest.mark.parametrize("form", ["w8", "w4", "asym"])
def test_general_fused_kernel(oracle, M, K, N, form):
    assert not gu.library_rule("_ZN4trdq22fused_takes_few_tokensElii", M, K, N) & 1
    wbits = 4 if form == "w4" else 8
    Xb, W, d, bias = wl.small_case(45, M, K, N, n_outliers=max(1, K // 144), outlier=40.0)
    w = trdq.prepare_weights(gu.f32_to_dev(W), gu.f32_to_dev(d), wbits=wbits)
    buf = torch.full((M + 1, N + 4), 7.0, dtype=torch.bfloat16, device=gu.dev())
    Y = buf[:M, :N]
    fused = trdq.linear_fused_asym if form == "asym" else trdq.linear_fused
    fused(gu.bf16_to_dev(Xb), gu.f32_to_dev(d), w, Y, bias=gu.f32_to_dev(bias))
    torch.cuda.synchronize()
    assert (buf[M] == 7.0).all() and (buf[:, N:] == 7.0).all()
    codes, _ = w.export()
    if form == "asym":
        ref = oracle.linear_asym(Xb, W, d, bias, exact_blas=True)
    else:
        ref = oracle.linear(Xb, W, d, bias, wbits=wbits, exact_blas=True)
    gu.assert_y_close(gu.bf16_to_host(Y), ref["Y"], "Y (fused, oracle end to end)",
                      *gu.narrow_code_masks(8, wbits, None, None, codes, ref["Wq"]))
    w.close()


# products with zero points: the 128 x 144 kernel whose two wave groups split K (an odd and an even number of units each), one
# workgroup per tile, two per compute unit, and the ring kernel (rows of Y that are 8-byte aligned only)
@pytest.mark.parametrize("M,K,N,pad", [(1280, 2432, 1152, 0), (1152, 4608, 1152, 0), (1024, 1280, 1152, 0), (4224, 640, 1152, 0),
                                       (1408, 1152, 1136, 4), (1500, 1152, 1136, 4)])
def test_products_with_zero_points(oracle, M, K, N, pad):
    assert _direct(M, K, N, True) == -1 and (pad % 8 != 0 or not _rows(M, K, N, True))
    Xb, W, d, bias = wl.small_case(42, M, K, N, n_outliers=max(1, K // 144), outlier=40.0)
    w = trdq.prepare_weights(gu.f32_to_dev(W), gu.f32_to_dev(d))
    Xq = torch.empty((M, K), dtype=torch.int8, device=gu.dev())
    sx, zc = torch.empty(M, device=gu.dev()), torch.empty(M, dtype=torch.int32, device=gu.dev())
    trdq.rotate_quant_asym(gu.bf16_to_dev(Xb), gu.f32_to_dev(d), Xq, sx, zc, warm=w)
    buf = torch.empty((M + 1, N + pad), dtype=torch.bfloat16, device=gu.dev())
    Y = buf[:M, :N]
    acc = torch.full((M, N), -7, dtype=torch.int32, device=gu.dev())
    for debug in (acc, None):
        buf.fill_(7.0)
        trdq.qgemm_asym(w, Xq, sx, zc, Y, bias=gu.f32_to_dev(bias), acc_debug=debug)
    torch.cuda.synchronize()
    assert (buf[M] == 7.0).all() and (buf[:, N:] == 7.0).all()
    codes, scales = w.export()
    q = Xq.cpu().numpy().astype(np.float64) + zc.cpu().numpy()[:, None]     # q - z, exact in float64 as the sums are
    want = (q @ codes.astype(np.float64)).astype(np.int32)
    assert np.array_equal(acc.cpu().numpy(), want), "int32 accumulators differ"
    y = oracle.dequant(want, sx.cpu().numpy(), scales, bias)
    gu.assert_y_same_codes(gu.bf16_to_host(Y), y, "Y (same codes)")
    w.close()
