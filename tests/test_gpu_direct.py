"""The product for launches with few output tiles (weights straight into registers, activations through areas of the waves'
own, K split over the waves) at the edges of its tiles, against exact integer sums and the oracle's epilogue on the GPU's own codes."""
import numpy as np
import pytest
import torch

from paper_2503_06564_amd import trdq, workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# every tile of the table, from both sides of its remainders: one unit per wave up to K = 1536, two to three beyond
# (13 units: 7 waves, the last with one; 25 units: 9 waves, the last with one), K = 128 with a single wave
SHAPES = [(1, 128, 16), (15, 256, 48), (17, 1152, 16), (16, 1152, 4608), (65, 1152, 1168), (129, 1152, 1152),
          (250, 768, 2304), (500, 1152, 1136), (33, 1664, 80), (1, 4608, 1152), (63, 3200, 272), (200, 4608, 1152),
          (769, 4608, 1152), (1000, 3072, 768), (2047, 256, 512)]


@pytest.mark.parametrize("M,K,N", SHAPES)
@pytest.mark.parametrize("asym", [False, True])
def test_edges(oracle, M, K, N, asym):
    Xb, W, d, bias = wl.small_case(900 + M, M, K, N, n_outliers=4)
    w = trdq.prepare_weights(gu.f32_to_dev(W), gu.f32_to_dev(d))
    X, dd = gu.bf16_to_dev(Xb), gu.f32_to_dev(d)
    Xq = torch.empty((M, K), dtype=torch.int8, device=gu.dev())
    sx = torch.empty(M, device=gu.dev())
    zc = torch.empty(M, dtype=torch.int32, device=gu.dev())
    buf = torch.full((M + 1, N + 8), 7.0, dtype=torch.bfloat16, device=gu.dev())
    Y = buf[:M, :N]
    acc = torch.full((M, N), -7, dtype=torch.int32, device=gu.dev())
    for debug in (acc, None):
        buf.fill_(7.0)
        if asym:
            trdq.rotate_quant_asym(X, dd, Xq, sx, zc, warm=w)
            trdq.qgemm_asym(w, Xq, sx, zc, Y, bias=gu.f32_to_dev(bias), acc_debug=debug)
        else:
            trdq.rotate_quant(X, dd, Xq, sx, warm=w)
            trdq.qgemm(w, Xq, sx, Y, bias=gu.f32_to_dev(bias), acc_debug=debug)
    torch.cuda.synchronize()
    assert (buf[M] == 7.0).all() and (buf[:, N:] == 7.0).all()      # nothing outside the output
    codes, scales = w.export()
    q = Xq.cpu().numpy().astype(np.float64)
    if asym:
        q = q + zc.cpu().numpy()[:, None]                            # q - z, exact in float64 as the sums are
    want = (q @ codes.astype(np.float64)).astype(np.int32)
    assert np.array_equal(acc.cpu().numpy(), want), "int32 accumulators differ"
    y = oracle.dequant(want, sx.cpu().numpy(), scales, bias)
    gu.assert_y_same_codes(gu.bf16_to_host(Y), y, "Y (same codes)")


# one and two units with workgroups for many per compute unit (the largest grids that this kernel takes), and widths of
# whole 128-channel tiles on both sides of the line to the kernels with tiles in LDS
@pytest.mark.parametrize("M,K,N,tile", [(4090, 128, 256, 0), (2040, 128, 496, 0), (2040, 256, 512, 1), (1010, 256, 1168, 1),
                                        (512, 1664, 1536, 4), (640, 1664, 1536, 4), (1024, 1664, 1536, -1), (1024, 3072, 1536, -1)])
@pytest.mark.parametrize("asym", [False, True])
def test_edges_of_the_choice(oracle, M, K, N, tile, asym):
    if asym and K == 3072:
        tile = 4                         # with zero points the line lies lower
    assert gu.library_rule("_ZN4trdq4gemm18qgemm8_direct_tileEliib", M, K, N, asym) == tile
    test_edges(oracle, M, K, N, asym)


# int4: one and two groups (no other tiled kernel takes them), one round of waves, several with a last round that is full
# (18, 36 groups), short (13, 25: some waves without a group), and the 64-token tiles from one tile on
SHAPES4 = [(1, 128, 16), (33, 256, 48), (17, 1152, 80), (31, 1536, 64), (40, 1664, 96), (65, 2304, 32), (50, 3200, 144),
           (1, 4608, 1152), (64, 384, 128), (129, 1152, 304), (250, 4608, 144), (1000, 512, 272)]


@pytest.mark.parametrize("M,K,N", SHAPES4)
@pytest.mark.parametrize("variant", [8, 9, 10, 11, "asym"])
def test_int4_edges(oracle, M, K, N, variant):
    """Group sums exact, outputs bit for bit those of the ring kernel (the folds keep its order)."""
    asym = variant == "asym"
    Xb, W, d, bias = wl.small_case(950 + M, M, K, N, n_outliers=4)
    w = trdq.prepare_weights(gu.f32_to_dev(W), gu.f32_to_dev(d), wbits=4)
    X, dd, bd = gu.bf16_to_dev(Xb), gu.f32_to_dev(d), gu.f32_to_dev(bias)
    Xq = torch.empty((M, K), dtype=torch.int8, device=gu.dev())
    sx = torch.empty(M, device=gu.dev())
    zc = torch.empty(M, dtype=torch.int32, device=gu.dev())
    if asym:
        trdq.rotate_quant_asym(X, dd, Xq, sx, zc, warm=w)
    else:
        trdq.rotate_quant(X, dd, Xq, sx, warm=w)
    buf = torch.full((M + 1, N + 8), 7.0, dtype=torch.bfloat16, device=gu.dev())
    Y, ring = buf[:M, :N], torch.empty((M, N), dtype=torch.bfloat16, device=gu.dev())
    acc = torch.full((K // 128, M, N), -7, dtype=torch.int32, device=gu.dev())
    try:
        if asym:                         # takes the library's choice
            trdq.qgemm_asym(w, Xq, sx, zc, Y, bias=bd, acc_debug=acc)
            buf.fill_(7.0)
            trdq.qgemm_asym(w, Xq, sx, zc, Y, bias=bd)
        else:
            trdq.qgemm_set_variant(6)
            trdq.qgemm(w, Xq, sx, ring, bias=bd)
            trdq.qgemm_set_variant(variant)
            trdq.qgemm(w, Xq, sx, Y, bias=bd, acc_debug=acc)
            buf.fill_(7.0)
            trdq.qgemm(w, Xq, sx, Y, bias=bd)
    finally:
        trdq.qgemm_set_variant(-1)
    torch.cuda.synchronize()
    assert (buf[M] == 7.0).all() and (buf[:, N:] == 7.0).all()      # nothing outside the output
    codes, scales = w.export()
    q = Xq.cpu().numpy().astype(np.float64)
    want = np.stack([q[:, g:g + 128] @ codes[g:g + 128].astype(np.float64) for g in range(0, K, 128)]).astype(np.int32)
    assert np.array_equal(acc.cpu().numpy(), want), "int32 group sums differ"
    if not asym:
        assert torch.equal(Y, ring)
        return
    z = zc.cpu().numpy().astype(np.float64)
    sums = want.astype(np.float64) + z[None, :, None] * codes.reshape(K // 128, 128, N).sum(axis=1)[:, None, :]
    y = (sums * scales[:, None, :]).sum(axis=0) * sx.cpu().numpy().astype(np.float64)[:, None] + bias
    got = Y.float().cpu().numpy().astype(np.float64)
    # one bf16 step of the value, and the float32 sums' part that the zero-point term cancels (up to 255 / range)
    assert (np.abs(got - y) <= 2.0 ** -8 * np.abs(y) + 1e-4 * np.abs(y).max(axis=1, keepdims=True)).all()
