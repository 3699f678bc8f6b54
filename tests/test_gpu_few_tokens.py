"""The fused few-token kernel at the edges of its ranges: token panels of 16, channel tiles that end past the matrix,
one to three rotation blocks per wave (the last wave's share incomplete), int8 / 6-bit / int4 weights, zero points."""
import pytest
import torch

from paper_2503_06564_amd import trdq, workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# (M, K, N): K = 128 one wave; 1536 / 1664 one -> two blocks per wave (13 blocks: the last wave holds one);
# 3072 / 3200 two -> three (25 blocks: 9 waves, the last holds one); 4608 the widest
SHAPES = [(1, 128, 16), (15, 256, 48), (16, 1152, 1152), (17, 1152, 272), (33, 1536, 80), (64, 1664, 144), (16, 3072, 272),
          (31, 3200, 48), (1, 4608, 1152), (80, 4608, 1152), (257, 1152, 144), (512, 384, 528)]


@pytest.mark.parametrize("wbits", [8, 6, 4])
@pytest.mark.parametrize("M,K,N", SHAPES)
def test_edges(oracle, M, K, N, wbits):
    Xb, W, d, bias = wl.small_case(700 + M, M, K, N, n_outliers=4)
    Wd, dd = gu.f32_to_dev(W), gu.f32_to_dev(d)
    w = trdq.prepare_weights(Wd, dd, wbits=wbits)
    buf = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device=gu.dev())
    Y = buf[:M]
    trdq.linear_fused(gu.bf16_to_dev(Xb), dd, w, Y, bias=gu.f32_to_dev(bias))
    torch.cuda.synchronize()
    assert (buf[M] == 7.0).all()                         # nothing past the last token
    Xq, sx = gu.gpu_rotate_quant(Xb, d)
    Yp, _ = gu.gpu_qgemm(w, Xq, sx, bias, N, debug=False)
    # the two paths order the rotation's sums differently: a code may differ by one step, which moves its row's
    # outputs by about s_x * s_w * |weight code|, 1e-3 x row absmax and less, and through the bf16 rounding many of them
    gu.assert_y_close(gu.bf16_to_host(Y), gu.bf16_to_host(Yp), "fused against the pair")
    codes, scales = w.export()
    group = 128 if wbits == 4 else None
    Xq_o, sx_o = oracle.rotate_quant(Xb, d)
    want = oracle.dequant(oracle.igemm(Xq_o, codes, group), sx_o, scales, bias)
    gu.assert_y_close(gu.bf16_to_host(Y), want, "fused against the oracle on the GPU's weight codes")


@pytest.mark.parametrize("M,K,N", [(1, 128, 16), (17, 1152, 272), (64, 1664, 144), (31, 3200, 48), (16, 4608, 1152)])
def test_edges_asym(M, K, N):
    Xb, W, d, bias = wl.small_case(800 + M, M, K, N, n_outliers=4)
    X, dd, bd = gu.bf16_to_dev(Xb), gu.f32_to_dev(d), gu.f32_to_dev(bias)
    w = trdq.prepare_weights(gu.f32_to_dev(W), dd)
    Y, Yp = (torch.empty((M, N), dtype=torch.bfloat16, device=gu.dev()) for _ in range(2))
    Xq = torch.empty((M, K), dtype=torch.int8, device=gu.dev())
    sx, zc = torch.empty(M, device=gu.dev()), torch.empty(M, dtype=torch.int32, device=gu.dev())
    trdq.linear_fused_asym(X, dd, w, Y, bias=bd)
    trdq.rotate_quant_asym(X, dd, Xq, sx, zc)
    trdq.qgemm_asym(w, Xq, sx, zc, Yp, bias=bd)
    gu.assert_y_close(gu.bf16_to_host(Y), gu.bf16_to_host(Yp), "fused asymmetric against the pair")


# one and two blocks with workgroups for several per compute unit: each number of channel tiles that such a grid takes
# (1, 2, 3, 5), token panels and channel tiles incomplete
@pytest.mark.parametrize("M,K,N", [(497, 128, 496), (700, 128, 528), (1000, 128, 528), (1300, 128, 816),
                                   (700, 256, 528), (1001, 256, 528), (1300, 256, 816)])
@pytest.mark.parametrize("form", ["w8", "w4", "asym"])
def test_narrow_rows_many_workgroups(M, K, N, form):
    Xb, W, d, bias = wl.small_case(850 + M, M, K, N, n_outliers=4)
    X, dd, bd = gu.bf16_to_dev(Xb), gu.f32_to_dev(d), gu.f32_to_dev(bias)
    w = trdq.prepare_weights(gu.f32_to_dev(W), dd, wbits=4 if form == "w4" else 8)
    buf = torch.full((M + 1, N), 7.0, dtype=torch.bfloat16, device=gu.dev())
    Y, Yp = buf[:M], torch.empty((M, N), dtype=torch.bfloat16, device=gu.dev())
    Xq = torch.empty((M, K), dtype=torch.int8, device=gu.dev())
    sx, zc = torch.empty(M, device=gu.dev()), torch.empty(M, dtype=torch.int32, device=gu.dev())
    if form == "asym":
        trdq.linear_fused_asym(X, dd, w, Y, bias=bd)
        trdq.rotate_quant_asym(X, dd, Xq, sx, zc)
        trdq.qgemm_asym(w, Xq, sx, zc, Yp, bias=bd)
    else:
        trdq.linear_fused(X, dd, w, Y, bias=bd)
        trdq.rotate_quant(X, dd, Xq, sx)
        trdq.qgemm(w, Xq, sx, Yp, bias=bd)
    torch.cuda.synchronize()
    assert (buf[M] == 7.0).all()
    gu.assert_y_close(gu.bf16_to_host(Y), gu.bf16_to_host(Yp), "fused against the pair")
