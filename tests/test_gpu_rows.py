"""The tiled products on row-major codes (last tiles moved back onto whole ones) at the edges of their tiles, against
exact integer sums and the oracle's epilogue on the GPU's own codes."""
import numpy as np
import pytest
import torch

from paper_2503_06564_amd import trdq, workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

ROWS = trdq.qgemm_num_variants() - 2

# one tile; one token or channel past a tile; a last tile that repeats all but one row; K split over two wave pairs with
# an odd and an even number of steps each (1152, 1024, 4608); more tiles than compute units: tall and short tiles mixed
# (1152 -> 4608 at 2177), tall only (768 -> 4608 at 4097); 16-byte rows that start at any token (1300)
SHAPES = [(128, 128, 144), (129, 256, 160), (255, 1152, 288), (300, 1024, 304), (383, 4608, 448), (1300, 1152, 1136),
          (2177, 1152, 4608), (4097, 768, 4608), (1024, 768, 2304)]


@pytest.fixture(autouse=True)
def rows_variant():
    trdq.qgemm_set_variant(ROWS)
    yield
    trdq.qgemm_set_variant(-1)


@pytest.mark.parametrize("M,K,N", SHAPES)
@pytest.mark.parametrize("asym", [False, True])
def test_edges(oracle, M, K, N, asym):
    Xb, W, d, bias = wl.small_case(700 + M, M, K, N, n_outliers=4)
    w = trdq.prepare_weights(gu.f32_to_dev(W), gu.f32_to_dev(d))
    X, dd, bd = gu.bf16_to_dev(Xb), gu.f32_to_dev(d), gu.f32_to_dev(bias)
    Xq = torch.empty((M, K), dtype=torch.int8, device=gu.dev())
    sx_buf = torch.empty(M + 1, device=gu.dev())
    sx = sx_buf[1:]                                                  # token scales on a 4-byte boundary
    zc = torch.empty(M, dtype=torch.int32, device=gu.dev())
    buf = torch.empty((M + 1, N + 8), dtype=torch.bfloat16, device=gu.dev())
    Y = buf[:M, :N]
    acc = torch.full((M, N), -7, dtype=torch.int32, device=gu.dev())
    for debug in (acc, None):
        buf.fill_(7.0)
        if asym:
            trdq.rotate_quant_asym(X, dd, Xq, sx, zc, warm=w)
            trdq.qgemm_asym(w, Xq, sx, zc, Y, bias=bd, acc_debug=debug)
        else:
            trdq.rotate_quant(X, dd, Xq, sx, warm=w)
            trdq.qgemm(w, Xq, sx, Y, bias=bd, acc_debug=debug)
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


# tall tiles with 2, 4, 6 and 18 k-steps: the loop over all but the last two of them empty, once round, and more (the fixture asks for this
# form, so that zero points take it at whole tiles too, where the library's choice is another kernel from K = 1024 on)
@pytest.mark.parametrize("M,K,N", [(33000, 128, 288), (33000, 256, 288), (16500, 384, 576), (4096, 1152, 3456), (4104, 1152, 3456)])
@pytest.mark.parametrize("asym", [False, True])
def test_tall_tiles(M, K, N, asym):
    g = torch.Generator(device="cuda").manual_seed(M + K)
    w = trdq.prepare_weights(0.02 * torch.randn(K, N, generator=g, device="cuda"), None)
    Xq = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    sx, bd = torch.rand(M, generator=g, device="cuda"), torch.randn(N, generator=g, device="cuda")
    zc = torch.randint(-127, 129, (M,), generator=g, device="cuda", dtype=torch.int32)
    Y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    acc = torch.full((M, N), -7, dtype=torch.int32, device="cuda")
    for debug in (acc, None):
        Y.fill_(7.0)
        if asym:
            trdq.qgemm_asym(w, Xq, sx, zc, Y, bias=bd, acc_debug=debug)
        else:
            trdq.qgemm(w, Xq, sx, Y, bias=bd, acc_debug=debug)
    codes, scales = w.export()
    q = Xq.float() + (zc.float()[:, None] if asym else 0.0)          # sums below 2^24: exact in float32
    want = q @ torch.from_numpy(codes.astype(np.float32)).cuda()
    if K > 256:                                                       # (beyond: in float64)
        want = q.double() @ torch.from_numpy(codes.astype(np.float64)).cuda()
    assert torch.equal(acc, want.int())
    y = acc.double() * sx.double()[:, None] * torch.from_numpy(scales.reshape(1, N).astype(np.float64)).cuda() + bd.double()
    # bf16 rounds to 2^-9 of the value; the float32 epilogue adds at most 4 * 2^-24 of the product's and the bias' size
    off = (Y.double() - y).abs() - 2.0 ** -8 * y.abs()
    assert (off <= 2.0 ** -21 * (y.abs() + 2.0 * bd.double().abs())).all()
