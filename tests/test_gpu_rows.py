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
