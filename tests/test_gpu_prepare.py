"""Weight preparation at the edges of its kernels (widths that are no multiple of a workgroup's 64 columns, one and
many blocks) against the oracle, and groups of a layer that are set again in place."""
import numpy as np
import pytest

from paper_2503_06564_amd import workloads as wl
from tests.gpu_util import assert_codes_close, assert_scales_close, bf16_to_dev, f32_to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def trdq():
    from paper_2503_06564_amd import trdq as t
    t.lib()
    return t


@pytest.mark.parametrize("wbits", [8, 6, 4])
@pytest.mark.parametrize("K,N", [(128, 16), (128, 64), (256, 80), (384, 128), (640, 144), (1152, 272), (4608, 48)])
@pytest.mark.parametrize("with_diag", [True, False])
def test_codes_and_scales(trdq, oracle, wbits, K, N, with_diag):
    _, W, d, _ = wl.small_case(31, 1, K, N, with_diag=with_diag)
    W[:, N // 2] = 0.0                                   # a dead channel: scale 0, codes 0
    w = trdq.prepare_weights(f32_to_dev(W), f32_to_dev(d) if with_diag else None, wbits=wbits)
    codes, scales = w.export()
    ref_codes, ref_scales = oracle.prepare_weights(W, d, 128, wbits)
    assert_codes_close(codes, ref_codes, "weight codes")
    assert_scales_close(scales, ref_scales, "weight scales")
    assert not codes[:, N // 2].any() and not np.asarray(scales).reshape(-1, N)[:, N // 2].any()


@pytest.mark.parametrize("wbits", [8, 4])
def test_group_set_again(trdq, wbits):
    """A group that is replaced holds what a fresh layer would hold: same diagonal form (refilled in place),
    then the diagonal dropped, then brought back."""
    import torch
    M, K, N = 40, 384, 144
    table = trdq.Table(4, 2)
    layer = trdq.Layer(table, K, N, wbits)
    ws = dict(Xq_ws=torch.empty((M, K), dtype=torch.int8, device="cuda"), sx_ws=torch.empty(M, device="cuda"))
    for seed, with_diag in ((1, True), (2, True), (3, False), (4, False), (5, True)):
        xb, W, d, bias = wl.small_case(seed, M, K, N)
        X, Wd, dd, bd = bf16_to_dev(xb), f32_to_dev(W), f32_to_dev(d) if with_diag else None, f32_to_dev(bias)
        layer.set_group(1, dd, Wd)
        fresh = trdq.Layer(table, K, N, wbits)
        fresh.set_group(1, dd, Wd)
        if with_diag:
            dd.fill_(float("nan"))                       # the layer keeps its own copy
        out = []
        for l in (layer, fresh):
            Y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
            l.forward(3, X, Y, bias=bd, **ws)
            out.append(Y.clone())
        assert torch.isfinite(out[0].float()).all() and torch.equal(out[0], out[1])
        for a, b in zip(layer.weights(1).export(), fresh.weights(1).export()):
            assert np.array_equal(a, b)
