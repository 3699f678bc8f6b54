"""The rotate + quantise pass at the edges of its work split, in each of its forms (rows, block-tiled, other widths, zero
points), against the oracle."""
import numpy as np
import pytest
import torch

from paper_2503_06564_amd import trdq, workloads as wl
from gpu_util import CODE_FRAC, assert_scales_close, bf16_to_dev, dev, f32_to_dev, library_rule

pytestmark = pytest.mark.gpu

# one block (workgroups of eight tokens) and more (of four), token counts on both sides; three blocks per wave with a last
# wave of one and two; nine blocks per wave: beyond 36 blocks, and from 8192 tokens beyond 24
SHAPES = [(1, 128), (7, 128), (9, 128), (17, 512), (5, 640), (3, 1152), (16, 4608), (4, 4736), (6, 6144), (3, 8192), (8195, 3200)]


def _close(got, want):
    # a float32 value lies up to 3e-5 of a step off: half a code in 10^4 may sit close enough to a rounding tie, and a small
    # array may hold one or two of them
    diff = np.abs(got.astype(np.int16) - np.asarray(want, dtype=np.int16))
    assert diff.max() <= 1 and np.count_nonzero(diff) <= max(2, CODE_FRAC * diff.size)


@pytest.mark.parametrize("M,K", SHAPES)
def test_forms_match_oracle(oracle, M, K):
    Xb, _, d, _ = wl.small_case(61, M, K, 16, n_outliers=max(1, K // 144), outlier=40.0)
    X, dd = bf16_to_dev(Xb), f32_to_dev(d)
    buf = torch.full((M + 1, K), 99, dtype=torch.int8, device=dev())
    sx = torch.full((M + 1,), -1.0, device=dev())
    trdq.rotate_quant(X, dd, buf[:M], sx[:M])
    torch.cuda.synchronize()
    want, want_s = oracle.rotate_quant(Xb, d)
    rows = buf[:M].cpu().numpy()
    _close(rows, want)
    assert_scales_close(sx[:M].cpu().numpy(), want_s, "s_x")
    assert (buf[M] == 99).all() and sx[M].item() == -1.0
    if K > 4608:
        return
    Xt = torch.zeros(trdq.xq_tiled_nbytes(M, K), dtype=torch.int8, device=dev())
    back, st = torch.empty_like(buf[:M]), torch.empty(M, device=dev())
    trdq.rotate_quant_tiled(X, dd, Xt, st)
    trdq.xq_untile(Xt, M, K, back)
    torch.cuda.synchronize()
    assert np.array_equal(back.cpu().numpy(), rows) and torch.equal(st, sx[:M])
    trdq.rotate_quant_bits(X, dd, back, st, 6)
    torch.cuda.synchronize()
    want6, want_s6 = oracle.rotate_quant(Xb, d, 128, abits=6)
    _close(back.cpu().numpy(), want6)
    assert_scales_close(st.cpu().numpy(), want_s6, "s_x (6 bits)")
    if M > 100:
        return
    zc = torch.empty(M, dtype=torch.int32, device=dev())
    trdq.rotate_quant_asym(X, dd, back, st, zc)
    torch.cuda.synchronize()
    V = oracle.rotate(Xb, d, 128)
    lo, hi = np.minimum(V.min(axis=1), 0), np.maximum(V.max(axis=1), 0)
    s = (hi - lo) / 255
    z = -np.rint(lo / s)
    assert np.array_equal(128 - zc.cpu().numpy(), z)
    _close(back.cpu().numpy().astype(np.int16) + 128, np.clip(np.rint(V / s[:, None]) + z[:, None], 0, 255))
    assert_scales_close(st.cpu().numpy(), s, "s_x (zero points)")


# from each launch shape's smallest token count on: a wave per quad (4 and 6 blocks); block-tiled: five blocks per wave, seven,
# four (eight and four tokens per workgroup), three; the last workgroup incomplete, blocks that do not fill the last wave
@pytest.mark.parametrize("M,K", [(24577, 512), (24583, 768), (8193, 2432), (8198, 2560), (8193, 2688), (6145, 3200), (6150, 3584),
                                 (3077, 3584), (3073, 3712), (8197, 3712), (8192, 4096), (4097, 4224), (3075, 4608)])
def test_many_tokens_like_few(M, K):
    """A token's codes do not depend on how many there are: bit for bit those of calls on 512 tokens."""
    g = torch.Generator(device="cuda").manual_seed(K)
    X = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    d = torch.exp(0.3 * torch.randn(K, generator=g, device="cuda"))
    want = torch.empty((M, K), dtype=torch.int8, device="cuda")
    want_s = torch.empty(M, device="cuda")
    for m in range(0, M, 512):
        trdq.rotate_quant(X[m:m + 512], d, want[m:m + 512], want_s[m:m + 512])
    buf = torch.full((M + 1, K), 99, dtype=torch.int8, device="cuda")
    sx = torch.full((M + 1,), -1.0, device="cuda")
    trdq.rotate_quant(X, d, buf[:M], sx[:M])
    assert torch.equal(buf[:M], want) and torch.equal(sx[:M], want_s)
    assert (buf[M] == 99).all() and sx[M].item() == -1.0
    n = trdq.xq_tiled_nbytes(M, K)
    Xt = torch.full((n + 64,), 99, dtype=torch.int8, device="cuda")
    sx.fill_(-1.0)
    trdq.rotate_quant_tiled(X, d, Xt[:n], sx[:M])
    back = torch.empty_like(want)
    trdq.xq_untile(Xt[:n], M, K, back)
    assert torch.equal(back, want) and torch.equal(sx[:M], want_s)
    assert (Xt[n:] == 99).all() and sx[M].item() == -1.0
    zc, zc_all = torch.empty(512, dtype=torch.int32, device="cuda"), torch.empty(M, dtype=torch.int32, device="cuda")
    trdq.rotate_quant_asym(X, d, buf[:M], sx[:M], zc_all)
    m = M - 300
    trdq.rotate_quant_asym(X[m:], d, back[m:], want_s[m:], zc[:300])
    assert torch.equal(buf[m:M], back[m:]) and torch.equal(sx[m:M], want_s[m:]) and torch.equal(zc_all[m:], zc[:300])


@pytest.mark.parametrize("M,K,once", [(19419, 4608, "none"), (19420, 4608, "none"), (699051, 128, "none"), (24575, 4608, "none"),
                                      (24576, 4608, "symmetric"), (884735, 128, "none"), (884736, 128, "symmetric"),
                                      (32767, 4608, "symmetric"), (32768, 4608, "all")])
def test_inputs_about_the_size_of_the_memory_side_cache(M, K, once):
    """Calls on either side of the sizes from which the input is read non-temporally (108 * 2^20 values, with zero points 144 * 2^20) against
    calls on parts of it: the same codes, scales and zero points for every form, rows that are further apart than K included."""
    rule = "_ZN4trdq23rotate_quant_reads_onceElib"
    assert (library_rule(rule, M, K, False) & 1, library_rule(rule, M, K, True) & 1) == (once != "none", once == "all")
    g = torch.Generator(device="cuda").manual_seed(M)
    X = torch.randn(M, K + 8, generator=g, device="cuda", dtype=torch.bfloat16)[:, :K]
    diag = torch.rand(K, generator=g, device="cuda") + 0.5
    part = 16 * (M // 64)
    calls = [lambda x, q, s, z: trdq.rotate_quant(x, diag, q, s), lambda x, q, s, z: trdq.rotate_quant_asym(x, diag, q, s, z),
             lambda x, q, s, z: trdq.rotate_quant_bits(x, diag, q, s, 6)]
    for n, call in enumerate(calls):
        out = []
        for step in (M, part):
            q = torch.full((M, K), 99, dtype=torch.int8, device="cuda")
            s, z = torch.full((M,), -1.0, device="cuda"), torch.full((M,), -7, dtype=torch.int32, device="cuda")
            for m in range(0, M, step):
                call(X[m:m + step], q[m:m + step], s[m:m + step], z[m:m + step])
            out.append((q, s, z))
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(*out)) and (out[0][1] > 0).all(), n
        if n == 0:
            tiled, s = torch.empty(trdq.xq_tiled_nbytes(M, K), dtype=torch.int8, device="cuda"), torch.empty(M, device="cuda")
            trdq.rotate_quant_tiled(X, diag, tiled, s)
            q = torch.empty_like(out[0][0])
            trdq.xq_untile(tiled, M, K, q)
            torch.cuda.synchronize()
            assert torch.equal(q, out[0][0]) and torch.equal(s, out[0][1])
