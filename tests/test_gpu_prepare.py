"""Weight preparation at the edges of its kernels (widths that are no multiple of a workgroup's 64 columns, one and
many blocks) against the oracle, and groups of a layer that are set again."""
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


# 16 / 17 blocks: one or three to a wave; 48 / 49: kept in registers, or a kernel for the maxima before; 2 ... 34 workgroups,
# whole groups of 32 or not
@pytest.mark.parametrize("wbits", [8, 6, 4])
@pytest.mark.parametrize("K,N", [(2048, 16), (2176, 272), (6144, 16), (6272, 32), (6272, 80)])
def test_codes_scales_and_sums_of_wide_rows(trdq, oracle, wbits, K, N):
    """... with a diagonal that has entries beyond the range in which the kernel divides by reciprocals."""
    import torch
    _, W, d, _ = wl.small_case(37, 1, K, N)
    for row, f in ((5, 1e-22), (K - 3, 1e21)):
        d[row] *= f
        W[row] *= np.float32(f)
    w = trdq.prepare_weights(f32_to_dev(W), f32_to_dev(d), wbits=wbits)
    codes, scales = w.export()
    ref_codes, ref_scales = oracle.prepare_weights(W, d, 128, wbits)
    assert_codes_close(codes, ref_codes, "weight codes")
    assert_scales_close(scales, ref_scales, "weight scales")
    if wbits == 4:
        return
    # the column sums, through the product that uses them: sum_k (code_x + zc) code_w
    rng = np.random.default_rng(K)
    Xq, zc = rng.integers(-128, 128, (20, K), dtype=np.int8), rng.integers(-127, 129, 20, dtype=np.int32)
    acc = torch.empty((20, N), dtype=torch.int32, device="cuda")
    trdq.qgemm_asym(w, torch.from_numpy(Xq).cuda(), torch.ones(20, device="cuda"), torch.from_numpy(zc).cuda(),
                    torch.empty((20, N), dtype=torch.bfloat16, device="cuda"), acc_debug=acc)
    torch.cuda.synchronize()
    assert np.array_equal(acc.cpu().numpy(), (Xq.astype(np.int64) + zc[:, None]) @ codes.astype(np.int64))


# large int4 sets: a kernel of their own for the codes, one for the sums; the codes of a part of the columns by the other kernel
@pytest.mark.parametrize("with_diag", [True, False])
def test_large_int4_sets(trdq, with_diag):
    import torch
    K, N, part = 2176, 15440, 1040                       # K * N just beyond 2^25, neither whole workgroups
    assert K * N > 1 << 25
    g = torch.Generator(device="cuda").manual_seed(3)
    W = 0.02 * torch.randn(K, N, generator=g, device="cuda")
    W[:, 7] = 0.0
    d = torch.rand(K, generator=g, device="cuda") + 0.5 if with_diag else None
    big, small = trdq.prepare_weights(W, d, wbits=4), trdq.prepare_weights(W[:, :part].contiguous(), d, wbits=4)
    codes, scales = big.export()
    want = small.export()
    assert np.array_equal(codes[:, :part], want[0]) and np.array_equal(scales[:, :part], want[1])
    last = trdq.prepare_weights(W[:, N - 48:].contiguous(), d, wbits=4).export()
    assert np.array_equal(codes[:, N - 48:], last[0]) and np.array_equal(scales[:, N - 48:], last[1])
    # packed blocks, widened blocks and column sums, through the products that read them
    Xq = torch.randint(-127, 128, (640, K), generator=g, device="cuda", dtype=torch.int8)
    sx, zc = torch.rand(640, generator=g, device="cuda"), torch.randint(-50, 50, (640,), generator=g, device="cuda", dtype=torch.int32)
    for M in (3, 128, 640):
        y, y_part = torch.empty((M, N), dtype=torch.bfloat16, device="cuda"), torch.empty((M, part), dtype=torch.bfloat16, device="cuda")
        for asym in (False, True):
            for w, out in ((big, y), (small, y_part)):
                if asym:
                    trdq.qgemm_asym(w, Xq[:M], sx[:M], zc[:M], out)
                else:
                    trdq.qgemm(w, Xq[:M], sx[:M], out)
            assert torch.equal(y[:, :part], y_part), (M, asym)


# values that are quantised without a rotation of the kernel's own: one block to a wave, three, and the kernel of large int4 sets
@pytest.mark.parametrize("K,N,wbits", [(2048, 48, 8), (4608, 16, 8), (4608, 80, 4), (2176, 15440, 4)])
def test_quantiser_alone(trdq, K, N, wbits):
    """Identity blocks pass the values on bit for bit: codes and scales are the float32 quantiser's, rounded in float64 on the GPU."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(K)
    W = torch.randn(K, N, generator=g, device="cuda")
    W[:, 3] = 0.0
    rot = trdq.Rotation(torch.eye(128, device="cuda").repeat(K // 128, 1, 1))
    codes, scales = trdq.prepare_weights_dense(W, rot, wbits=wbits).export()
    most = 7.0 if wbits == 4 else 127.0
    blocks = W.view(K // 128, 128, N) if wbits == 4 else W.view(1, K, N)
    a = blocks.abs().amax(dim=1, keepdim=True)
    inv = torch.where(a > 0, torch.full_like(a, most) / a, torch.zeros_like(a))     # (a number / a tensor is a reciprocal, then a product)
    want = (blocks.double() * inv.double()).round().clamp(-most, most).view(K, N)
    assert np.array_equal(codes, want.to(torch.int8).cpu().numpy())
    assert np.array_equal(scales.reshape(-1, N), a.view(-1, N).cpu().numpy() * (np.float32(1.0) / np.float32(most)))
    rot.close()


@pytest.mark.parametrize("K,N,copies", [(256, 131072, 2), (65536, 112, 2), (384, 32768, 4)])
def test_memory_of_int4_sets(trdq, K, N, copies):
    """Packed rows and packed blocks, and as many bytes again for widened codes where a product reads them."""
    import torch
    W = torch.zeros(K, N, device="cuda")
    trdq.prepare_weights(W, None, wbits=4).close()       # what the runtime takes for a first launch
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    w = trdq.prepare_weights(W, None, wbits=4)
    used = free - torch.cuda.mem_get_info()[0]
    want = copies * K * N // 2 + 4 * (K // 128 + 1) * N
    assert abs(used - want) <= 4 << 20, (used, want)     # whole pages of 2 MB
    Xq, sx = torch.ones((64, K), dtype=torch.int8, device="cuda"), torch.ones(64, device="cuda")
    Y = torch.empty((64, N), dtype=torch.bfloat16, device="cuda")
    trdq.rotate_quant_tiled(torch.ones((64, K), dtype=torch.bfloat16, device="cuda")[:, :min(K, 4608)].contiguous(), None,
                            torch.empty(64 * min(K, 4608), dtype=torch.int8, device="cuda"), sx, warm=w)
    trdq.qgemm(w, Xq, sx, Y)
    assert not Y.float().any()


@pytest.mark.parametrize("wbits", [8, 4])
def test_products_of_a_set_that_was_replaced(trdq, wbits):
    """Every copy of the codes follows a replacement that fills a set again: few tokens, 64-token tiles on either copy, block-tiled."""
    import torch
    K, N = 384, 1152
    g = torch.Generator(device="cuda").manual_seed(5)
    layer, fresh = trdq.Layer(trdq.Table(1, 1), K, N, wbits), trdq.Layer(trdq.Table(1, 1), K, N, wbits)
    for _ in range(4):
        W, d = 0.02 * torch.randn(K, N, generator=g, device="cuda"), torch.rand(K, generator=g, device="cuda") + 0.5
        layer.set_group(0, d, W)
    fresh.set_group(0, d, W)
    for M in (3, 100, 1000, 4600, 6016):
        X = torch.randn(M, K, generator=g, device="cuda").bfloat16()
        Xq, sx = torch.empty((M, K), dtype=torch.int8, device="cuda"), torch.empty(M, device="cuda")
        got, want = (torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        for fused in (True, False):
            layer.forward(0, X, got, fused=fused, Xq_ws=Xq, sx_ws=sx)
            fresh.forward(0, X, want, fused=fused, Xq_ws=Xq, sx_ws=sx)
            assert torch.equal(got, want), (M, fused)
    assert trdq.qgemm_tiled_preferred(layer.weights(0), 6016)


def test_preparation_of_very_long_rows_takes_little_longer(trdq):
    """18432 rows against 6144, 128 channels: 1.45 times (in one kernel 3 times, the wall clock of a replacement)."""
    import time

    import torch
    best = {}
    layers = {}
    for K in (6144, 18432):
        W = 0.02 * torch.randn(K, 128, device="cuda")
        layers[K] = trdq.Layer(trdq.Table(1, 1), K, 128, 8), torch.ones(K, device="cuda"), W
    for rep in range(40):
        for K, (layer, d, W) in layers.items():
            torch.cuda.synchronize()
            start = time.perf_counter()
            layer.set_group(0, d, W)
            best[K] = min(best.get(K, 1.0), time.perf_counter() - start)
    assert best[18432] < 2.2 * best[6144], best


# one block to a wave, three, and the two kernels of longer rows (int8); values[row 3 of a block, channel 5], the diagonal's entry there
@pytest.mark.parametrize("wbits", [8, 6, 4])
@pytest.mark.parametrize("K", [256, 2176, 6272])
@pytest.mark.parametrize("value,entry", [(None, None), (np.inf, 0.5), (-np.inf, 2.0), (np.nan, 2.0), (3e38, 0.25), (1e25, 1e-19),
                                         (1e-30, 1e14), (3e-39, 1.5), (-0.0, 3.0), (0.01, 1e-22)])
def test_division_by_the_diagonal_is_a_float32_division(trdq, wbits, K, value, entry):
    """Bit for bit what the quotients, rounded by the host, give without a diagonal: infinite, subnormal and overflowing ones too
    (an infinite channel keeps its infinite scale).  Block 1 holds the value alone and with values of its own size."""
    N = 32
    _, W, d, _ = wl.small_case(41, 1, K, N)
    if value is not None:
        W[3, 5] = W[128 + 3, 5] = value
        d[3] = d[128 + 3] = entry
        if np.isfinite(value):
            W[128:256, 7] *= np.float32(value)
    with np.errstate(all="ignore"):
        quotients = W / d[:, None]
    assert quotients.dtype == np.float32
    got = trdq.prepare_weights(f32_to_dev(W), f32_to_dev(d), wbits=wbits).export()
    want = trdq.prepare_weights(f32_to_dev(quotients), None, wbits=wbits).export()
    assert np.array_equal(got[0], want[0])
    assert np.array_equal(got[1].view(np.uint32), want[1].view(np.uint32))
    if np.isinf(quotients[3, 5]):
        assert np.isinf(got[1].reshape(-1, N)[0, 5])


@pytest.mark.parametrize("wbits", [8, 4])
def test_group_set_again(trdq, wbits):
    """A group that is replaced holds what a fresh layer would hold: same diagonal form, then the diagonal dropped, then
    brought back."""
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


def test_replaced_set_is_left_alone(trdq):
    """Replacing a group writes another set than the one that calls may still be reading, the first time and when it
    fills a set that was replaced before."""
    K, N = 384, 144
    layer = trdq.Layer(trdq.Table(4, 2), K, N, 8)
    held = []
    for seed in range(5):
        _, W, d, _ = wl.small_case(seed, 4, K, N)
        layer.set_group(1, f32_to_dev(d), f32_to_dev(W))
        w = layer.weights(1)
        if held:
            before, codes, scales = held[-1]
            assert w.handle.value != before.handle.value
            got = before.export()            # the set just replaced, not yet filled again
            assert np.array_equal(got[0], codes) and np.array_equal(got[1], scales)
        held.append((w, *w.export()))
    assert held[0][0].handle.value == held[2][0].handle.value == held[4][0].handle.value     # two sets take turns


@pytest.mark.parametrize("recorded", [False, True])
def test_calls_before_a_replacement_keep_their_set(trdq, recorded):
    """Forward calls that wait on another stream, launched or replayed from a graph, give the outputs of the set they were
    given, however many replacements follow at once."""
    import torch
    M, K, N = 1024, 384, 2304
    layer = trdq.Layer(trdq.Table(4, 2), K, N, 8)
    xb, W, d, _ = wl.small_case(3, M, K, N)
    X, dd = bf16_to_dev(xb), f32_to_dev(d)
    weights = [f32_to_dev((1.0 + i) * W) for i in range(4)]
    ws = dict(Xq_ws=torch.empty((M, K), dtype=torch.int8, device="cuda"), sx_ws=torch.empty(M, device="cuda"))
    want = []
    for Wd in weights:
        layer.set_group(1, dd, Wd)
        Y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        layer.forward(3, X, Y, **ws)
        torch.cuda.synchronize()
        want.append(Y)
    assert not torch.equal(want[2], want[3])
    side, busy = torch.cuda.Stream(), torch.empty(1 << 28, device="cuda")
    layer.set_group(1, dd, weights[0])
    got = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    graph = torch.cuda.CUDAGraph()
    if recorded:
        with torch.cuda.graph(graph, stream=side):
            layer.forward(3, X, got, **ws, stream=side.cuda_stream)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(4):
            busy.add_(1.0)                               # about a millisecond in front of the call
        if recorded:
            graph.replay()
        else:
            layer.forward(3, X, got, **ws, stream=side.cuda_stream)
    for Wd in weights[1:]:
        layer.set_group(1, dd, Wd)
    torch.cuda.synchronize()
    assert torch.equal(got, want[0])
    layer.forward(3, X, got, **ws)
    torch.cuda.synchronize()
    assert torch.equal(got, want[3])


@pytest.mark.parametrize("capturing", [False, True])
def test_first_replacement_waits_for_its_own_stream_only(trdq, capturing):
    """Long work on another stream does not hold it up, and a capture there (relaxed: allocations stay allowed) does not refuse
    it; the replacements that follow leave the set that the other stream's call reads alone until it has ended."""
    import ctypes as C

    import torch
    hip = trdq.lib()
    M, K, N = 1024, 384, 2304
    xb, W, d, _ = wl.small_case(5, M, K, N)
    X, dd = bf16_to_dev(xb), f32_to_dev(d)
    weights = [f32_to_dev((1.0 + i) * W) for i in range(3)]
    ws = [dict(Xq_ws=torch.empty((M, K), dtype=torch.int8, device="cuda"), sx_ws=torch.empty(M, device="cuda")) for _ in range(2)]
    want, got, after = (torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for _ in range(3))
    layer = trdq.Layer(trdq.Table(4, 2), K, N, 8)
    layer.set_group(1, dd, weights[0])
    layer.forward(3, X, want, **ws[0])
    side, busy, done = torch.cuda.Stream(), torch.empty(1 << 28, device="cuda"), torch.cuda.Event()

    def occupy():
        with torch.cuda.stream(side):
            for _ in range(100):
                busy.add_(1.0)                           # some 35 ms
            done.record()

    # a stream that does not share a hardware queue with `side`
    for own in (torch.cuda.Stream() for _ in range(8)):
        torch.cuda.synchronize()
        occupy()
        with torch.cuda.stream(own):
            torch.zeros(1, device="cuda")
        own.synchronize()
        if not done.query():
            break
    else:
        pytest.skip("every stream shares a hardware queue with the busy one")
    torch.cuda.synchronize()
    if capturing:
        stream, graph = C.c_void_p(), C.c_void_p()
        assert hip.hipStreamCreate(C.byref(stream)) == 0
        assert hip.hipStreamBeginCapture(stream, 2) == 0
        layer.set_group(1, dd, weights[1], stream=own.cuda_stream)
        assert hip.hipStreamEndCapture(stream, C.byref(graph)) == 0
        assert hip.hipGraphDestroy(graph) == 0 and hip.hipStreamDestroy(stream) == 0
    else:
        occupy()
        layer.forward(3, X, got, **ws[1], stream=side.cuda_stream)
        with torch.cuda.stream(side):
            done.record()
        layer.set_group(1, dd, weights[1], stream=own.cuda_stream)
        assert not done.query()
        layer.set_group(1, dd, weights[2], stream=own.cuda_stream)      # fills the set that the call on `side` reads
        assert done.query()
        assert torch.equal(got, want)
    layer.forward(3, X, after, **ws[0])
    fresh = trdq.Layer(trdq.Table(4, 2), K, N, 8)
    fresh.set_group(1, dd, weights[1] if capturing else weights[2])
    fresh.forward(3, X, want, **ws[0])
    torch.cuda.synchronize()
    assert torch.equal(after, want)


@pytest.mark.parametrize("replaced_before", [0, 1, 2])
def test_failed_replacement_keeps_the_group(trdq, replaced_before):
    """The preparation of a group ends with a wait for its stream, which a capturing stream refuses."""
    import ctypes as C

    import torch
    hip = trdq.lib()                     # finds the runtime that the library itself is linked to
    M, K, N = 8, 384, 144
    layer = trdq.Layer(trdq.Table(4, 2), K, N, 8)
    xb, W, d, _ = wl.small_case(1, M, K, N)
    X, dd, Wd = bf16_to_dev(xb), f32_to_dev(d), f32_to_dev(W)
    other = f32_to_dev(2.0 * W)
    for _ in range(replaced_before):
        layer.set_group(1, dd, other)
    layer.set_group(1, dd, Wd)
    ws = dict(Xq_ws=torch.empty((M, K), dtype=torch.int8, device="cuda"), sx_ws=torch.empty(M, device="cuda"))
    want, got = (torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    layer.forward(3, X, want, **ws)
    torch.cuda.synchronize()
    stream, graph = C.c_void_p(), C.c_void_p()
    assert hip.hipStreamCreate(C.byref(stream)) == 0
    assert hip.hipStreamBeginCapture(stream, 2) == 0                    # relaxed: allocations stay allowed
    with pytest.raises(trdq.TrdqError) as e:
        layer.set_group(1, dd, other, stream=stream.value)
    assert e.value.status == trdq.ERR_HIP
    hip.hipStreamEndCapture(stream, C.byref(graph))                     # an invalidated capture: no graph comes out
    hip.hipGetLastError()
    assert hip.hipStreamDestroy(stream) == 0
    layer.forward(3, X, got, **ws)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    layer.set_group(1, dd, other)                                       # and it can be replaced afterwards
    layer.forward(3, X, got, **ws)
    torch.cuda.synchronize()
    assert not torch.equal(got, want) and torch.isfinite(got.float()).all()
