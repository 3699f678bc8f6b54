"""What the rotated low-bit linear is used for, as cases that can be timed and compared.

A case is one call, or one transformer block's four calls, through the package's public entry points
(`paper_2503_06564_amd.trdq`) on inputs that are resident on the GPU, as a denoiser holds them.  Inputs follow the
recipe of `paper_2503_06564_amd.workloads` (unit-normal activations with a few massive channels, N(0, 0.02)
weights, log-normal diagonals), drawn on the GPU from the seed.

    op          what a pass calls
    layer       Layer.forward with the library's own choice of path (w 8, 6 or 4 bits)
    bits        rotate_quant_bits + qgemm: W6A6
    rpr         rotate_quant_rpr + qgemm: rotation, zigzag permutation, rotation
    asym        rotate_quant_asym + qgemm_asym: per-token zero points
    dense       rotate_quant_dense + qgemm: arbitrary orthogonal blocks
    dense_rpr   rotate_quant_dense_rpr_ws + qgemm: both rotations with arbitrary orthogonal blocks
    setup       Layer.set_group and the first call of the group: the weight side
    share       cosine_similarity: attention outputs of the two guidance passes, block by block

`shape` is "linear" (k -> n) or "block": the qkv, proj, fc1 and fc2 linears of a transformer block of width k.
"""
import math

import torch

from paper_2503_06564_amd import trdq

# tokens x (k -> n) of the largest listed case: a drawn case does no more products than that
_MOST_PRODUCTS = 32768 * 12 * 1152 * 1152
_SETUP_TOKENS = 32


def listed():
    def case(name, op, tokens, k, n=0, wbits=8):
        return {"name": name, "op": op, "shape": "linear" if n else "block", "tokens": tokens, "k": k, "n": n, "wbits": wbits}

    return [
        # one call on a batch of conditioning vectors (8 images x 2 guidance passes): launches and latency
        case("condition_16", "layer", 16, 1152, 1152),
        # one linear of one 512-token image
        case("single_512", "layer", 512, 1152, 1152),
        # text tokens (16 prompts of 77) through a key/value projection of a width that is no DiT-XL width, 4-bit weights
        case("text_1232_w4", "layer", 1232, 1024, 2048, 4),
        # a token count that is no multiple of any tile (e.g. 4 crops of 250 patches), a block of width 768
        case("ragged_1000_block", "layer", 1000, 768),
        # the block of DiT-XL/2 at 256 x 256: batch 8, guidance, 256 patches
        case("dit_4096_block", "layer", 4096, 1152),
        # the same block at 512 x 512 with 4-bit weights
        case("dit_16384_block_w4", "layer", 16384, 1152, 0, 4),
        # a video denoiser's block: batch 4, guidance, 16 frames of 256 patches
        case("video_32768_block", "layer", 32768, 1152),
        # the full transform with Hadamard blocks
        case("rpr_4096_block", "rpr", 4096, 1152),
        # per-token zero points
        case("asym_4096_block", "asym", 4096, 1152),
        # the full transform with calibrated (dense) blocks
        case("dense_rpr_4096_block", "dense_rpr", 4096, 1152),
        # a time-step group's weights: transform, quantise, lay out, first call
        case("setup_block", "setup", _SETUP_TOKENS, 1152),
        # attention outputs of 28 transformer blocks for 16 images, conditional against unconditional
        case("share_28x4096", "share", 4096, 1152, 28),
    ]


def draw(rng):
    op = rng.choices(["layer", "bits", "rpr", "asym", "dense", "dense_rpr", "setup", "share"],
                     [12, 2, 3, 3, 2, 2, 1, 1])[0]
    tokens = int(round(2.0 ** rng.uniform(0.0, 15.0)))
    if rng.random() < 0.5 and tokens > 64:      # image grids: whole rows of patches
        tokens -= tokens % 64
    if op == "share":
        return {"op": op, "shape": "linear", "tokens": max(16, min(tokens, 4096)), "k": 128 * rng.randint(2, 9),
                "n": rng.randint(1, 28), "wbits": 8}
    wbits = {"layer": rng.choice([8, 8, 8, 6, 4, 4]), "bits": 6, "rpr": rng.choice([8, 8, 4]),
             "setup": rng.choice([8, 8, 6, 4])}.get(op, 8)
    shape = "block" if op != "setup" and rng.random() < 0.4 else "linear"
    if op == "setup":
        tokens = _SETUP_TOKENS
    if op in ("dense", "dense_rpr"):            # dense blocks: their products count too
        tokens = min(tokens, 8192)
    if shape == "block":
        k = 128 * rng.randint(2, 12 if op == "layer" else 9)     # fc2 reads 4 k channels: 4608 at most but for a layer
        return {"op": op, "shape": shape, "tokens": max(1, min(tokens, _MOST_PRODUCTS // (12 * k * k))), "k": k, "n": 0,
                "wbits": wbits}
    k = 128 * int(round(2.0 ** rng.uniform(0.0, math.log2(36))))
    n = 16 * int(round(2.0 ** rng.uniform(3.0, math.log2(288))))
    return {"op": op, "shape": shape, "tokens": max(1, min(tokens, _MOST_PRODUCTS // (k * n))), "k": k, "n": n, "wbits": wbits}


def _linears(case):
    k, n = case["k"], case["n"]
    return [(k, n)] if case["shape"] == "linear" else [(k, 3 * k), (k, k), (k, 4 * k), (4 * k, k)]


def _orthogonal(gen, blocks):
    q, r = torch.linalg.qr(torch.randn(blocks, 128, 128, generator=gen, dtype=torch.float64))
    return (q * torch.sign(torch.diagonal(r, dim1=-2, dim2=-1)).unsqueeze(-2)).float().contiguous().cuda()


def prepare(case, seed):
    op, M = case["op"], case["tokens"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    host = torch.Generator().manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda")

    if op == "share":
        a = normal(case["n"], M * case["k"])
        b = a + 0.3 * normal(case["n"], M * case["k"])     # the two passes are alike, block by block
        return {"op": op, "a": a.bfloat16(), "b": b.bfloat16(),
                "ws": torch.empty(3 * case["n"], dtype=torch.float64, device="cuda"),
                "out": torch.empty(case["n"], device="cuda")}

    linears = []
    most_k = max(k for k, _ in _linears(case))
    ws = {"Xq": torch.empty(M * most_k, dtype=torch.int8, device="cuda"), "sx": torch.empty(M, device="cuda"),
          "zc": torch.empty(M, dtype=torch.int32, device="cuda"), "dense": None}
    if op == "dense_rpr":
        need = max(trdq.rotate_quant_dense_rpr_ws_nbytes(M, k) for k, _ in _linears(case))
        ws["dense"] = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    step = int(torch.randint(20, (1,), generator=host))
    table = trdq.Table(20, 5)
    group = table.lookup(step)
    for K, N in _linears(case):
        x = normal(M, K)
        massive = torch.randperm(K, generator=host)[: max(1, 8 * K // 1152)].cuda()
        x[:, massive] *= 10.0 + 70.0 * float(torch.rand(1, generator=host))
        d = {"K": K, "N": N, "X": x.bfloat16(), "Y": torch.empty(M, N, dtype=torch.bfloat16, device="cuda"),
             "Xq": ws["Xq"][: M * K].view(M, K), "bias": 0.1 * normal(N), "diag": torch.exp(0.3 * normal(K))}
        W = 0.02 * normal(K, N)
        wbits = case["wbits"]
        if op in ("layer", "setup"):
            d["layer"] = trdq.Layer(table, K, N, wbits)
            if op == "setup":
                d["W"] = W
            else:
                d["layer"].set_group(group, d["diag"], W)
        elif op in ("bits", "asym"):
            d["w"] = trdq.prepare_weights(W, d["diag"], wbits=wbits)
        elif op == "rpr":
            mag = torch.empty(K, device="cuda")
            trdq.channel_absmax(d["X"], d["diag"], mag, rotate=True)
            d["perm"] = torch.from_numpy(trdq.zigzag_permutation(mag.cpu().numpy())).cuda()
            d["w"] = trdq.prepare_weights_rpr(W, d["diag"], d["perm"], wbits=wbits)
        elif op == "dense":
            d["rot"] = trdq.Rotation(_orthogonal(host, K // 128), d["diag"])
            d["w"] = trdq.prepare_weights_dense(W, d["rot"], wbits=wbits)
        else:
            d["rot"] = trdq.Rotation(_orthogonal(host, K // 128), d["diag"])
            d["rot2"] = trdq.Rotation(_orthogonal(host, K // 128))
            mag = torch.empty(K, device="cuda")
            trdq.channel_absmax_dense(d["X"], d["rot"], mag)
            d["perm"] = torch.from_numpy(trdq.zigzag_permutation(mag.cpu().numpy())).cuda()
            d["w"] = trdq.prepare_weights_dense_rpr(W, d["rot"], d["perm"], d["rot2"], wbits=wbits)
        linears.append(d)
    return {"op": op, "linears": linears, "ws": ws, "step": step, "group": group}


def run(state):
    op = state["op"]
    if op == "share":
        trdq.cosine_similarity(state["a"], state["b"], state["ws"], state["out"])
        return state["out"]
    ws = state["ws"]
    sx = ws["sx"]
    for d in state["linears"]:
        X, Y, Xq, bias = d["X"], d["Y"], d["Xq"], d["bias"]
        if op == "setup":
            d["layer"].set_group(state["group"], d["diag"], d["W"])
        if op in ("layer", "setup"):
            d["layer"].forward(state["step"], X, Y, bias=bias, fused=None, Xq_ws=Xq, sx_ws=sx)
            continue
        if op == "asym":
            trdq.rotate_quant_asym(X, d["diag"], Xq, sx, ws["zc"], warm=d["w"])
            trdq.qgemm_asym(d["w"], Xq, sx, ws["zc"], Y, bias=bias)
            continue
        if op == "bits":
            trdq.rotate_quant_bits(X, d["diag"], Xq, sx, 6, warm=d["w"])
        elif op == "rpr":
            trdq.rotate_quant_rpr(X, d["diag"], d["perm"], Xq, sx, warm=d["w"])
        elif op == "dense":
            trdq.rotate_quant_dense(X, d["rot"], Xq, sx)
        else:
            trdq.rotate_quant_dense_rpr_ws(X, d["rot"], d["perm"], d["rot2"], Xq, sx, ws["dense"])
        trdq.qgemm(d["w"], Xq, sx, Y, bias=bias)
    return [d["Y"] for d in state["linears"]]


def work(case):
    op, M = case["op"], case["tokens"]
    if op == "share":
        values = case["n"] * M * case["k"]
        return {"bytes": 4 * values, "flops": 6 * values}
    total = {"bytes": 0, "flops": 0}
    for K, N in _linears(case):
        code_bytes = K * N // 2 if case["wbits"] == 4 else K * N
        scales = K // 128 * N if case["wbits"] == 4 else N
        total["bytes"] += 2 * M * K + 2 * M * N + code_bytes + 4 * (scales + N + K)
        total["flops"] += 2 * M * K * N
        # the rotation: seven butterfly stages, or a 128 x 128 product, per block and rotation
        per_value = {"rpr": 14, "dense": 256, "dense_rpr": 512}.get(op, 7)
        total["flops"] += per_value * M * K
        if op in ("rpr", "dense_rpr"):
            total["bytes"] += 4 * K
        if op in ("dense", "dense_rpr"):
            total["bytes"] += 4 * 128 * K * (2 if op == "dense_rpr" else 1)
        if op == "setup":
            total["bytes"] += 4 * K * N
            total["flops"] += 7 * K * N
    return total


def tolerance(case):
    # share: float32 results of sums kept in float64.  The rest: bf16 outputs of integer products on codes that may
    # differ by one step where the rotation's float32 sums are ordered differently (about one code in 10^5).
    if case["op"] == "share":
        return {"rel": 2e-6}
    return {"rel": 1e-3, "max": 0.03}
