"""The work that users of this library have it do, as cases a timing harness can run.

A case is a dict of plain values.  `prepare` makes what a user's program holds before the call
(seeded inputs, packed weights, buffers), `run` is one pass through the public entry points of
`paper_2604_03957_amd.binding`, `work` the bytes and operations one pass cannot do without, and
`tolerance` how far another correct implementation may differ.

Paths (`case["path"]`):
  linear     bwta_linear on fp16 activations: one layer, as an inference engine calls it
  gemm       bwta_gemm from bit planes, or bwta_quantize_pack_act from int8 ternary values first
  grouped    bwta_gemm_grouped: a decode step's independent matrices in one call
  block      the seven linears of a decoder block: bwta_prepare_act_autoscale per activation,
             bwta_gemm_prepared per weight matrix
  attention  the paper's two attention products with the scales and packers in front of them
  weights    bwta_prepare_weights: an fp16 checkpoint matrix to packed signs and scales
"""
import torch

from paper_2604_03957_amd import binding as B

DEV = "cuda"

MAX_WORK = 2.2e11  # operations of the largest product a drawn case may hold


def listed():
    return [
        # the smallest layer call: 64 tokens through one 768-wide projection
        {"name": "linear_tiny", "path": "linear", "M": 64, "N": 768, "K": 768, "scale": "vector"},
        # one generated token through the up/gate projection of a 7B decoder
        {"name": "linear_one_token", "path": "linear", "M": 1, "N": 11008, "K": 4096, "scale": "vector"},
        # the two layers of an encoder FFN on a batch of 32 sequences of 128 tokens
        {"name": "linear_encoder_up", "path": "linear", "M": 4096, "N": 3072, "K": 768, "scale": "vector"},
        {"name": "linear_encoder_down", "path": "linear", "M": 4096, "N": 768, "K": 3072, "scale": "vector"},
        # a 2048-token prompt through the up/gate projection of a 7B decoder
        {"name": "linear_prefill", "path": "linear", "M": 2048, "N": 11008, "K": 4096, "scale": "vector"},
        # sizes that are multiples of nothing: rows without 16-byte alignment on both sides, one layerwise scale
        {"name": "linear_ragged", "path": "linear", "M": 777, "N": 3001, "K": 2999, "scale": "scalar"},
        # the down projection of the same prompt from activations that are packed already
        {"name": "gemm_prefill_down", "path": "gemm", "M": 2048, "N": 4096, "K": 11008, "source": "planes"},
        # a decode step over 64 matrices (more than the caches hold): one token, and a batch of 16
        {"name": "decode_one_token", "path": "grouped", "M": 1, "N": 11008, "K": 4096, "count": 64},
        {"name": "decode_batch_16", "path": "grouped", "M": 16, "N": 4096, "K": 11008, "count": 64},
        # all seven linears of a 7B decoder block on a 2048-token prompt
        {"name": "block_prefill", "path": "block", "M": 2048, "hidden": 4096, "ffn": 11008},
        # the attention products of that block: 32 heads of 128 over 2048 tokens
        {"name": "attention", "path": "attention", "heads": 32, "seq": 2048, "dim": 128},
        # loading a checkpoint: the largest matrix of that block, from fp16
        {"name": "weights", "path": "weights", "N": 4096, "K": 11008},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _size(rng, lo, hi):
    """A size spread over the logarithm of its range: half of them whole (a multiple of 128), the
    others anything, odd ones among them."""
    n = _log_int(rng, lo, hi)
    return max(lo, n // 128 * 128) if rng.random() < 0.5 and n >= 128 else n


def draw(rng):
    path = rng.choice(["linear", "linear", "linear", "gemm", "grouped", "block", "attention", "weights"])
    while True:
        if path == "linear":
            c = {"path": path, "M": _size(rng, 1, 8192), "N": _size(rng, 128, 11008), "K": _size(rng, 128, 11008),
                 "scale": rng.choice(["vector", "vector", "scalar"])}
            ok = c["M"] * c["N"] * c["K"] * 2.0 <= MAX_WORK
        elif path == "gemm":
            c = {"path": path, "M": _size(rng, 1, 4096), "N": _size(rng, 128, 11008), "K": _size(rng, 128, 11008),
                 "source": rng.choice(["planes", "int8", "binary"])}
            ok = c["M"] * c["N"] * c["K"] * 2.0 <= MAX_WORK
        elif path == "grouped":
            c = {"path": path, "M": _log_int(rng, 1, 128), "N": _size(rng, 768, 11008), "K": _size(rng, 768, 11008),
                 "count": _log_int(rng, 2, 64)}
            ok = c["M"] * c["N"] * c["K"] * c["count"] * 2.0 <= MAX_WORK
        elif path == "block":
            hidden = rng.choice([768, 1024, 2048, 4096])
            c = {"path": path, "M": _log_int(rng, 1, 2048), "hidden": hidden,
                 "ffn": {768: 3072, 1024: 4096, 2048: 5504, 4096: 11008}[hidden]}
            ok = True
        elif path == "attention":
            c = {"path": path, "heads": rng.choice([4, 8, 12, 16, 32]), "seq": _log_int(rng, 64, 2048),
                 "dim": rng.choice([64, 128, 128])}
            ok = True
        else:
            c = {"path": path, "N": _size(rng, 768, 11008), "K": _size(rng, 768, 11008)}
            ok = c["N"] * c["K"] <= 4096 * 11008
        if ok:
            return c


# ---- inputs --------------------------------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _f16(*shape):
    return torch.empty(shape, dtype=torch.float16, device=DEV)


def _i32(*shape):
    return torch.empty(shape, dtype=torch.int32, device=DEV)


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)


def _words(g, rows, K):
    """Random packed rows: K bits each, padding bits zero."""
    rw = B.plane_row_words(K)
    w = torch.randint(-2 ** 31, 2 ** 31, (rows, rw), dtype=torch.int64, device=DEV, generator=g)
    left = torch.clamp(K - 32 * torch.arange(rw, device=DEV), 0, 32)
    return torch.where(left > 0, w & ((1 << left) - 1), torch.zeros_like(w)).to(torch.int32)


def _channel_scales(g, n):
    return (0.5 + torch.rand(n, device=DEV, generator=g)).half()


def _activations(g, M, K):
    """Transformer activations: N(0, 1), 2 % of the channels twenty times as large."""
    a = torch.randn((M, K), device=DEV, generator=g)
    heavy = torch.rand(K, device=DEV, generator=g) < 0.02
    return torch.where(heavy, 20.0 * a, a).half()


def _laplace(g, M, K):
    """Decoder hidden states: Laplace(0, 1)."""
    u = torch.rand((M, K), device=DEV, generator=g) - 0.5
    return (-torch.sign(u) * torch.log1p(-2.0 * u.abs().clamp(max=0.499999))).half()


def _token_scales(a, mode):
    """The value training starts the activation scale from, 2 mean |a|: per token, or one for the layer."""
    s = 2.0 * a.float().abs().mean(dim=1)
    return s.half() if mode == "vector" else s.mean().reshape(1).half()


def _planes(g, M, K):
    """Packed ternary activations, half of them zero: mask, and sign as a subset of it."""
    mask = _words(g, M, K)
    return mask, _words(g, M, K) & mask


BLOCK_LINEARS = [("q", "h", "hidden", "hidden"), ("k", "h", "hidden", "hidden"), ("v", "h", "hidden", "hidden"),
                 ("o", "att", "hidden", "hidden"), ("gate", "h2", "hidden", "ffn"), ("up", "h2", "hidden", "ffn"),
                 ("down", "act", "ffn", "hidden")]


def prepare(case, seed):
    g = _gen(seed)
    st = dict(case)
    path = case["path"]
    if path == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        st["A"] = _activations(g, M, K)
        st["s_a"] = _token_scales(st["A"], case["scale"])
        st["w"], st["s_w"] = _words(g, N, K), _channel_scales(g, N)
        st["out"], st["ws"] = _f16(M, N), _bytes(B.workspace_bytes(M, N, K))
    elif path == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        if case["source"] == "int8":
            st["t"] = torch.randint(0, 2, (M, K), device=DEV, generator=g, dtype=torch.int8)
            st["t"] *= torch.randint(0, 2, (M, K), device=DEV, generator=g, dtype=torch.int8) * 2 - 1
            st["mask"], st["sign"] = _i32(M, B.plane_row_words(K)), _i32(M, B.plane_row_words(K))
        elif case["source"] == "planes":
            st["mask"], st["sign"] = _planes(g, M, K)
        else:  # binary activations have no mask plane
            st["mask"], st["sign"] = None, _words(g, M, K)
        st["w"], st["s_w"], st["s_a"] = _words(g, N, K), _channel_scales(g, N), _channel_scales(g, M)
        st["out"], st["ws"] = _f16(M, N), _bytes(B.workspace_bytes(M, N, K))
    elif path == "grouped":
        M, N, K, count = case["M"], case["N"], case["K"], case["count"]
        mask, sign = _planes(g, M, K)
        s_a = _channel_scales(g, M)
        keep = [(mask, sign, _words(g, N, K), s_a, _channel_scales(g, N), None, _f16(M, N)) for _ in range(count)]
        st["keep"], st["problems"] = keep, B.make_problems(keep)
        st["out"] = [p[6] for p in keep]
        st["ws"] = _bytes(count * B.workspace_bytes(M, N, K))
    elif path == "block":
        M = case["M"]
        for nm in ("h", "att", "h2", "act"):
            st[nm] = _laplace(g, M, case["ffn" if nm == "act" else "hidden"])
            st["s_" + nm] = _f16(M)
        for nm, _, k, n in BLOCK_LINEARS:
            K, N = case[k], case[n]
            st["w_" + nm] = _words(g, N, K)
            st["sw_" + nm] = (_channel_scales(g, N).float() / K ** 0.5).half()
            st["out_" + nm] = _f16(M, N)
        for K in (case["hidden"], case["ffn"]):
            st["prep_%d" % K] = _bytes(B.prepared_bytes(M, K))
    elif path == "attention":
        heads, S, D = case["heads"], case["seq"], case["dim"]
        rows = heads * S
        st["q"], st["k"] = _laplace(g, rows, D), _laplace(g, rows, D)
        st["vt"] = _laplace(g, heads * D, S)  # V transposed per head: packed along the sequence
        logits = torch.randn((heads, S, S), device=DEV, generator=g)
        causal = torch.ones((S, S), dtype=torch.bool, device=DEV).triu_(1)
        st["p"] = torch.softmax(logits.masked_fill_(causal, float("-inf")), dim=-1).half().view(rows, S)
        for nm, n in (("q", rows), ("k", rows), ("p", rows), ("vt", heads * D)):
            st["s_" + nm] = _f16(n)
        rd, rs = B.plane_row_words(D), B.plane_row_words(S)
        for nm in ("q", "k"):
            st[nm + "_mask"], st[nm + "_sign"] = _i32(rows, rd), _i32(rows, rd)
        st["p_mask"] = _i32(rows, rs)
        if D % 128 == 0:
            st["prep"] = _bytes(B.prepared_bytes(heads * D, S))
        else:
            st["vt_mask"], st["vt_sign"] = _i32(heads * D, rs), _i32(heads * D, rs)
        st["scores"], st["ctx"] = _f16(heads, S, S), _f16(heads, S, D)
    else:
        N, K = case["N"], case["K"]
        st["W"] = (0.02 * torch.randn((N, K), device=DEV, generator=g)).half()
        st["w"], st["s_w"] = _i32(N, B.plane_row_words(K)), _f16(N)
    return st


# ---- one pass ------------------------------------------------------------------------------------


def run(st):
    path = st["path"]
    if path == "linear":
        B.bwta_linear(st["A"], st["s_a"], st["w"], st["s_w"], st["out"], st["ws"], M=st["M"], N=st["N"], K=st["K"])
        return st["out"]
    if path == "gemm":
        M, N, K = st["M"], st["N"], st["K"]
        if st["source"] == "int8":
            B.bwta_quantize_pack_act(st["t"], None, st["mask"], st["sign"], None, M=M, K=K, a_dtype=B.DTYPE_INT8)
        B.bwta_gemm(st["mask"], st["sign"], st["w"], st["s_a"], st["s_w"], None, st["out"], st["ws"], M=M, N=N, K=K)
        return (st["mask"], st["sign"], st["out"]) if st["source"] == "int8" else st["out"]
    if path == "grouped":
        B.bwta_gemm_grouped(st["problems"], st["ws"], M=st["M"], N=st["N"], K=st["K"])
        return st["out"]
    if path == "block":
        M, fmt, last = st["M"], None, None
        for nm, src, k, n in BLOCK_LINEARS:
            K, N = st[k], st[n]
            prep = st["prep_%d" % K]
            if src != last:  # one ternarisation feeds every matrix that reads this activation
                fmt = B.bwta_prepare_act_autoscale(st[src], st["s_" + src], prep, M=M, K=K)
                last = src
            B.bwta_gemm_prepared(prep, st["w_" + nm], st["s_" + src], st["sw_" + nm], None, st["out_" + nm], fmt=fmt,
                                 M=M, N=N, K=K)
        return [st["out_" + nm] for nm, _, _, _ in BLOCK_LINEARS] + [st["s_" + nm] for nm in ("h", "att", "h2", "act")]
    if path == "attention":
        heads, S, D = st["heads"], st["seq"], st["dim"]
        rows = heads * S
        for nm in ("q", "k"):
            B.bwta_act_scale(st[nm], st["s_" + nm], M=rows, K=D)
            B.bwta_quantize_pack_act(st[nm], st["s_" + nm], st[nm + "_mask"], st[nm + "_sign"], None, M=rows, K=D)
        B.bwta_matmul_tt(st["q_mask"], st["q_sign"], st["k_mask"], st["k_sign"], st["s_q"], st["s_k"], None, st["scores"],
                         batch=heads, M=S, N=S, K=D, alpha=1.0 / D ** 0.5)
        B.bwta_act_scale(st["p"], st["s_p"], M=rows, K=S)
        B.bwta_quantize_pack_bool(st["p"], st["s_p"], st["p_mask"], M=rows, K=S)
        if D % 128 == 0:
            fmt = B.bwta_prepare_act_autoscale(st["vt"], st["s_vt"], st["prep"], M=heads * D, K=S)
            B.bwta_matmul_bool_prepared(st["p_mask"], st["prep"], st["s_p"], st["s_vt"], st["ctx"], fmt=fmt, batch=heads,
                                        M=S, N=D, K=S)
        else:
            B.bwta_act_scale(st["vt"], st["s_vt"], M=heads * D, K=S)
            B.bwta_quantize_pack_act(st["vt"], st["s_vt"], st["vt_mask"], st["vt_sign"], None, M=heads * D, K=S)
            B.bwta_matmul_tt(st["p_mask"], None, st["vt_mask"], st["vt_sign"], st["s_p"], st["s_vt"], None, st["ctx"],
                             batch=heads, M=S, N=D, K=S)
        return (st["scores"], st["ctx"], st["s_q"], st["s_k"], st["s_p"], st["s_vt"], st["q_mask"], st["q_sign"],
                st["k_mask"], st["k_sign"], st["p_mask"])
    B.bwta_prepare_weights(st["W"], st["w"], st["s_w"], N=st["N"], K=st["K"])
    return st["w"], st["s_w"]


# ---- what one pass cannot do without ---------------------------------------------------------------


def _row_bytes(K):
    return 4 * B.plane_row_words(K)


def work(case):
    path = case["path"]
    if path == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 2 * M * K + N * _row_bytes(K) + 2 * (M + N) + 2 * M * N, "flops": 2.0 * M * N * K}
    if path == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        act = {"planes": 2, "binary": 1, "int8": 2}[case["source"]] * M * _row_bytes(K)
        if case["source"] == "int8":
            act += M * K
        return {"bytes": act + N * _row_bytes(K) + 2 * (M + N) + 2 * M * N, "flops": 2.0 * M * N * K}
    if path == "grouped":
        M, N, K, count = case["M"], case["N"], case["K"], case["count"]
        each = N * _row_bytes(K) + 2 * N + 2 * M * N
        return {"bytes": count * each + 2 * M * _row_bytes(K) + 2 * M, "flops": 2.0 * M * N * K * count}
    if path == "block":
        M, H, F = case["M"], case["hidden"], case["ffn"]
        total = {"bytes": 2 * M * (3 * H + F) + 4 * 2 * M, "flops": 0.0}
        for _, _, k, n in BLOCK_LINEARS:
            K, N = case[k], case[n]
            total["bytes"] += N * _row_bytes(K) + 2 * N + 2 * M * N
            total["flops"] += 2.0 * M * N * K
        return total
    if path == "attention":
        heads, S, D = case["heads"], case["seq"], case["dim"]
        rows = heads * S
        reads = 2 * (3 * rows * D + rows * S)
        writes = 2 * (rows * S + rows * D) + 2 * (3 * rows + heads * D) + 4 * rows * _row_bytes(D) + rows * _row_bytes(S)
        return {"bytes": reads + writes, "flops": 4.0 * heads * S * S * D}
    N, K = case["N"], case["K"]  # a sum, a difference, a magnitude and another sum per element
    return {"bytes": 2 * N * K + N * _row_bytes(K) + 2 * N, "flops": 4.0 * N * K}


def tolerance(case):
    """Planes and integer sums are whole numbers, and every fp16 result is the exact product rounded
    once (twice, at stated places, for the attention products): any two correct implementations agree
    bit for bit, and on the GPU the kernel families of this library do."""
    return "exact"
