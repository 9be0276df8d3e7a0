"""GPU parity: every entry point of the C ABI against the CPU oracle, element by element.

Bars: packed planes, nnz and int32 accumulators bit-exact; fp16 outputs within 1e-3
relative (the kernels are built to round exactly once, so in practice they are bit-equal
and the tests report that too).
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import (dev, gpu_gemm, gpu_linear, gpu_pack_weights, gpu_quantize_pack, host_u32,
                      max_rel_err, same_half)
from paper_2604_03957_amd import binding as B
import inputs
import synth

pytestmark = pytest.mark.gpu
RTOL = 1e-3
PATHS = [B.PATH_POPC, B.PATH_MFMA, B.PATH_FP4]


def _say(*a):
    print(*a, flush=True)


# ---- ternarise + pack ---------------------------------------------------------------------

def _activation_case(seed, M, K, lda=None):
    lda = K if lda is None else lda
    A = (synth.gaussian(seed, 1, M * lda).reshape(M, lda) * 1.3).astype(np.float16)
    s = synth.scales(seed, 2, M, 0.3, 2.5)
    # plant exact ties and special values
    for m in range(min(M, 6)):
        h = np.float16(0.5 * float(s[m]))
        vals = [h, -h, np.nextafter(h, np.float16(0)), np.nextafter(-h, np.float16(-np.inf)),
                np.float16(np.nan), np.float16(np.inf), np.float16(-np.inf), np.float16(-0.0)]
        for i, v in enumerate(vals):
            if i < K:
                A[m, (7 * m + 5 * i) % K] = v
    return A, s


@pytest.mark.parametrize("M,K,lda", [(5, 40, None), (64, 768, None), (33, 300, 304), (257, 1001, 1003),
                                     (3, 4096, None), (2, 11008, None), (1, 1, None), (130, 129, 136)])
def test_quantize_pack_fp16_matches_oracle(M, K, lda):
    _say("quantize fp16", M, K, lda)
    A, s = _activation_case(100 + M, M, K, lda)
    t = oracle.ternarize(np.ascontiguousarray(A[:, :K]), s)
    want = oracle.pack_act(t)
    got = gpu_quantize_pack(A, s, K=K)
    for w, g, name in zip(want, got, ("mask", "sign", "nnz")):
        assert np.array_equal(w, g), name


@pytest.mark.parametrize("M,K,lda", [(2100, 4096, None), (2300, 3720, 3728), (70000, 128, None)])
def test_quantize_pack_fp16_large_aligned_rows(M, K, lda):
    """Sizes at which aligned fp16 rows take the four-groups-per-thread kernel: whole rows, rows with
    padding groups past K, rows narrower than a wavefront's span; a few invalid scales among them."""
    _say("quantize fp16 large", M, K, lda)
    A, s = _activation_case(300 + K, M, K, lda)
    s[5], s[17], s[M - 1] = 0.0, np.nan, np.inf
    want = oracle.pack_act(oracle.ternarize(np.ascontiguousarray(A[:, :K]), s))
    got = gpu_quantize_pack(A, s, K=K)
    for w, g, name in zip(want, got, ("mask", "sign", "nnz")):
        assert np.array_equal(w, g), name
    sc = np.array([0.75], np.float16)                                  # one scale for the whole tensor
    want = oracle.pack_act(oracle.ternarize(np.ascontiguousarray(A[:, :K]), sc))
    got = gpu_quantize_pack(A, sc, K=K)
    assert all(np.array_equal(w, g) for w, g in zip(want, got))


@pytest.mark.parametrize("M,K,lda,shift", [(3, 7, 7, 1), (5, 8, 9, 1), (4, 129, 131, 3), (2300, 3717, 3719, 1),
                                           (40000, 200, 203, 5), (33000, 252, 252, 0)])
def test_quantize_pack_rows_on_any_address(M, K, lda, shift):
    """Rows that start on any element and end inside a group of 8, in the kernels of one and of four
    groups per thread: ternary and boolean planes of fp16, ternary planes of int8.  What lies past a
    row's end is large (fp16) or non-zero (int8) and must not show."""
    _say("quantize rows on any address", M, K, lda, shift)
    A, s = _activation_case(500 + K, M, K, lda)
    inputs.poison_gap(A, K)
    t = oracle.ternarize(np.ascontiguousarray(A[:, :K]), s)
    mask, sign, _ = oracle.pack_act(t)
    rw = B.plane_row_words(K)
    m, g = (torch.full((M, rw), -1, dtype=torch.int32, device="cuda:0") for _ in range(2))
    flat = torch.full((shift + A.size,), 65504.0, dtype=torch.float16, device="cuda:0")
    flat[shift:] = dev(A).reshape(-1)
    B.bwta_quantize_pack_act(flat[shift:], dev(s), m, g, None, M=M, K=K, lda=lda)
    torch.cuda.synchronize()
    assert np.array_equal(host_u32(m), mask) and np.array_equal(host_u32(g), sign)
    B.bwta_quantize_pack_bool(flat[shift:], dev(s), m, M=M, K=K, lda=lda)
    torch.cuda.synchronize()
    assert np.array_equal(host_u32(m), mask & ~sign)
    t8 = np.full((M, lda), 1, np.int8)
    t8[:, :K] = t
    flat8 = torch.full((shift + t8.size,), 1, dtype=torch.int8, device="cuda:0")
    flat8[shift:] = dev(t8).reshape(-1)
    B.bwta_quantize_pack_act(flat8[shift:], None, m, g, None, M=M, K=K, lda=lda, a_dtype=B.DTYPE_INT8)
    torch.cuda.synchronize()
    assert np.array_equal(host_u32(m), mask) and np.array_equal(host_u32(g), sign)


def test_quantize_pack_scale_modes_and_bad_scales():
    M, K = 9, 200
    A, _ = _activation_case(7, M, K)
    one = oracle.pack_act(oracle.ternarize(A, None))
    got = gpu_quantize_pack(A, None)
    assert all(np.array_equal(w, g) for w, g in zip(one, got))
    sc = np.array([0.75], np.float16)
    want = oracle.pack_act(oracle.ternarize(A, sc))
    got = gpu_quantize_pack(A, sc)
    assert all(np.array_equal(w, g) for w, g in zip(want, got))
    bad = np.array([1.0, 0.0, -1.0, np.inf, np.nan, 2.0 ** -24, 6e-5, 65504.0, 1.5], np.float16)
    want = oracle.pack_act(oracle.ternarize(A, bad))
    got = gpu_quantize_pack(A, bad)
    assert all(np.array_equal(w, g) for w, g in zip(want, got))
    assert not got[0][1:5].any()          # rows with an invalid scale are all zero


def test_quantize_pack_every_half_pattern():
    A = np.arange(65536, dtype=np.uint32).astype(np.uint16).view(np.float16).reshape(16, 4096)
    for sv in (1.0, 0.37, 2.0 ** -14, 2.0 ** -24, 900.0):
        s = np.full(16, sv, np.float16)
        want = oracle.pack_act(oracle.ternarize(A, s))
        got = gpu_quantize_pack(A, s)
        assert all(np.array_equal(w, g) for w, g in zip(want, got)), sv


def test_fragment_routes_every_half_pattern():
    """All 65 536 fp16 bit patterns, each under every one of 14 scales, through the two kernels that
    ternarise straight into matrix-core fragments (bwta_prepare_act on the tiled path, and the
    one-launch linear).  The scales include the smallest subnormal, odd and even subnormals, the
    values around 2^-14 and 2^-13 (where half the scale stops being a binary16 value) and the largest
    finite one.  The fragments are opaque, so the check is on what they produce against 64 random
    weight rows: one wrong decision changes every accumulator of its token by 1 or 2."""
    M, K, N = 256, 256, 64
    A = np.arange(65536, dtype=np.uint32).astype(np.uint16).view(np.float16).reshape(M, K)
    svals = np.array([0x3c00, 0x3800, 0x3e00, 0x0001, 0x0002, 0x0003, 0x03ff, 0x0400, 0x0401, 0x07ff, 0x0800,
                      0x0801, 0x7bff, 0x2e65], np.uint16).view(np.float16)
    w = synth.binary_pm1(35, 1, (N, K))
    ones = np.ones(N, np.float16)
    wsign = gpu_pack_weights(w)
    wsign2 = gpu_pack_weights(np.concatenate([w, w], axis=0))  # the one-launch kernel wants at least 128 channels
    prep = torch.empty(B.prepared_bytes(M, K), dtype=torch.uint8, device="cuda:0")
    ws = torch.empty(B.workspace_bytes(M, 128, K), dtype=torch.uint8, device="cuda:0")
    B.set_path(B.PATH_FP4)
    try:
        for rot in range(len(svals)):
            s = svals[(np.arange(M) + rot) % len(svals)]
            _, want_acc, want_out = oracle.linear(A, s, w, ones)
            acc = torch.full((M, N), 123456, dtype=torch.int32, device="cuda:0")
            B.set_tile(0)
            fmt = B.bwta_prepare_act(dev(A), dev(s), prep, M=M, K=K)
            B.bwta_gemm_prepared(prep, wsign, dev(s), dev(ones), acc, None, fmt=fmt, M=M, N=N, K=K)
            torch.cuda.synchronize()
            assert np.array_equal(acc.cpu().numpy(), want_acc), rot
            out = torch.full((M, 128), 7.0, dtype=torch.float16, device="cuda:0")
            B.set_tile(901)
            B.bwta_linear(dev(A), dev(s), wsign2, dev(np.ones(128, np.float16)), out, ws, M=M, N=128, K=K)
            torch.cuda.synchronize()
            got = out.cpu().numpy()
            assert same_half(np.ascontiguousarray(got[:, :N]), want_out), rot
            assert same_half(np.ascontiguousarray(got[:, N:]), want_out), rot
    finally:
        B.set_tile(0)
        B.set_path(B.PATH_AUTO)


@pytest.mark.parametrize("M,K,lda", [(64, 768, None), (7, 333, 335), (2, 11008, None)])
def test_quantize_pack_int8_matches_oracle(M, K, lda):
    lda = K if lda is None else lda
    t = synth.ternary(5, M, (M, lda), 0.4)
    want = oracle.pack_act(np.ascontiguousarray(t[:, :K]))
    got = gpu_quantize_pack(t, None, K=K)
    assert all(np.array_equal(w, g) for w, g in zip(want, got))


def test_quantize_pack_unaligned_base_pointer():
    M, K = 6, 264
    A, s = _activation_case(3, M, K + 8)
    flat = dev(A.reshape(-1))
    view = flat[1:]                                   # 2-byte aligned only
    ref = A.reshape(-1)[1:1 + (M - 1) * (K + 8) + K]
    rows = np.stack([ref[m * (K + 8): m * (K + 8) + K] for m in range(M)])
    want = oracle.pack_act(oracle.ternarize(rows, s))
    rw = B.plane_row_words(K)
    mask = torch.zeros((M, rw), dtype=torch.int32, device="cuda:0")
    sign = torch.zeros_like(mask)
    B.bwta_quantize_pack_act(view, dev(s), mask, sign, None, M=M, K=K, lda=K + 8)
    torch.cuda.synchronize()
    assert np.array_equal(host_u32(mask), want[0]) and np.array_equal(host_u32(sign), want[1])


@pytest.mark.parametrize("N,K", [(5, 40), (768, 768), (17, 1001), (3, 11008)])
def test_pack_weights_matches_oracle(N, K):
    w = synth.binary_pm1(11, N, (N, K))
    want = oracle.pack_weights(w)
    assert np.array_equal(host_u32(gpu_pack_weights(w)), want)
    Wf = (synth.gaussian(12, N, N * K).reshape(N, K)).astype(np.float16)
    Wf[0, :4] = np.array([0.0, -0.0, np.nan, -1e-7], np.float16)
    want = oracle.pack_weights(oracle.sign_weights(Wf))
    assert np.array_equal(host_u32(gpu_pack_weights(Wf)), want)


# ---- product + epilogue ---------------------------------------------------------------------

def _gemm_case(seed, M, N, K, p0=0.45):
    t = synth.ternary(seed, 1, (M, K), p0)
    w = synth.binary_pm1(seed, 2, (N, K))
    return t, w, synth.scales(seed, 3, M), synth.scales(seed, 4, N)


def _check_gemm(t, w, s_a, s_w, path, dirty_sign=False):
    M, K = t.shape
    N = w.shape[0]
    mask, sign, _ = oracle.pack_act(t)
    ws = oracle.pack_weights(w)
    want_acc = oracle.gemm_unpacked(t, w)
    want_out = oracle.epilogue(want_acc, s_a, s_w)
    if dirty_sign:
        sign = sign | (~mask & np.uint32(0x5A5A5A5A))
    acc, out = gpu_gemm(mask, sign, ws, s_a, s_w, M, N, K, path=path)
    assert np.array_equal(acc, want_acc), "int32 accumulators differ"
    err = max_rel_err(out, want_out)
    assert err <= RTOL, err
    return same_half(out, want_out)


GEMM_SHAPES = [(64, 768, 768), (1, 64, 128), (3, 5, 33), (16, 100, 4096), (130, 200, 1000),
               (300, 260, 2048), (257, 513, 1408), (70, 129, 11008), (4, 300, 11008)]


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm_matches_oracle(M, N, K, path):
    _say("gemm", M, N, K, "path", path)
    t, w, s_a, s_w = _gemm_case(1000 + M + N, M, N, K)
    exact = _check_gemm(t, w, s_a, s_w, path)
    assert exact, "fp16 outputs are within tolerance but not bit-equal"


DECODE_SHAPES = [(1, 7, 33), (2, 130, 128), (3, 257, 1000), (1, 1001, 4096), (4, 999, 4096), (8, 300, 4096),
                 (5, 258, 8192), (1, 515, 11008), (4, 130, 11008), (8, 67, 11008), (2, 70, 16384),
                 (3, 40, 16512), (9, 100, 4096), (13, 77, 1408), (16, 257, 11008), (16, 90, 768),
                 (16, 40, 17000), (7, 33, 30000), (12, 16, 512), (15, 17, 513), (17, 100, 4096), (33, 70, 11008),
                 (64, 130, 1000), (48, 17, 128), (65, 200, 4096), (100, 70, 11008), (128, 129, 1000)]


@pytest.mark.parametrize("M,N,K", DECODE_SHAPES)
def test_decode_shaped_gemm_matches_oracle(M, N, K):
    _say("decode gemm", M, N, K)
    t, w, s_a, s_w = _gemm_case(2000 + M + N, M, N, K, p0=0.5)
    assert _check_gemm(t, w, s_a, s_w, B.PATH_AUTO)
    assert _check_gemm(t, w, s_a, s_w, B.PATH_POPC, dirty_sign=True)
    assert _check_gemm(t, w, s_a, s_w, B.PATH_FP4, dirty_sign=True)


@pytest.mark.parametrize("rpw,tiles,pf", [(1, 2, 2), (1, 8, 2), (1, 8, 4), (1, 6, 3), (2, 2, 2), (2, 4, 2), (2, 8, 2),
                                          (2, 8, 4), (2, 16, 4), (2, 6, 3), (2, 4, 4), (3, 2, 2), (3, 4, 2), (3, 8, 2),
                                          (3, 6, 3), (3, 9, 3), (4, 2, 2), (4, 4, 2), (4, 8, 2),
                                          (1, 1, 1), (2, 1, 1), (2, 3, 1), (3, 1, 1), (4, 1, 1)])
def test_matrix_core_decode_every_work_split(rpw, tiles, pf):
    """Chunks per wavefront x channel tiles per workgroup x ring depth of the matrix-core decode
    kernel, on shapes with ragged N, a K tail inside a chunk, and more tiles than one workgroup takes."""
    _say("decode fp4 split", rpw, tiles, pf)
    B.set_tile(2000 + 1024 * pf + 64 * rpw + tiles)
    try:
        for M, N, K in [(16, 100, 4096), (11, 70, 11008), (1, 33, 200), (5, 1000, 1000), (40, 50, 600)]:
            if -(-B.plane_row_words(K) // 16) > 16 * rpw:
                continue
            t, w, s_a, s_w = _gemm_case(2500 + M + rpw, M, N, K, p0=0.5)
            assert _check_gemm(t, w, s_a, s_w, B.PATH_FP4)
    finally:
        B.set_tile(0)


def test_decode_seeded_random_shapes():
    """Twenty decode-sized problems with shapes drawn from a seeded generator (token counts across
    the token-group boundaries, ragged channel counts, K tails anywhere inside a 512-k chunk), on
    both decode kernel families and the dispatcher's choice."""
    rng = np.random.default_rng(20260403)
    for case in range(20):
        M = int(rng.choice([1, 2, 3, 5, 8, 15, 16, 17, 31, 33, 48, 63, 64, 65, 96, 127, 128]))
        N = int(rng.integers(1, 700))
        K = int(rng.integers(1, 9000))
        _say("decode random", case, M, N, K)
        t, w, s_a, s_w = _gemm_case(4000 + case, M, N, K, p0=float(rng.uniform(0.1, 0.9)))
        assert _check_gemm(t, w, s_a, s_w, B.PATH_AUTO, dirty_sign=True)
        assert _check_gemm(t, w, s_a, s_w, B.PATH_FP4)
        if M <= 16:
            assert _check_gemm(t, w, s_a, s_w, B.PATH_POPC)


@pytest.mark.parametrize("tile", [0, 22, 23, 21, 12, 11, 13, 222])
def test_tiled_matrix_core_kernel_every_tile_variant(tile):
    """The tiled FP4 kernel's workgroup tiles (128x128 at two and three wavefronts per SIMD, 128x64,
    64x128, 64x64, 128x96, split-K) and the dispatcher's own choice (0: 64x64 tiles for these few-tile
    shapes), fp16 output only (the int32 output always takes the 128x128 variant), ragged in M, N and K."""
    _say("fp4 tile variant", tile)
    B.set_tile(tile)
    try:
        for M, N, K in [(300, 260, 2048), (129, 70, 1100), (200, 513, 4096 + 64)]:
            t, w, s_a, s_w = _gemm_case(3000 + M, M, N, K)
            mask, sign, _ = oracle.pack_act(t)
            want = oracle.epilogue(oracle.gemm_unpacked(t, w), s_a, s_w)
            _, out = gpu_gemm(mask, sign, oracle.pack_weights(w), s_a, s_w, M, N, K, path=B.PATH_FP4, want_acc=False)
            assert same_half(out, want)
    finally:
        B.set_tile(0)


@pytest.mark.parametrize("path", PATHS)
def test_gemm_config1_tiny(path):
    c = synth.config1()
    assert _check_gemm(c["t"], c["w"], c["s_a"], c["s_w"], path)


@pytest.mark.parametrize("path", PATHS)
def test_gemm_degenerate_inputs(path):
    M, N, K = 40, 70, 600
    t, w, s_a, s_w = _gemm_case(77, M, N, K)
    _check_gemm(np.zeros_like(t), w, s_a, s_w, path)              # all-zero activation -> all-zero output
    _check_gemm(np.ones_like(t), np.ones_like(w), s_a, s_w, path)   # every product +1 -> K
    _check_gemm(-np.ones_like(t), np.ones_like(w), s_a, s_w, path)  # -> -K
    _check_gemm(t, w, s_a, s_w, path, dirty_sign=True)            # sign bits under a zero mask are ignored
    big = s_a.copy(); big[:] = np.float16(60000.0)                # overflow to +-Inf in the epilogue
    _check_gemm(t, w, big, s_w, path)
    tiny = s_w.copy(); tiny[:] = np.float16(2.0 ** -24)           # subnormal fp16 results
    assert _check_gemm(t, w, np.full(M, 2.0 ** -10, np.float16), tiny, path)
    neg = s_a.copy(); neg[::2] *= -1                              # negative scales, signed zeros
    sparse = t.copy(); sparse[:, 3:] = 0
    assert _check_gemm(sparse, w, neg, s_w, path)
    assert _check_gemm(t, w, neg, -s_w, path)


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("M,N,K", [(20, 36, 256), (200, 130, 600)])  # decode kernels / tiled kernels
def test_gemm_output_selection_and_scale_modes(path, M, N, K):
    t, w, s_a, s_w = _gemm_case(5, M, N, K)
    mask, sign, _ = oracle.pack_act(t)
    ws = oracle.pack_weights(w)
    want_acc = oracle.gemm_unpacked(t, w)
    acc, out = gpu_gemm(mask, sign, ws, None, None, M, N, K, path=path)
    assert np.array_equal(acc, want_acc) and same_half(out, oracle.epilogue(want_acc, None, None))
    acc, _ = gpu_gemm(mask, sign, ws, s_a, s_w, M, N, K, path=path, want_out=False)
    assert np.array_equal(acc, want_acc)
    _, out = gpu_gemm(mask, sign, ws, s_a[:1], s_w[:1], M, N, K, path=path, want_acc=False)
    assert same_half(out, oracle.epilogue(want_acc, s_a[:1], s_w[:1]))


def test_empty_problem_is_a_noop():
    ws = torch.empty(256, dtype=torch.uint8, device="cuda:0")
    z = torch.empty(0, dtype=torch.int32, device="cuda:0")
    B.bwta_gemm(z, z, z, None, None, z, None, ws, M=0, N=8, K=128)
    B.bwta_quantize_pack_act(z, None, z, z, None, M=0, K=128)
    torch.cuda.synchronize()


# ---- the whole layer ----------------------------------------------------------------------

@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("which", ["up", "down"])
def test_linear_ffn_reduced_m(which, path):
    c = inputs.config2(which, M=200)
    _say("linear", c["name"], "path", path)
    _, _, want = oracle.linear(c["A"], c["s_a"], c["w"], c["s_w"])
    wsign = gpu_pack_weights(c["w"])
    out = gpu_linear(c["A"], c["s_a"], wsign, c["s_w"], c["N"], path=path)
    assert max_rel_err(out, want) <= RTOL
    assert same_half(out, want)


@pytest.mark.parametrize("path", PATHS)
def test_linear_laplace_block_input(path):
    x = synth.laplace_activations(4, 1, 96, 4096)
    s = oracle.act_scale(x)
    w = synth.binary_pm1(4, 10, (160, 4096))
    s_w = synth.scales(4, 11, 160)
    _, _, want = oracle.linear(x, s, w, s_w)
    out = gpu_linear(x, s, gpu_pack_weights(w), s_w, 160, path=path)
    assert same_half(out, want)


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("M,N,K", [(1, 9, 40), (37, 130, 1001), (130, 70, 129), (257, 300, 2500), (33, 64, 11008)])
def test_linear_ragged_shapes_and_special_values(M, N, K, path):
    _say("linear ragged", M, N, K, "path", path)
    A, s = _activation_case(300 + M, M, K)          # ties, NaN, Inf, -0.0 planted
    if M > 4:
        s[3] = np.float16(0.0)                      # an invalid scale zeroes the token
    w = synth.binary_pm1(31, M + N, (N, K))
    s_w = synth.scales(31, 5, N)
    _, _, want = oracle.linear(A, s, w, s_w)
    out = gpu_linear(A, s, gpu_pack_weights(w), s_w, N, path=path)
    assert same_half(out, want)


@pytest.mark.parametrize("hook", [0, 901, 902, 903, 906, 912])
@pytest.mark.parametrize("M,N,K", [(256, 128, 128), (300, 260, 768), (1000, 3072, 768), (289, 1000, 1000), (700, 513, 1024), (257, 130, 136),
                                   (129, 130, 136), (200, 513, 768), (2, 130, 136), (16, 513, 768), (100, 3072, 1000)])
def test_linear_one_launch_short_k(M, N, K, hook):
    """bwta_linear as a single kernel (K <= 1024): every chunk count, channel splits forced to
    1, 2, 3, 6 and 12 as well as the launcher's own choice (which makes every group width appear; 0 = the
    dispatcher decides whether to use the kernel at all),
    ragged M and N, special values, an invalid token scale."""
    _say("one-launch linear", M, N, K, "hook", hook)
    A, s = _activation_case(500 + M, M, K)
    s[min(5, M - 1)] = np.float16(0.0)
    w = synth.binary_pm1(33, M + N, (N, K))
    s_w = synth.scales(33, 7, N)
    _, _, want = oracle.linear(A, s, w, s_w)
    B.set_tile(hook)
    try:
        out = gpu_linear(A, s, gpu_pack_weights(w), s_w, N, path=B.PATH_FP4)
    finally:
        B.set_tile(0)
    assert same_half(out, want)


@pytest.mark.parametrize("K", [200, 504, 760, 1000])
@pytest.mark.parametrize("N", [250, 440, 512, 1000])
def test_linear_one_launch_every_kernel_instance(N, K):
    """With two channel splits forced, N = 250 / 440 / 512 / 1000 leaves a workgroup 4 / 7 / 8 / 16
    channel blocks: workgroups of 4 or 8 wavefronts with groups of one or two blocks; K = 200 ..
    1000 gives one to four chunks of 256 k.  Together every instance of the kernel runs, on ragged
    M, N and K."""
    M = 300
    _say("one-launch linear, instance sweep", M, N, K)
    A, s = _activation_case(900 + N + K, M, K)
    w = synth.binary_pm1(36, N + K, (N, K))
    s_w = synth.scales(36, 8, N)
    _, _, want = oracle.linear(A, s, w, s_w)
    B.set_tile(902)
    try:
        assert B.linear_launches(M, N, K) == 1
        out = gpu_linear(A, s, gpu_pack_weights(w), s_w, N, path=B.PATH_FP4)
    finally:
        B.set_tile(0)
    assert same_half(out, want)


@pytest.mark.parametrize("M,N,K", [(1590, 2490, 1030), (330, 8200, 1024), (1190, 2500, 3071), (410, 5000, 1530), (300, 11007, 1100),
                                   (1270, 3299, 1300), (2040, 1536, 1530)])
def test_tiled_product_between_rounds_of_workgroups(M, N, K):
    """Products whose 128 x 128 tiles come to a little more than one per compute unit, or to few enough to leave
    many without one: tiles of 64 x 128, ragged on all sides, fp16 output; the last two just outside their windows."""
    _say("tiled product between rounds", M, N, K)
    assert B.planned_tile(M, N, K) == {1270: 223, 2040: 13}.get(M, 12)
    t = synth.ternary(90, M + N, (M, K), 0.5)
    w = synth.binary_pm1(91, M + K, (N, K))
    s_a, s_w = synth.scales(92, 1, M), synth.scales(92, 2, N)
    want = oracle.epilogue(oracle.gemm_unpacked(t, w), s_a, s_w)
    mask, sign, _ = oracle.pack_act(t)
    _, out = gpu_gemm(mask, sign, gpu_pack_weights(w), s_a, s_w, M, N, K, want_acc=False, want_out=True)
    assert same_half(out, want)


def _scratch(M, N, K):
    return torch.empty(max(B.workspace_bytes(M, N, K), 256), dtype=torch.uint8, device="cuda:0")


@pytest.mark.parametrize("K", [8, 300, 1024, 1025, 2048, 2999, 3900, 4096, 4097, 5000, 8192, 8193, 11008, 12288, 12289, 16384])
@pytest.mark.parametrize("N", [1, 9, 1031, 2050])
def test_linear_one_token_one_launch(N, K):
    """One token in one launch: both sides of every row split (lanes per row, chunks per lane), rows that
    end inside a word and inside a group of 8, one pass per wavefront and where 32 lanes share a row two, the three
    scale modes, an invalid scale, and results that overwrite the activations.  (More passes: the tall matrices.)"""
    rng = np.random.default_rng(N + K)
    _say("one-launch linear, one token", N, K)
    assert B.planned_kernel(B.OPERAND_FP16, 1, N, K) == B.KERNEL_LINEAR_ONE
    A, s = _activation_case(40 + N + K, 1, K)
    w = synth.binary_pm1(38, N + K, (N, K))
    s_w = synth.scales(38, 9, N)
    wsign = gpu_pack_weights(w)
    for s_a, sw in ((s, s_w), (np.float16([0.0]), s_w), (s, s_w[:1]), (None, None)):
        _, _, want = oracle.linear(A, s_a, w, sw)
        out = torch.full((1, N), float("nan"), dtype=torch.float16, device="cuda:0")
        off = int(rng.integers(0, 8))  # rows of any address
        buf = torch.full((K + 8,), 65504.0, dtype=torch.float16, device="cuda:0")  # and large values beside it
        a = buf[off:off + K]
        a.copy_(dev(A)[0])
        B.bwta_linear(a, None if s_a is None else dev(s_a), wsign, None if sw is None else dev(sw), out,
                      _scratch(1, N, K), M=1, N=N, K=K)
        torch.cuda.synchronize()
        assert same_half(out.cpu().numpy(), want)
        if N <= K:  # in place
            B.bwta_linear(a, None if s_a is None else dev(s_a), wsign, None if sw is None else dev(sw), a,
                          _scratch(1, N, K), M=1, N=N, K=K)
            torch.cuda.synchronize()
            assert same_half(a[:N].cpu().numpy()[None], want)


@pytest.mark.parametrize("K", [1024, 890, 2048, 1900, 4096, 3900, 8192, 8000, 12288, 12001, 16384, 16000])
@pytest.mark.parametrize("passes", [2, 4])
def test_linear_one_token_tall_matrices(passes, K):
    """One token against matrices whose rows take two and four passes per wavefront: every row split (lanes per row,
    chunks per lane), rows that are whole 128-byte lines and rows that are not, a last workgroup that is partly empty."""
    lanes = 8 if K <= 1024 else 16 if K <= 2048 else 32
    N = (65536 if passes == 2 else 6 * 65536) // lanes + 77
    _say("one-launch linear, one token, tall", passes, N, K)
    assert B.planned_kernel(B.OPERAND_FP16, 1, N, K) == B.KERNEL_LINEAR_ONE
    A, s = _activation_case(42 + N + K, 1, K)
    block = synth.binary_pm1(43, K, (64, K))
    w = np.ascontiguousarray(block[np.arange(N) % 64] * synth.binary_pm1(44, N, (N, 1))).astype(np.int8)
    s_w = synth.scales(43, 9, N)
    _, _, want = oracle.linear(A, s, w, s_w)
    assert same_half(gpu_linear(A, s, gpu_pack_weights(w), s_w, N), want)


@pytest.mark.parametrize("M,N,K", [(2, 1, 1025), (31, 129, 1536), (128, 250, 3072), (97, 8191, 1031), (129, 128, 1537),
                                   (300, 500, 2047), (250, 4096, 1025), (200, 70, 11003), (513, 1900, 1100),
                                   (777, 1500, 2560), (2050, 383, 1800), (2048, 1536, 1030), (2300, 1100, 2049),
                                   (33, 5000, 900), (128, 5200, 3072), (65, 10100, 2999), (70, 4000, 2500), (520, 1100, 16390),
                                   (2, 33001, 1537), (31, 17000, 1536), (4111, 100, 1537), (300, 1900, 2047), (250, 4096, 1290),
                                   (200, 70, 13003), (513, 1900, 1301), (33, 17000, 900), (531, 1850, 5629), (930, 300, 8651)])
@pytest.mark.parametrize("scales", ["vector", "scalar", "none"])
def test_linear_slabs_one_launch(M, N, K, scales):
    """The one-launch linear that walks K in slabs of 512: one, two and three channel blocks per wavefront, tokens
    and channels around the tile edges, two slabs and more, odd and even counts, K that ends on a slab, inside a
    word and inside a group of 8, rows of any address and pitch, ties, infinities and NaN, an invalid scale, scales
    below 2^-13 with an odd last bit and above 8192, and results that overwrite the activations.  The same of its
    neighbours: strips of 16 tokens where tokens or channels are few, the decode kernel where outputs are few for that K."""
    _say("one-launch linear, slabs", M, N, K, scales)
    strips16 = ((2, 1, 1025), (31, 129, 1536), (129, 128, 1537), (300, 500, 2047), (250, 4096, 1025), (200, 70, 11003), (513, 1900, 1100),
                (33, 5000, 900))
    kernel = B.KERNEL_LINEAR_ROWS if (M, N, K) in strips16 else B.KERNEL_GEMV_FP4 if (M, N, K) == (128, 250, 3072) else B.KERNEL_LINEAR_STRIP
    assert B.planned_kernel(B.OPERAND_FP16, M, N, K) == kernel
    lda = K + M % 3
    A, s = _activation_case(60 + M + K, M, K, lda)
    A, s = A[:, :K].copy(), s.copy()
    s[0], s[M // 2] = np.float16(0.0), np.float16(9000.0)
    A[M // 2, ::3], A[M // 2, 1::3] = np.float16(4500.0), np.float16(-4500.0)
    s[M - 1] = np.uint16(0x0405).view(np.float16)  # T = s / 2 lies between two binary16 values
    A[M - 1, ::2], A[M - 1, 1::2] = np.uint16(0x0203).view(np.float16), np.uint16(0x8202).view(np.float16)
    w = synth.binary_pm1(39, M + N + K, (N, K))
    s_w = synth.scales(39, 10, N)
    s_a, sw = {"vector": (s, s_w), "scalar": (s[1:2], s_w[:1]), "none": (None, None)}[scales]
    _, _, want = oracle.linear(A, s_a, w, sw)
    wsign = gpu_pack_weights(w)
    ldo = N + N % 2
    pitch = max(lda, ldo)
    buf = torch.zeros(M * pitch + 8, dtype=torch.float16, device="cuda:0")
    a = buf[M % 8:M % 8 + M * pitch].view(M, pitch)
    rows = np.zeros((M, pitch), np.float16)
    rows[:, :K] = A
    inputs.poison_gap(rows, K)
    a.copy_(dev(rows))
    out = torch.full((M, ldo), float("nan"), dtype=torch.float16, device="cuda:0")
    args = (None if s_a is None else dev(s_a), wsign, None if sw is None else dev(sw))
    modes = dict(a_scale_mode=B.SCALE_VECTOR, w_scale_mode=B.SCALE_VECTOR) if scales == "vector" else {}
    B.bwta_linear(a, *args, out, _scratch(M, N, K), M=M, N=N, K=K, lda=pitch, ldo=ldo, **modes)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert same_half(np.ascontiguousarray(got[:, :N]), want)
    assert np.all(np.isnan(got[:, N:]))
    B.bwta_linear(a, *args, a, _scratch(M, N, K), M=M, N=N, K=K, lda=pitch, ldo=pitch, **modes)
    torch.cuda.synchronize()
    assert same_half(np.ascontiguousarray(a[:, :N].cpu().numpy()), want)


@pytest.mark.parametrize("M,N,K,pitch,start", [
    (300, 515, 515, 515, 0), (300, 768, 768, 768, 0),     # in place, ragged and aligned rows, several channel splits
    (64, 500, 515, 515, 0), (2050, 1000, 1023, 1024, 0), (33, 130, 9, 131, 0),
    (200, 400, 768, 768, 300),                            # results start inside the activations' rows ..
    (200, 700, 700, 704, -704 * 3),                       # .. three rows above them
    (500, 300, 515, 900, 520), (500, 256, 512, 768, 512),  # side by side in rows of one pitch: no element shared
    (500, 300, 515, 815, -300),
    # the same with outputs enough for strips of 32 tokens
    (1100, 1000, 515, 1000, 0), (1100, 1024, 768, 1024, 0), (33, 17100, 9, 17101, 0), (2100, 400, 768, 768, 300),
    (1500, 700, 700, 704, -704 * 3), (3000, 300, 515, 900, 520), (4200, 256, 512, 768, 512), (3000, 300, 515, 815, -300)])
def test_linear_results_share_memory_with_the_activations(M, N, K, pitch, start):
    """Short K, where every workgroup of a strip of tokens reads the strip's whole rows: results written over the
    activations, over part of them, and between their rows.  The elements are the oracle's on the original
    activations, and what belongs to neither stays."""
    _say("linear, results in the activations' rows", M, N, K, pitch, start)
    few = (M + 15) // 16 * ((N + 127) // 128) <= 256  # without the overlap: strips of 16 tokens, or of 32
    assert B.planned_kernel(B.OPERAND_FP16, M, N, K) == (B.KERNEL_LINEAR_ROWS if few else B.KERNEL_LINEAR_FUSED)
    A, s = _activation_case(970 + M + K, M, K)
    w = synth.binary_pm1(40, M + N + K, (N, K))
    s_w = synth.scales(40, 11, N)
    _, _, want = oracle.linear(A, s, w, s_w)
    front = max(0, -start)
    front += front % 8
    flat = np.full(front + M * pitch + pitch + max(0, start), 7.0, np.float16)
    rows = np.arange(M)[:, None] * pitch
    at_a, at_o = front + rows + np.arange(K), front + start + rows + np.arange(N)
    flat[at_a] = A
    buf = dev(flat)
    B.bwta_linear(buf[front:], dev(s), gpu_pack_weights(w), dev(s_w), buf[front + start:], _scratch(M, N, K), M=M, N=N, K=K,
                  lda=pitch, ldo=pitch, a_scale_mode=B.SCALE_VECTOR, w_scale_mode=B.SCALE_VECTOR)
    torch.cuda.synchronize()
    flat[at_o] = want
    assert same_half(buf.cpu().numpy(), flat)


@pytest.mark.parametrize("M,N", [(2, 4300), (70, 3001), (297, 4990), (513, 4090), (513, 10990), (1000, 9000), (8230, 130)])
@pytest.mark.parametrize("K", [200, 300, 515, 900])
def test_linear_one_launch_strips_beyond_a_round_of_xcds(M, N, K):
    """Token strips that do not come in whole rounds of 8 and with many workgroups each: their workgroups are dealt to
    the XCDs one by one.  One strip alone, a few, some behind whole rounds, and strips that are not split; four and eight wavefronts, one and two
    channel blocks per group, one to four chunks of K; every (strip, split) must be done once."""
    _say("one-launch linear, partial round of strips", M, N, K)
    B.set_tile(901)  # K = 900 also beyond 4096 channels
    try:
        assert B.planned_kernel(B.OPERAND_FP16, M, N, K) == B.KERNEL_LINEAR_FUSED
        A, s = _activation_case(980 + M + K, M, K)
        w = synth.binary_pm1(41, M + N + K, (N, K))
        s_w = synth.scales(41, 12, N)
        _, _, want = oracle.linear(A, s, w, s_w)
        assert same_half(gpu_linear(A, s, gpu_pack_weights(w), s_w, N), want)
    finally:
        B.set_tile(0)


def test_linear_one_launch_seeded_random_shapes():
    """40 seeded random shapes (M 256..1500, N 128..2500, K 8..1024 in steps of 8) through the
    dispatcher's own choice of launch form, split count and kernel instance."""
    rng = np.random.default_rng(20260404)
    for case in range(40):
        M, N, K = int(rng.integers(256, 1501)), int(rng.integers(128, 2501)), 8 * int(rng.integers(1, 129))
        _say("one-launch linear, random shape", case, M, N, K)
        A, s = _activation_case(2000 + case, M, K)
        w = synth.binary_pm1(37, case, (N, K))
        s_w = synth.scales(37, 100 + case, N)
        _, _, want = oracle.linear(A, s, w, s_w)
        assert B.linear_launches(M, N, K) == 1
        out = gpu_linear(A, s, gpu_pack_weights(w), s_w, N)
        assert same_half(out, want), (case, M, N, K)


def test_linear_one_launch_of_32_token_strips_seeded_random_shapes():
    """20 seeded random shapes (M 1500..4000, N 1000..3000, K 8..1023) with outputs enough for the one-launch linear of
    32-token strips."""
    rng = np.random.default_rng(20260406)
    for case in range(20):
        M, N, K = int(rng.integers(1500, 4001)), int(rng.integers(1000, 3001)), int(rng.integers(8, 1024))
        _say("one-launch linear, 32-token strips, random shape", case, M, N, K)
        A, s = _activation_case(2100 + case, M, K)
        w = synth.binary_pm1(38, case, (N, K))
        s_w = synth.scales(38, 100 + case, N)
        _, _, want = oracle.linear(A, s, w, s_w)
        assert B.planned_kernel(B.OPERAND_FP16, M, N, K) == B.KERNEL_LINEAR_FUSED
        assert same_half(gpu_linear(A, s, gpu_pack_weights(w), s_w, N), want), (case, M, N, K)


def test_every_entry_and_family_seeded_random_shapes():
    """60 seeded random problems (prefill-sized with any K, short K, decode-sized) with planted
    ties, infinities, NaN, -0 and now and then an invalid token scale: bwta_linear as dispatched,
    and bwta_gemm on the dispatcher's choice and on each kernel family, int32 and fp16."""
    rng = np.random.default_rng(20260405)
    for case in range(60):
        kind = case % 3
        if kind == 0:
            M, N, K = int(rng.integers(129, 1200)), int(rng.integers(1, 1500)), int(rng.integers(1, 3000))
        elif kind == 1:
            M, N, K = int(rng.integers(256, 3000)), int(rng.integers(128, 3000)), 8 * int(rng.integers(1, 129))
        else:
            M, N, K = int(rng.integers(1, 129)), int(rng.integers(1, 2000)), int(rng.integers(1, 12000))
        _say("random problem", case, M, N, K)
        A = (synth.gaussian(9000 + case, 1, M * K) * float(rng.uniform(0.01, 30))).astype(np.float16).reshape(M, K)
        s = oracle.act_scale(A)
        if M * K > 8:
            flat = A.reshape(-1)
            idx = rng.integers(0, flat.size, 6)
            flat[idx[0]] = np.float16(0.5) * s[idx[0] // K]
            flat[idx[1]] = -(np.float16(0.5) * s[idx[1] // K])
            flat[idx[2]], flat[idx[3]], flat[idx[4]], flat[idx[5]] = np.inf, -np.inf, np.nan, -0.0
        if case % 4 == 0:
            s[int(rng.integers(0, M))] = np.float16([0.0, -1.0, np.inf, np.nan][(case // 4) % 4])
        w = synth.binary_pm1(9100 + case, 2, (N, K))
        s_w = synth.scales(9200 + case, 3, N)
        t, acc_want, want = oracle.linear(A, s, w, s_w)
        wsign = gpu_pack_weights(w)
        assert same_half(gpu_linear(A, s, wsign, s_w, N), want), (case, M, N, K)
        mask, sign, _ = oracle.pack_act(t)
        for path in [B.PATH_AUTO] + PATHS:
            acc, out = gpu_gemm(mask, sign, wsign, s, s_w, M, N, K, path=path)
            assert np.array_equal(acc, acc_want) and same_half(out, want), (case, M, N, K, path)


def test_linear_one_launch_scale_modes_and_strides():
    """The one-launch kernel with layerwise (scalar) scales, with no scales at all, and with strided
    input and output (nothing written past N)."""
    M, N, K, lda = 300, 260, 512, 520
    A, _ = _activation_case(601, M, lda)
    w = synth.binary_pm1(34, 1, (N, K))
    Ak = np.ascontiguousarray(A[:, :K])
    one_a, one_w = np.array([0.75], np.float16), np.array([1.25], np.float16)
    ws = torch.empty(B.workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda:0")
    wsign = gpu_pack_weights(w)
    B.set_tile(901)
    B.set_path(B.PATH_FP4)
    try:
        for (s_a, s_w), ldo in (((one_a, one_w), 272), ((None, None), 263)):  # 263: rows not 16-byte aligned
            fa = np.full(M, 1.0 if s_a is None else s_a[0], np.float16)
            fw = np.full(N, 1.0 if s_w is None else s_w[0], np.float16)
            _, _, want = oracle.linear(Ak, fa, w, fw)
            out = torch.full((M, ldo), 7.0, dtype=torch.float16, device="cuda:0")
            B.bwta_linear(dev(A), None if s_a is None else dev(s_a), wsign, None if s_w is None else dev(s_w), out, ws,
                          M=M, N=N, K=K, lda=lda, ldo=ldo)
            torch.cuda.synchronize()
            got = out.cpu().numpy()
            assert same_half(np.ascontiguousarray(got[:, :N]), want)
            assert np.all(got[:, N:] == 7.0)
    finally:
        B.set_path(B.PATH_AUTO)
        B.set_tile(0)


@pytest.mark.parametrize("M,N,K,tile", [(33, 129, 9, 0), (70, 131, 257, 0), (40, 200, 1023, 0), (300, 650, 768, 0),
                                        (5, 130, 1500, 0), (300, 131, 1029, 0), (300, 261, 1100, 243), (150, 131, 1100, 223)])
def test_linear_rows_on_any_address(M, N, K, tile):
    """bwta_linear with input and output rows that start on odd elements, lengths that end inside a group
    of 8 on both sides: the one-launch kernel, the decode kernel and the tiled kernels.  Large values lie
    between the input rows; what lies between the output rows stays."""
    _say("linear on any address", M, N, K, tile)
    lda, ldo = K + 3, N + 2
    A, s = _activation_case(900 + K, M, K, lda)
    inputs.poison_gap(A, K)
    w = synth.binary_pm1(901 + K, 2, (N, K))
    s_w = synth.scales(901 + K, 3, N)
    _, _, want = oracle.linear(np.ascontiguousarray(A[:, :K]), s, w, s_w)
    a = torch.zeros(1 + A.size, dtype=torch.float16, device="cuda:0")
    a[1:] = dev(A).reshape(-1)
    out = torch.full((1 + M * ldo,), 7.0, dtype=torch.float16, device="cuda:0")
    ws = torch.empty(B.workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda:0")
    B.set_tile(tile)
    try:
        B.bwta_linear(a[1:], dev(s), gpu_pack_weights(w), dev(s_w), out[1:], ws, M=M, N=N, K=K, lda=lda, ldo=ldo)
        torch.cuda.synchronize()
    finally:
        B.set_tile(0)
    got = out.cpu().numpy()
    rows = got[1:].reshape(M, ldo)
    assert same_half(np.ascontiguousarray(rows[:, :N]), want)
    assert got[0] == 7 and (rows[:, N:] == 7).all()


def test_linear_strided_input_and_output():
    M, N, K, lda, ldo = 50, 72, 520, 528, 80
    A, s = _activation_case(9, M, lda)
    w = synth.binary_pm1(32, 1, (N, K))
    s_w = synth.scales(32, 2, N)
    _, _, want = oracle.linear(np.ascontiguousarray(A[:, :K]), s, w, s_w)
    out = torch.full((M, ldo), 7.0, dtype=torch.float16, device="cuda:0")
    ws = torch.empty(B.workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda:0")
    for path in PATHS:
        B.set_path(path)
        out.fill_(7.0)
        B.bwta_linear(dev(A), dev(s), gpu_pack_weights(w), dev(s_w), out, ws, M=M, N=N, K=K, lda=lda, ldo=ldo)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert same_half(np.ascontiguousarray(got[:, :N]), want), path
        assert np.all(got[:, N:] == 7.0)            # nothing written past N
    B.set_path(B.PATH_AUTO)


@pytest.mark.parametrize("path", PATHS)
def test_prepare_once_feed_several_weight_matrices(path):
    M, K = 70, 1300
    A, s = _activation_case(55, M, K)
    prep = torch.empty(B.prepared_bytes(M, K), dtype=torch.uint8, device="cuda:0")
    B.set_path(path)
    try:
        fmt = B.bwta_prepare_act(dev(A), dev(s), prep, M=M, K=K)
        for i, N in enumerate((40, 129)):
            w = synth.binary_pm1(60 + i, 1, (N, K))
            s_w = synth.scales(60 + i, 2, N)
            t, acc_want, want = oracle.linear(A, s, w, s_w)
            out = torch.empty((M, N), dtype=torch.float16, device="cuda:0")
            acc = torch.empty((M, N), dtype=torch.int32, device="cuda:0")
            B.bwta_gemm_prepared(prep, gpu_pack_weights(w), dev(s), dev(s_w), acc, out, fmt=fmt, M=M, N=N, K=K)
            torch.cuda.synchronize()
            assert np.array_equal(acc.cpu().numpy(), acc_want)
            assert same_half(out.cpu().numpy(), want)
    finally:
        B.set_path(B.PATH_AUTO)


@pytest.mark.parametrize("path", [B.PATH_AUTO, B.PATH_POPC, B.PATH_FP4])
@pytest.mark.parametrize("M,N,K,count", [(1, 300, 4096, 3), (4, 130, 11008, 2), (8, 70, 1000, 35), (16, 64, 512, 2), (37, 50, 640, 3)])
def test_gemm_grouped_matches_oracle(M, N, K, count, path):
    _say("grouped", M, N, K, count, path)
    t, _, s_a, _ = _gemm_case(3000 + M, M, N, K, p0=0.5)
    mask, sign, _ = oracle.pack_act(t)
    dm, dsg, dsa = dev(mask), dev(sign), dev(s_a)
    keep, probs, want = [], [], []
    for i in range(count):
        w = synth.binary_pm1(3100 + i, M, (N, K))
        s_w = synth.scales(3200 + i, M, N)
        acc_want = oracle.gemm_unpacked(t, w)
        want.append((acc_want, oracle.epilogue(acc_want, s_a, s_w)))
        dw, dsw = gpu_pack_weights(w), dev(s_w)
        acc = torch.full((M, N), -9, dtype=torch.int32, device="cuda:0")
        out = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda:0")
        keep.append((dw, dsw, acc, out))
        probs.append((dm, dsg, dw, dsa, dsw, acc, out))
    ws = torch.empty(max(B.workspace_bytes(M, N, K), 256) * count, dtype=torch.uint8, device="cuda:0")
    B.set_path(path)
    try:
        B.bwta_gemm_grouped(B.make_problems(probs), ws, M=M, N=N, K=K)
        torch.cuda.synchronize()
    finally:
        B.set_path(B.PATH_AUTO)
    for (dw, dsw, acc, out), (acc_want, out_want) in zip(keep, want):
        assert np.array_equal(acc.cpu().numpy(), acc_want)
        assert same_half(out.cpu().numpy(), out_want)


@pytest.mark.parametrize("path", [B.PATH_AUTO, B.PATH_POPC, B.PATH_FP4])
@pytest.mark.parametrize("M", [1, 5, 12, 40])
def test_gemm_grouped_mixed_null_scales(M, path):
    """Problems of one grouped call may leave either scale out (NULL reads as 1) independently of
    their neighbours, the first problem included."""
    N, K = 150, 700
    _say("grouped mixed scales", M, N, K, path)
    t, _, s_a, _ = _gemm_case(3300 + M, M, N, K, p0=0.5)
    mask, sign, _ = oracle.pack_act(t)
    dm, dsg, dsa = dev(mask), dev(sign), dev(s_a)
    have = [(False, False), (True, True), (False, True), (True, False), (True, True)]  # (s_a, s_w) present?
    keep, probs, want = [], [], []
    for i, (ha, hw) in enumerate(have):
        w = synth.binary_pm1(3400 + i, M, (N, K))
        s_w = synth.scales(3500 + i, M, N)
        acc_want = oracle.gemm_unpacked(t, w)
        want.append(oracle.epilogue(acc_want, s_a if ha else None, s_w if hw else None))
        dw, dsw = gpu_pack_weights(w), dev(s_w)
        out = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda:0")
        keep.append((dw, dsw, out))
        probs.append((dm, dsg, dw, dsa if ha else None, dsw if hw else None, None, out))
    ws = torch.empty(max(B.workspace_bytes(M, N, K), 256) * len(have), dtype=torch.uint8, device="cuda:0")
    B.set_path(path)
    try:
        B.bwta_gemm_grouped(B.make_problems(probs), ws, M=M, N=N, K=K)
        torch.cuda.synchronize()
    finally:
        B.set_path(B.PATH_AUTO)
    for i, ((dw, dsw, out), out_want) in enumerate(zip(keep, want)):
        assert same_half(out.cpu().numpy(), out_want), (i, have[i])


@pytest.mark.parametrize("path", [B.PATH_AUTO] + PATHS)
@pytest.mark.parametrize("M,N,K", [(64, 96, 768), (3, 130, 1000), (130, 70, 129), (16, 257, 4096), (300, 200, 1000)])
def test_binary_activations_w1a1(M, N, K, path):
    """mask == NULL: binary (+-1) activations, the W1A1 "Binary Linear" special case
    acc = K - 2 popc(x ^ w); the activation signs are packed with the sign packer."""
    _say("w1a1", M, N, K, path)
    x = synth.binary_pm1(4000 + M, 1, (M, K))
    w = synth.binary_pm1(4000 + M, 2, (N, K))
    s_a, s_w = synth.scales(4000, 3, M), synth.scales(4000, 4, N)
    want_acc = oracle.gemm_unpacked(x, w)
    xs, wsn = oracle.pack_weights(x), oracle.pack_weights(w)
    xor_popc = np.array([[bin(int.from_bytes((xs[m] ^ wsn[n]).tobytes(), "little")).count("1") for n in range(N)] for m in range(min(M, 4))])
    assert np.array_equal(want_acc[:min(M, 4)], K - 2 * xor_popc)           # the textbook XNOR-popcount form
    acc, out = gpu_gemm(None, xs, wsn, s_a, s_w, M, N, K, path=path)
    assert np.array_equal(acc, want_acc)
    assert same_half(out, oracle.epilogue(want_acc, s_a, s_w))


@pytest.mark.parametrize("variant", [223, 243, 323])
@pytest.mark.parametrize("M,N,K", [(129, 256, 256), (300, 200, 1000), (257, 513, 2100), (1000, 700, 4096), (130, 90, 11008),
                                   (1000, 704, 4096), (256, 288, 256), (136, 64, 11008), (2048, 1024, 768),
                                   (4096, 4608, 384)])
def test_lds_staged_tiled_kernel_variants(M, N, K, variant):
    """The tiled FP4 kernel whose operands reach LDS by direct global->LDS loads, every tile / ring
    variant forced through the tuning hook: int32 accumulators and fp16 outputs, from planes
    (bwta_gemm) and from fp16 activations (bwta_linear's two-kernel form)."""
    _say("lds-staged", M, N, K, variant)
    t, w, s_a, s_w = _gemm_case(5000 + M + variant, M, N, K, p0=0.5)
    mask, sign, _ = oracle.pack_act(t)
    wsign = oracle.pack_weights(w)
    want_acc = oracle.gemm_unpacked(t, w)
    want_out = oracle.epilogue(want_acc, s_a, s_w)
    B.set_tile(variant)
    try:
        acc, out = gpu_gemm(mask, sign, wsign, s_a, s_w, M, N, K, path=B.PATH_FP4, want_acc=True, want_out=False)
        assert np.array_equal(acc, want_acc)
        _, out = gpu_gemm(mask, sign, wsign, s_a, s_w, M, N, K, path=B.PATH_FP4, want_acc=False, want_out=True)
        assert same_half(out, want_out)
        # from fp16 activations: +-1 / 0 under a unit scale ternarise to themselves
        B.set_tile(variant)
        A16 = t.astype(np.float16)
        dA = dev(A16)
        prep = torch.empty(B.prepared_bytes(M, K), dtype=torch.uint8, device="cuda:0")
        B.set_path(B.PATH_FP4)
        if B.prepared_format(M, K) == B.PREPARED_FP4:
            fmt = B.bwta_prepare_act(dA, None, prep, M=M, K=K)
            o2 = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda:0")
            B.bwta_gemm_prepared(prep, dev(wsign), dev(s_a), dev(s_w), None, o2, fmt=fmt, M=M, N=N, K=K)
            torch.cuda.synchronize()
            assert same_half(o2.cpu().numpy(), want_out)
    finally:
        B.set_path(B.PATH_AUTO)
        B.set_tile(0)


def test_lds_staged_seeded_random_shapes():
    """30 seeded random problems on the LDS-staged tiled kernel (every tile variant in turn, forced
    through the tuning hook): ragged token and channel counts, any K from two slabs up, planted
    ties / infinities / NaN, from fp16 through bwta_linear's two-kernel form and from planes,
    int32 and fp16."""
    rng = np.random.default_rng(20261128)
    variants = [243, 223, 323]
    for case in range(30):
        M, N, K = int(rng.integers(129, 900)), int(rng.integers(1, 1300)), int(rng.integers(129, 7000))  # tiled-kernel token counts
        variant = variants[case % 3]
        _say("random lds-staged problem", case, M, N, K, variant)
        A = (synth.gaussian(9500 + case, 1, M * K) * float(rng.uniform(0.01, 30))).astype(np.float16).reshape(M, K)
        s = oracle.act_scale(A)
        flat = A.reshape(-1)
        idx = rng.integers(0, flat.size, 6)
        flat[idx[0]] = np.float16(0.5) * s[idx[0] // K]
        flat[idx[1]] = -(np.float16(0.5) * s[idx[1] // K])
        flat[idx[2]], flat[idx[3]], flat[idx[4]], flat[idx[5]] = np.inf, -np.inf, np.nan, -0.0
        w = synth.binary_pm1(9600 + case, 2, (N, K))
        s_w = synth.scales(9700 + case, 3, N)
        t, acc_want, want = oracle.linear(A, s, w, s_w)
        wsign = gpu_pack_weights(w)
        mask, sign, _ = oracle.pack_act(t)
        B.set_tile(variant)
        try:
            acc, out = gpu_gemm(mask, sign, wsign, s, s_w, M, N, K, path=B.PATH_FP4)
            assert np.array_equal(acc, acc_want) and same_half(out, want), (case, M, N, K, variant)
            B.set_tile(variant)
            if K > 1024:  # longer than the one-launch linear takes: ternarise to fragments, then this kernel
                assert same_half(gpu_linear(A, s, wsign, s_w, N, path=B.PATH_FP4), want), (case, M, N, K, variant)
        finally:
            B.set_tile(0)


@pytest.mark.parametrize("variant", [422, 521, 611])
@pytest.mark.parametrize("M,N,K", [(129, 1, 100), (300, 200, 1000), (257, 513, 2100), (64 * 5 + 1, 700, 4096), (130, 90, 11008), (192, 256, 3500),
                                   (1000, 704, 600), (129, 129, 513)])
def test_tiled_product_of_16x16_blocks(M, N, K, variant):
    """The kernel of 16 x 16 blocks, every tile forced: one pair of slabs, pairs that do not divide by the groups that
    share K (some groups get none), ragged tokens and channels, whole and odd rows of results, the three scale
    modes; what lies between the rows stays."""
    _say("16 x 16 blocks", M, N, K, variant)
    t, w, s_a, s_w = _gemm_case(6000 + M + variant, M, N, K, p0=0.5)
    acc = oracle.gemm_unpacked(t, w)
    prep = torch.empty(B.prepared_bytes(M, K), dtype=torch.uint8, device="cuda:0")
    dw = dev(oracle.pack_weights(w))
    B.set_path(B.PATH_FP4)
    B.set_tile(variant)
    try:
        assert B.planned_wide(M, N, K) == variant
        assert B.prepared_format(M, K) == B.PREPARED_FP4
        fmt = B.bwta_prepare_act(dev(t.astype(np.float16)), None, prep, M=M, K=K)  # +-1 / 0 under scale 1: themselves
        for ldo, off, sa, sw in ((N, 0, s_a, s_w), (N + 3, 1, s_a[:1], s_w), ((N + 15) // 8 * 8, 0, None, None)):
            out = torch.full((off + M * ldo,), 7.0, dtype=torch.float16, device="cuda:0")
            B.bwta_gemm_prepared(prep, dw, None if sa is None else dev(sa), None if sw is None else dev(sw), None, out[off:],
                                 fmt=fmt, M=M, N=N, K=K, ldo=ldo)
            torch.cuda.synchronize()
            rows = out.cpu().numpy()[off:].reshape(M, ldo)
            ones_a, ones_w = np.ones(M, np.float16), np.ones(N, np.float16)
            want = oracle.epilogue(acc, ones_a if sa is None else np.resize(sa, M), ones_w if sw is None else sw)
            assert same_half(np.ascontiguousarray(rows[:, :N]), want), (ldo, off)
            assert (rows[:, N:] == 7).all() and (off == 0 or out[0].item() == 7)
    finally:
        B.set_path(B.PATH_AUTO)
        B.set_tile(0)


@pytest.mark.parametrize("M,N,K", [(2, 1, 8), (16, 128, 512), (17, 129, 513), (100, 5000, 1024), (40, 77, 1025), (100, 4000, 1536), (5, 70, 1537),
                                   (60, 2500, 2000), (130, 2200, 2048), (150, 130, 3000), (200, 1000, 2999), (300, 1500, 3072), (129, 65, 4000),
                                   (260, 900, 4096), (400, 1200, 3500), (140, 200, 6100), (330, 700, 5000), (390, 1250, 4500), (131, 500, 8192),
                                   (150, 300, 11003), (250, 4000, 700)])
def test_linear_strips_of_16_tokens(M, N, K):
    """The one-launch linear of 16-token strips: every number of chunks of 512 k and of groups that share them, one row
    of workgroups and two, ragged tokens and channels, K that ends inside a group of 8, a word and a chunk, rows of any
    address and pitch, ties, infinities and NaN, the three scale modes, results that overwrite the activations."""
    _say("one-launch linear, strips of 16 tokens", M, N, K)
    assert B.planned_rows(M, N, K) == 1
    lda, ldo = K + 3, N + 2
    A, s = _activation_case(1200 + K, M, K, lda)
    inputs.poison_gap(A, K)
    w = synth.binary_pm1(1201 + K, 2, (N, K))
    s_w = synth.scales(1201 + K, 3, N)
    rows = np.ascontiguousarray(A[:, :K])
    wsign = gpu_pack_weights(w)
    a = torch.zeros(1 + A.size, dtype=torch.float16, device="cuda:0")
    a[1:] = dev(A).reshape(-1)
    for sa, sw in ((s, s_w), (s[:1], s_w[:1]), (None, None)):
        full = np.ones(M, np.float16) if sa is None else np.resize(sa, M)
        _, _, want = oracle.linear(rows, full, w, np.ones(N, np.float16) if sw is None else np.resize(sw, N))
        out = torch.full((1 + M * ldo,), 7.0, dtype=torch.float16, device="cuda:0")
        B.bwta_linear(a[1:], None if sa is None else dev(sa), wsign, None if sw is None else dev(sw), out[1:], _scratch(M, N, K), M=M, N=N, K=K,
                      lda=lda, ldo=ldo)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert same_half(np.ascontiguousarray(got[1:].reshape(M, ldo)[:, :N]), want)
        assert got[0] == 7 and (got[1:].reshape(M, ldo)[:, N:] == 7).all()
    _, _, want = oracle.linear(rows, s, w, s_w)
    pitch = max(K, N)
    both = torch.zeros((M, pitch), dtype=torch.float16, device="cuda:0")
    both[:, :K] = dev(rows)
    B.bwta_linear(both, dev(s), wsign, dev(s_w), both, _scratch(M, N, K), M=M, N=N, K=K, lda=pitch, ldo=pitch)
    assert same_half(np.ascontiguousarray(both.cpu().numpy()[:, :N]), want)


@pytest.mark.parametrize("M,N,K,tile", [(129, 70, 1000, 11), (1500, 1990, 511, 11), (1500, 2055, 700, 12), (2050, 2690, 130, 12), (2050, 2900, 250, 23)])
def test_short_products_by_tile(M, N, K, tile):
    """Products of short K on prepared fragments, on both sides of where the tile changes, ragged on all sides."""
    _say("short product", M, N, K, tile)
    assert B.planned_tile(M, N, K) == tile and B.planned_wide(M, N, K) == 0
    t, w, s_a, s_w = _gemm_case(7000 + M, M, N, K, p0=0.5)
    want = oracle.epilogue(oracle.gemm_unpacked(t, w), s_a, s_w)
    prep = torch.empty(B.prepared_bytes(M, K), dtype=torch.uint8, device="cuda:0")
    fmt = B.bwta_prepare_act(dev(t.astype(np.float16)), None, prep, M=M, K=K)
    assert fmt == B.PREPARED_FP4
    out = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda:0")
    B.bwta_gemm_prepared(prep, gpu_pack_weights(w), dev(s_a), dev(s_w), None, out, fmt=fmt, M=M, N=N, K=K)
    torch.cuda.synchronize()
    assert same_half(out.cpu().numpy(), want)


@pytest.mark.parametrize("M,N,K,fresh,kept", [(300, 515, 3100, 611, 0), (140, 700, 4200, 611, 0), (513, 1990, 3329, 611, 611), (1030, 2050, 3300, 611, 0),
                                             (1397, 1530, 3631, 611, 521), (1397, 1536, 3631, 0, 0)])
def test_products_of_an_operand_that_is_kept(M, N, K, fresh, kept):
    """Around where a product on an operand prepared by its own call takes another tile than bwta_gemm on the same planes:
    both against the oracle."""
    _say("kept operand", M, N, K, fresh, kept)
    assert (B.planned_wide(M, N, K), B.planned_wide(M, N, K, prepared=True)) == (fresh, kept)
    t, w, s_a, s_w = _gemm_case(7050 + M, M, N, K, p0=0.5)
    want = oracle.epilogue(oracle.gemm_unpacked(t, w), s_a, s_w)
    prep = torch.empty(B.prepared_bytes(M, K), dtype=torch.uint8, device="cuda:0")
    wsign = gpu_pack_weights(w)
    fmt = B.bwta_prepare_act(dev(t.astype(np.float16)), None, prep, M=M, K=K)
    for _ in range(2):
        out = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda:0")
        B.bwta_gemm_prepared(prep, wsign, dev(s_a), dev(s_w), None, out, fmt=fmt, M=M, N=N, K=K)
        torch.cuda.synchronize()
        assert same_half(out.cpu().numpy(), want)
    mask, sign, _ = oracle.pack_act(t)
    _, out = gpu_gemm(mask, sign, wsign, s_a, s_w, M, N, K, want_acc=False, want_out=True)
    assert same_half(out, want)


@pytest.mark.parametrize("M,N,K,count", [
    (16, 2041, 4500, 24),   # one round of two blocks of 4 tiles, a ragged last tile
    (2, 4090, 5000, 32),    # four blocks of 4 tiles in place of 8 tiles
    (3, 4096, 4500, 64),    # eight blocks
    (40, 1000, 11000, 16),  # three groups of tokens, the last one of 8
    (128, 4090, 11008, 1),  # one matrix, eight groups of tokens
    (4, 2048, 20480, 8),    # ten wavefronts: two blocks of 2 tiles
    (4, 2040, 20480, 16),   # the same, four blocks
    (2, 828, 6044, 32),     # two chunks per wavefront, rows of whole 128-byte lines
    (2, 775, 9160, 32),     # three
    (2, 771, 12381, 32), (2, 794, 13247, 32),  # four, eight wavefronts, rows that are not and that are whole lines
    (17, 771, 14400, 24),   # the same, two groups of tokens, two blocks of 2 tiles
    (2, 507, 16699, 32),    # four, nine wavefronts, rows that are not whole lines
])
def test_decode_of_several_blocks_per_workgroup(M, N, K, count):
    """Launches whose workgroups go on from one block of channel tiles to the next, with and without int32 results."""
    _say("decode blocks", M, N, K, count)
    assert B.planned_decode_blocks(M, N, K, count) > 1
    sides = []
    for i in range(min(count, 2)):
        t, w, s_a, s_w = _gemm_case(7100 + 10 * i + M, M, N, K, p0=0.5)
        mask, sign, _ = oracle.pack_act(t)
        acc = oracle.gemm_unpacked(t, w)
        sides.append((dev(mask), dev(sign), gpu_pack_weights(w), dev(s_a), dev(s_w), acc, oracle.epilogue(acc, s_a, s_w)))
    probs, got = [], []
    for i in range(count):
        dm, dsg, dw, dsa, dsw, _, _ = sides[i % len(sides)]
        acc = torch.full((M, N), -9, dtype=torch.int32, device="cuda:0") if i % 3 == 0 else None
        out = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda:0")
        got.append((acc, out))
        probs.append((dm, dsg, dw, dsa, dsw, acc, out))
    ws = torch.empty(max(B.workspace_bytes(M, N, K), 256) * count, dtype=torch.uint8, device="cuda:0")
    B.bwta_gemm_grouped(B.make_problems(probs), ws, M=M, N=N, K=K)
    torch.cuda.synchronize()
    for i, (acc, out) in enumerate(got):
        assert acc is None or np.array_equal(acc.cpu().numpy(), sides[i % len(sides)][5])
        assert same_half(out.cpu().numpy(), sides[i % len(sides)][6])
