"""GPU parity of weight preparation (mean-centring, sign, channel scale) and of the activation
scale's starting value against the oracle, through the C ABI.  Planes are bit-identical (every
decision is an exact integer comparison on both sides); the fp16 scales are compared to 1e-3
relative, the bar for floating point, and are in fact bit-identical on these inputs."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, gpu_gemm, host_u32, max_rel_err, same_half
from paper_2604_03957_amd import binding as B
import inputs
import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _say(*a):
    print(*a, flush=True)


def gpu_prepare(W, K=None):
    N = W.shape[0]
    K = W.shape[1] if K is None else K
    ws = torch.full((N, B.plane_row_words(K)), -1, dtype=torch.int32, device=DEV)
    sw = torch.full((N,), float("nan"), dtype=torch.float16, device=DEV)
    B.bwta_prepare_weights(dev(W), ws, sw, N=N, K=K, ldw=W.shape[1])
    torch.cuda.synchronize()
    return host_u32(ws), sw.cpu().numpy()


@pytest.mark.parametrize("N,K,ldw", [(5, 40, 40), (768, 768, 768), (17, 1001, 1003), (3, 11008, 11008), (2, 32768, 32768)])
def test_prepare_weights_matches_oracle(N, K, ldw):
    _say("prepare weights", N, K, ldw)
    W = (synth.gaussian(50 + N, 1, N * ldw) * 0.03 + 0.002).astype(np.float16).reshape(N, ldw)
    W[0, :min(K, 6)] = np.array([6e-8, -6e-8, 65504.0, -65504.0, 0.0, -0.0], np.float16)[:min(K, 6)]
    Wk = np.ascontiguousarray(W[:, :K])
    w, s = oracle.prepare_weights(Wk)
    planes, sw = gpu_prepare(W, K)
    assert np.array_equal(planes, oracle.pack_weights(w))
    assert max_rel_err(sw.reshape(1, -1), s.reshape(1, -1)) <= 1e-3
    assert same_half(sw, s)


@pytest.mark.parametrize("K", [1, 5, 8, 127, 512, 515, 1024, 1025, 2048, 2055, 4096, 4098, 8192, 8200, 12288, 12290, 16384,
                               16391])
def test_prepare_weights_at_the_edges_of_its_row_splits(K):
    """Row lengths around every change of threads per row and groups per thread, rows on odd addresses:
    plain rows, a row with NaN / +-Inf in it (its wavefronts go element by element), rows whose mean is
    positive (zeros beyond the row's end must not count as below it), subnormals, the largest values."""
    N, ldw = 7, K + 1
    _say("prepare weights edges", K)
    W = (synth.gaussian(500 + K, 1, N * ldw) * 0.03).astype(np.float16).reshape(N, ldw)
    W[1] += np.float16(0.05)
    W[2, ::3] = [np.inf, -np.inf, np.nan][K % 3]
    W[2, K - 1] = -np.inf
    W[6, K // 2] = np.nan
    W[3] = np.float16(6e-8) * synth.binary_pm1(500, K, (ldw,)).astype(np.float16)
    W[4] = np.float16(65504.0)
    W[5, ::2] = np.float16(-65504.0)
    W[:, K:] = np.nan
    w, s = oracle.prepare_weights(np.ascontiguousarray(W[:, :K]))
    planes, sw = gpu_prepare(W, K)
    assert np.array_equal(planes, oracle.pack_weights(w))
    assert same_half(sw, s)


@pytest.mark.parametrize("K", [8, 509, 4096, 4100, 11008, 12288])
def test_prepare_weights_around_the_limit_of_the_fp32_sums(K):
    """Rows whose groups of 8 have squares adding to just below and just above the 0.12 up to which their sums
    are taken in fp32, all of one sign (the largest partial sums) and with subnormals among them; one such
    group in a row of small ones; one large or non-finite value in a row of small ones."""
    _say("prepare weights, fp32 limit", K)
    N = 8
    W = (synth.gaussian(700 + K, 1, N * K) * 0.02).astype(np.float16).reshape(N, K)
    W[0], W[1], W[2] = np.float16(0.1224), np.float16(-0.1226), np.float16(0.16)
    W[0, ::7] = np.float16(6e-8)
    W[1, ::5] = np.float16(-3e-6)
    W[3, K - 8:] = np.float16(0.35)
    W[4, K // 2] = np.float16(40.0)
    W[5, K // 3] = np.nan
    W[6] = (synth.gaussian(701 + K, 1, K) * 1e-6).astype(np.float16)
    W[7] += np.float16(0.1)
    w, s = oracle.prepare_weights(W)
    planes, sw = gpu_prepare(W, K)
    assert np.array_equal(planes, oracle.pack_weights(w))
    assert same_half(sw, s)


def test_prepare_weights_special_rows():
    K = 300
    W = (synth.laplace(60, 1, 6 * K) * 0.02).astype(np.float16).reshape(6, K)
    W[0] = np.float16(0.125)                                   # all equal to the mean: every sign +1, scale 0
    W[1, :4] = [np.inf, -np.inf, np.nan, 1.0]                  # non-finite entries stay out of mean and scale
    W[2] = 0.0
    W[3, ::2] = np.float16(1.0); W[3, 1::2] = np.float16(-1.0) # mean exactly 0: ties nowhere, scale exactly 1
    W[4] = np.float16(2.0 ** -24)                              # smallest subnormal everywhere
    w, s = oracle.prepare_weights(W)
    planes, sw = gpu_prepare(W)
    assert np.array_equal(planes, oracle.pack_weights(w))
    assert same_half(sw, s)
    assert sw[0] == 0 and sw[3] == 1 and not planes[0].any()


@pytest.mark.parametrize("M,K,lda", [(5, 40, 40), (64, 768, 768), (33, 300, 304), (7, 11008, 11008), (3, 32768, 32768)])
def test_act_scale_matches_oracle(M, K, lda):
    _say("act scale", M, K, lda)
    A = np.ascontiguousarray(synth.gaussian_outlier_activations(70 + M, 1, M, lda))
    A[0, :min(K, 4)] = np.array([np.nan, np.inf, 65504.0, 6e-8], np.float16)[:min(K, 4)]
    want = oracle.act_scale(np.ascontiguousarray(A[:, :K]))
    s = torch.full((M,), float("nan"), dtype=torch.float16, device=DEV)
    B.bwta_act_scale(dev(A), s, M=M, K=K, lda=lda)
    torch.cuda.synchronize()
    got = s.cpu().numpy()
    assert max_rel_err(got.reshape(1, -1), want.reshape(1, -1)) <= 1e-3
    assert same_half(got, want)


# row lengths on both sides of every change of lanes per row, groups per lane and rows per wavefront,
# rows shorter than one load, and lengths that leave 1..7 elements in the last load
SCALE_K = [1, 3, 7, 8, 9, 63, 64, 65, 127, 128, 130, 256, 257, 511, 512, 515, 1024, 1029, 2048, 2054, 4096, 4103, 8192,
           8193, 12288, 12290, 16384, 16390]


@pytest.mark.parametrize("K", SCALE_K)
@pytest.mark.parametrize("M", [1, 67, 515])  # up to 512 rows and beyond: a workgroup or a wavefront per long row
def test_act_scale_at_the_edges_of_its_row_splits(M, K):
    """Exact at every split: odd leading dimensions (rows start on any 2-byte boundary), a row with
    NaN and Inf beside finite ones, subnormals, the largest values, an all-zero row.  What lies between
    the rows is large and must not show."""
    _say("act scale edges", M, K)
    lda = K + 3
    A = np.ascontiguousarray(synth.gaussian_outlier_activations(300 + K, 1, M, lda))
    inputs.poison_gap(A, K)
    A[0, K - 1] = np.float16(-65504.0)
    if M > 4:
        A[1, :K] = np.float16(6e-8)
        A[2, :K:2] = np.nan
        A[2, K - 1] = -np.inf
        A[5, K // 2] = np.nan
        A[3, :K] = 0
        A[4, :K] = np.float16(65504.0)
    want = oracle.act_scale(np.ascontiguousarray(A[:, :K]))
    s = torch.full((M,), float("nan"), dtype=torch.float16, device=DEV)
    B.bwta_act_scale(dev(A), s, M=M, K=K, lda=lda)
    torch.cuda.synchronize()
    assert same_half(s.cpu().numpy(), want)


def test_prepared_weights_feed_the_linear_layer():
    """fp16 checkpoint -> prepare -> BWTA linear equals the oracle's chain on the same inputs."""
    M, N, K = 70, 130, 1000
    W = (synth.gaussian(80, 1, N * K) * 0.02 + 0.001).astype(np.float16).reshape(N, K)
    t = synth.ternary(80, 2, (M, K), 0.5)
    s_a = synth.scales(80, 3, M)
    w, s_w = oracle.prepare_weights(W)
    want_acc = oracle.gemm_unpacked(t, w)
    want = oracle.epilogue(want_acc, s_a, s_w)
    ws = torch.empty((N, B.plane_row_words(K)), dtype=torch.int32, device=DEV)
    sw = torch.empty((N,), dtype=torch.float16, device=DEV)
    B.bwta_prepare_weights(dev(W), ws, sw, N=N, K=K)
    mask, sign, _ = oracle.pack_act(t)
    acc, out = gpu_gemm(mask, sign, ws, s_a, sw.cpu().numpy(), M, N, K)
    assert np.array_equal(acc, want_acc) and same_half(out, want)


@pytest.mark.parametrize("path", [B.PATH_AUTO, B.PATH_POPC, B.PATH_FP4])
@pytest.mark.parametrize("M,N,K,lda", [(5, 40, 40, 40), (64, 70, 768, 768), (33, 50, 300, 304), (130, 96, 1001, 1003),
                                       (257, 130, 4096, 4096), (300, 64, 11008, 11008), (200, 33, 520, 528)])
def test_scale_and_ternarise_in_one_pass(M, N, K, lda, path):
    """bwta_prepare_act_autoscale: the token scales it writes are the oracle's act_scale (to the
    floating-point bar, and bit for bit on these inputs), and the operand it prepares, fed to
    bwta_gemm_prepared with those scales, gives the oracle's linear layer exactly.  Both operand
    forms (bit planes below 129 tokens and on the popcount path, matrix-core fragments above),
    ragged and strided rows, NaN / Inf entries, an all-zero token (scale 0: the token is zero)."""
    _say("scale + ternarise", M, N, K, lda, "path", path)
    A = np.ascontiguousarray(synth.gaussian_outlier_activations(90 + M, 1, M, lda))
    A[0, :min(K, 4)] = np.array([np.nan, np.inf, 65504.0, 6e-8], np.float16)[:min(K, 4)]
    A[2, :] = 0
    Ak = np.ascontiguousarray(A[:, :K])
    s_want = oracle.act_scale(Ak)
    assert s_want[2] == 0
    w = synth.binary_pm1(91, M + N, (N, K))
    s_w = synth.scales(91, 3, N)
    _, _, want = oracle.linear(Ak, s_want, w, s_w)
    B.set_path(path)
    try:
        s = torch.full((M,), float("nan"), dtype=torch.float16, device=DEV)
        prep = torch.empty(B.prepared_bytes(M, K), dtype=torch.uint8, device=DEV)
        out = torch.full((M, N), 7.0, dtype=torch.float16, device=DEV)
        ws = torch.empty((N, B.plane_row_words(K)), dtype=torch.int32, device=DEV)
        B.bwta_pack_weights(dev(w), ws, N=N, K=K)
        fmt = B.bwta_prepare_act_autoscale(dev(A), s, prep, M=M, K=K, lda=lda)
        B.bwta_gemm_prepared(prep, ws, s, dev(s_w), None, out, fmt=fmt, M=M, N=N, K=K)
        torch.cuda.synchronize()
    finally:
        B.set_path(B.PATH_AUTO)
    got_s = s.cpu().numpy()
    assert max_rel_err(got_s.reshape(1, -1), s_want.reshape(1, -1)) <= 1e-3
    assert same_half(got_s, s_want)
    assert same_half(out.cpu().numpy(), want)


@pytest.mark.parametrize("K", [1, 7, 129, 512, 513, 1024, 1031, 2048, 2050, 4096, 4100, 6144, 6150, 8192, 8195, 11264, 11270,
                               12288, 12289, 16384, 16385])
@pytest.mark.parametrize("M", [133, 411, 643])
def test_one_pass_fragments_at_the_edges_of_their_row_splits(M, K):
    """Fragments of bwta_prepare_act_autoscale against bwta_act_scale + bwta_prepare_act (both held to the
    oracle above), bit for bit over the whole padded operand: row lengths around every change of
    wavefronts and groups per thread with one, two and four rows per workgroup, row counts that leave padding
    rows, rows on odd addresses with large values between them."""
    lda = K + 1
    _say("one-pass fragments", M, K)
    A = np.ascontiguousarray(synth.gaussian_outlier_activations(400 + K, 1, M, lda))
    inputs.poison_gap(A, K)
    A[1, K - 1] = np.inf
    A[2, :] = 0
    dA = dev(A)
    n = B.prepared_bytes(M, K)
    one, two = (torch.zeros(n, dtype=torch.uint8, device=DEV) for _ in range(2))
    s1, s2 = (torch.full((M,), float("nan"), dtype=torch.float16, device=DEV) for _ in range(2))
    f1 = B.bwta_prepare_act_autoscale(dA, s1, one, M=M, K=K, lda=lda)
    B.bwta_act_scale(dA, s2, M=M, K=K, lda=lda)
    f2 = B.bwta_prepare_act(dA, s2, two, M=M, K=K, lda=lda)
    torch.cuda.synchronize()
    assert f1 == f2 == B.PREPARED_FP4
    assert same_half(s1.cpu().numpy(), s2.cpu().numpy()) and torch.equal(one, two)


@pytest.mark.parametrize("N,K", [(2561, 40), (2562, 1000), (2563, 1500), (2567, 2047), (2050, 3000), (5, 2500), (1001, 3071), (901, 6001), (897, 4097)])
def test_prepare_weights_rows_side_by_side(N, K):
    """Weight rows that share a workgroup: row counts that do not divide by theirs, rows of odd pitch that end inside a
    group of 8, rows of small values, of large ones, of ties around the mean, and with NaN and infinities beside finite
    neighbours; signs and scales bit for bit."""
    _say("prepare weights, rows side by side", N, K)
    ldw = K + 1
    W = (synth.gaussian(70 + K, 1, N * ldw) * 0.03 + 0.002).astype(np.float16).reshape(N, ldw)
    W[1] *= np.float16(1000.0)
    W[2, :K] = np.float16(0.25)
    W[3, :4] = np.array([np.nan, np.inf, -np.inf, 65504.0], np.float16)
    W[N - 1, K - 1] = np.nan
    W[N - 2, :K] = 0
    inputs.poison_gap(W, K)
    w, s = oracle.prepare_weights(np.ascontiguousarray(W[:, :K]))
    planes, sw = gpu_prepare(W, K)
    assert np.array_equal(planes, oracle.pack_weights(w))
    assert np.array_equal(sw.view(np.uint16), s.view(np.uint16))
