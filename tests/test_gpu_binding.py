"""The natively marshalled calls on the GPU: the ordinary form of each reaches the C entry point with the same arguments as
the Python form (identical results), on the current stream, and raises the same errors."""
import ctypes

import pytest
import torch

from paper_2604_03957_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _native_only(name):
    """The native function with a fallback that fails the test."""
    def no_fallback(*a, **k):
        raise AssertionError("%s fell back to its Python form" % name)
    return B._native.bind(name, ctypes.cast(getattr(B.raw(), name), ctypes.c_void_p).value, no_fallback)


def _calls():
    """(name, positional arguments with None in the outputs' places, keywords, {place: output maker})"""
    g = torch.Generator(device=DEV).manual_seed(7)
    M, N, K, H = 130, 128, 640, 3  # H heads
    rw = B.plane_row_words(K)
    f16 = lambda *s: lambda: torch.full(s, float("nan"), dtype=torch.float16, device=DEV)
    i32 = lambda *s: lambda: torch.full(s, -9, dtype=torch.int32, device=DEV)
    zeros = lambda n: lambda: torch.zeros(max(n, 256), dtype=torch.uint8, device=DEV)
    A = torch.randn((H * M, K), device=DEV, generator=g).half()
    s_a, s_w = torch.rand(H * M, device=DEV, generator=g).half() + 0.5, torch.rand(H * N, device=DEV, generator=g).half()
    one = s_w[:1]
    word = lambda rows: torch.randint(-2 ** 31, 2 ** 31, (rows, rw), device=DEV, generator=g).to(torch.int32)
    mask, w, wm = word(H * M), word(H * N), word(H * N)
    sign, wsg = mask & word(H * M), wm & word(H * N)
    ws = B.workspace_bytes(M, N, K)
    prep = torch.zeros(B.prepared_bytes(M, K), dtype=torch.uint8, device=DEV)
    fmt = B.bwta_prepare_act(A, s_a, prep, M=M, K=K, stream=torch.cuda.current_stream())
    vprep = torch.zeros(B.prepared_bytes(H * N, K), dtype=torch.uint8, device=DEV)
    vfmt = B.bwta_prepare_act(A[:H * N], s_w, vprep, M=H * N, K=K, stream=torch.cuda.current_stream())
    mnk = dict(M=M, N=N, K=K)
    return [
        ("bwta_linear", [A, s_a, w, s_w, None, None], mnk, {4: f16(M, N), 5: zeros(ws)}),
        ("bwta_linear", [A, one, w, None, None, None], dict(mnk, ldo=N + 8, lda=K, workspace_bytes=ws), {4: f16(M, N + 8), 5: zeros(ws)}),
        ("bwta_gemm", [mask, sign, w, s_a, one, None, None, None], mnk, {5: i32(M, N), 6: f16(M, N), 7: zeros(ws)}),
        ("bwta_gemm", [None, sign, w, None, s_w, None, None, None], dict(mnk, a_scale_mode=0), {6: f16(M, N), 7: zeros(ws)}),
        ("bwta_gemm_prepared", [prep, w, s_a, s_w, None, None], dict(mnk, fmt=fmt), {5: f16(M, N)}),
        ("bwta_prepare_act", [A, s_a, None], dict(M=M, K=K), {2: zeros(B.prepared_bytes(M, K))}),
        ("bwta_prepare_act_autoscale", [A, None, None], dict(M=M, K=K), {1: f16(M), 2: zeros(B.prepared_bytes(M, K))}),
        ("bwta_quantize_pack_act", [A, s_a, None, None], dict(M=M, K=K - 5, lda=K), {2: i32(M, rw), 3: i32(M, rw)}),
        ("bwta_quantize_pack_act", [A.to(torch.int8), None, None, None, None], dict(M=M, K=K, a_dtype=B.DTYPE_INT8), {2: i32(M, rw), 3: i32(M, rw), 4: i32(M)}),
        ("bwta_quantize_pack_bool", [A, one, None], dict(M=M, K=K), {2: i32(M, rw)}),
        ("bwta_act_scale", [A, None], dict(M=M, K=K), {1: f16(M)}),
        ("bwta_prepare_weights", [A, None, None], dict(N=M, K=K), {1: i32(M, rw), 2: f16(M)}),
        ("bwta_matmul_tt", [mask, sign, wm, wsg, s_a, s_w, None, None], dict(mnk, batch=H, alpha=0.25), {6: i32(H, M, N), 7: f16(H, M, N)}),
        ("bwta_matmul_bool_prepared", [mask, vprep, s_a, s_w, None], dict(mnk, batch=H, fmt=vfmt), {4: f16(H, M, N)}),
    ]


def test_native_calls_match_the_python_forms():
    other = torch.cuda.Stream()
    for name, args, kw, outs in _calls():
        print("native call", name, kw, flush=True)
        results = []
        for how in range(3):
            a = list(args)
            for i, make in outs.items():
                a[i] = make()
            torch.cuda.synchronize()
            if how == 0:
                r = getattr(B, name)(*a, **kw, stream=torch.cuda.current_stream())  # a given stream: the Python form
            elif how == 1:
                r = _native_only(name)(*a, **kw)
            else:
                with torch.cuda.stream(other):
                    r = _native_only(name)(*a, **kw)
                other.synchronize()
            torch.cuda.synchronize()
            results.append([r] + [a[i].view(torch.int16 if a[i].dtype == torch.float16 else a[i].dtype) for i in outs])
        for r in results[1:]:
            assert r[0] == results[0][0] and all(torch.equal(x, y) for x, y in zip(r[1:], results[0][1:])), name


def test_native_calls_raise_the_same_errors():
    A = torch.zeros((4, 128), dtype=torch.float16, device=DEV)
    s = torch.ones(4, dtype=torch.float16, device=DEV)
    w = torch.zeros((8, 4), dtype=torch.int32, device=DEV)
    out = torch.full((4, 8), 5.0, dtype=torch.float16, device=DEV)
    ws = torch.zeros(B.workspace_bytes(4, 8, 128), dtype=torch.uint8, device=DEV)
    f = _native_only("bwta_linear")
    for args, kw, code in (((A, s, w, s, None, ws), dict(M=4, N=4, K=128), B.ERR_NULL), ((A, s, w, s, out, ws), dict(M=4, N=4, K=128, lda=100), B.ERR_SHAPE),
                           ((A, s, w, s, out, None), dict(M=4, N=4, K=128), B.ERR_WORKSPACE), ((A, s, w[0, 1:], s, out, ws), dict(M=4, N=4, K=128), B.ERR_ALIGN)):
        with pytest.raises(B.BwtaError) as e:
            f(*args, **kw)
        assert e.value.code == code
    torch.cuda.synchronize()
    assert (out == 5).all()
