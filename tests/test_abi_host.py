"""Host-side checks of the C ABI that need no GPU: the library loads, exports every function
the header declares, and rejects bad arguments before anything could be enqueued."""
import ctypes
import os
import re

import pytest
import torch

from paper_2604_03957_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = 0x7F0000001000  # a well-aligned, never dereferenced "device" address


def declared_functions():
    names = set()
    for header in ("bwta.h", "bwta_tuning.h"):
        text = open(os.path.join(ROOT, "include", header)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(bwta_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_every_declared_symbol_is_exported():
    names = declared_functions()
    assert set(names) == set(B.EXPORTS)
    for n in names:
        assert hasattr(B.raw(), n), n


def test_row_words_and_workspace():
    assert [B.plane_row_words(k) for k in (0, 1, 128, 129, 768, 4096, 11008)] == [0, 4, 4, 8, 24, 128, 344]
    assert B.workspace_bytes(0, 5, 5) == 0
    ws = B.workspace_bytes(4096, 3072, 768)
    assert ws % 256 == 0 and ws >= 2 * 4096 * 24 * 4 + 4096 * 768 // 2
    assert B.version() >= 1
    assert B.strerror(B.ERR_ALIGN) and B.strerror(0) == "ok"


def test_path_selection():
    assert B.get_path() == B.PATH_AUTO
    B.set_path(B.PATH_POPC)
    assert B.get_path() == B.PATH_POPC
    B.set_path(B.PATH_AUTO)
    with pytest.raises(B.BwtaError) as e:
        B.set_path(7)
    assert e.value.code == B.ERR_UNSUPPORTED
    assert B.auto_path(1, 11008, 4096) == B.PATH_POPC and B.auto_path(16, 11008, 4096) == B.PATH_FP4
    assert B.auto_path(2048, 4096, 4096) in (B.PATH_MFMA, B.PATH_FP4)
    # launches of bwta_linear: one kernel for short K, for few outputs and for one token; two otherwise; the hook
    # turns it off
    assert B.linear_launches(4096, 3072, 768) == 1 and B.linear_launches(4096, 768, 3072) == 1
    assert B.linear_launches(1, 768, 768) == 1 and B.linear_launches(16384, 11008, 1024) == 2
    assert B.linear_launches(16, 768, 768) == 1 and B.linear_launches(2048, 11008, 4096) == 2
    assert B.linear_launches(0, 8, 8) == 0 and B.linear_launches(8, 8, -1) == 0
    B.set_tile(900)
    try:
        for M, N, K in ((4096, 3072, 768), (4096, 768, 3072), (1, 768, 768)):
            assert B.linear_launches(M, N, K) == 2
    finally:
        B.set_tile(0)
    assert B.linear_launches(4096, 3072, 768) == 1


def test_planned_kernel_of_the_linear():
    """Which kernel bwta_linear takes on fp16 rows: the four one-launch kernels each where its rule says, the product
    kernel behind a ternarise launch elsewhere; the launch count follows."""
    def plan(M, N, K):
        k = B.planned_kernel(B.OPERAND_FP16, M, N, K)
        one = k in (B.KERNEL_LINEAR_FUSED, B.KERNEL_LINEAR_STRIP, B.KERNEL_LINEAR_ONE, B.KERNEL_LINEAR_ROWS)
        assert B.planned_rows(M, N, K) == (k == B.KERNEL_LINEAR_ROWS), (M, N, K)
        assert B.linear_launches(M, N, K) == (1 if one else 2), (M, N, K)
        return k

    assert plan(4096, 3072, 768) == plan(2, 49153, 8) == plan(520, 2049, 515) == B.KERNEL_LINEAR_FUSED
    assert plan(4096, 768, 3072) == plan(65, 8193, 2048) == plan(4200, 100, 1300) == B.KERNEL_LINEAR_STRIP
    for shape in ((2, 128, 8), (300, 515, 515), (64, 1536, 2048), (300, 100, 768)):
        assert plan(*shape) == B.KERNEL_LINEAR_ROWS, shape
    # bounds in K: of the strips of 16 tokens and of the slab kernel at decode-sized token counts, of the latter on wide matrices
    for (M, N), last in (((64, 768), 2048), ((2, 28000), 2048), ((2, 40000), 2048), ((64, 4096), 2560), ((64, 8193), 3072), ((128, 8192), 3072),
                         ((777, 2500), 16384), ((777, 1152), 32768), ((2048, 1536), 8192), ((4096, 768), 32768), ((256, 4096), 32768)):
        few = (M, N) in ((64, 768), (2, 28000))
        assert plan(M, N, last) == (B.KERNEL_LINEAR_ROWS if few else B.KERNEL_LINEAR_STRIP), (M, N, last)
        assert last == 32768 or plan(M, N, last + 1) in (B.KERNEL_GEMV_FP4, B.KERNEL_GEMM_FP4), (M, N, last)
    assert plan(512, 4096, 4096) == plan(1024, 3072, 4096) == B.KERNEL_GEMM_FP4
    assert plan(1, 11008, 4096) == plan(1, 1, 8) == plan(1, 128, 16384) == B.KERNEL_LINEAR_ONE
    assert plan(1, 128, 7) == B.KERNEL_GEMV_POPC and plan(16, 11008, 4096) == B.KERNEL_GEMV_FP4
    assert plan(2048, 11008, 4096) == B.KERNEL_GEMM_FP4
    assert B.planned_kernel(B.OPERAND_FP16, 0, 8, 8) == 0
    try:
        for path, want in ((B.PATH_POPC, B.KERNEL_GEMM_POPC), (B.PATH_MFMA, B.KERNEL_GEMM_MFMA_I8)):
            B.set_path(path)
            assert plan(4096, 768, 3072) == want
    finally:
        B.set_path(B.PATH_AUTO)


def test_planned_tile_of_the_tiled_product():
    """Tiles of 64 x 128 only in the windows where they are ahead: few more 128 x 128 tiles than compute units while the
    64 x 128 ones come to two each; 129 to 223, where 128 x 96 ones make one round only for a short K."""
    t = B.planned_tile
    assert t(300, 11008, 2048) == t(1600, 2500, 3072) == t(400, 9216, 1024) == 12        # 430, 500, 504 tiles of 64 x 128
    assert t(1024, 4608, 2048) == t(384, 11008, 1536) == t(1280, 3300, 3072) == 223      # 576, 516, 520 of them
    assert t(300, 11008, 3073) == t(1024, 4608, 1024) == t(1024, 4608, 1281) == 223 and t(1024, 4608, 1025) == 12
    assert t(600, 4096, 1536) == t(900, 2500, 1024) == t(300, 6144, 1536) == 12
    assert t(2048, 1536, 1280) == t(4096, 768, 1024) == 12 and t(2048, 1536, 1281) == t(4096, 768, 1536) == 13  # 96 divides N
    assert t(600, 4096, 1537) == t(900, 3001, 2048) == 13
    assert t(1200, 2500, 3072) == t(900, 3300, 2048) == t(384, 8192, 2048) == 12          # 128 x 96: more than a round
    assert t(384, 8192, 3073) == t(1200, 2500, 3073) == 22
    assert t(2048, 11008, 4096) == 243 and t(1024, 4096, 4096) == 223 and t(512, 4096, 4096) == 11
    assert t(4096, 3072, 768) == 23 and t(0, 8, 8) == 0
    huge_n = (1 << 32) // (344 * 4) + 1          # packed weights beyond the LDS-staged kernel's 32-bit offsets
    try:
        for forced in (22, 12, 243, 323):
            B.set_tile(forced)
            assert t(700, 700, 700) == forced
        assert t(700, huge_n, 11008) == 22 and t(700, 700, 700) == 323
        B.set_tile(5)                            # no tile: the rule's
        assert t(512, 4096, 4096) == 11
    finally:
        B.set_tile(0)


def test_planned_tile_of_short_products():
    """Below K = 1024 the tile follows the number of 128 x 128 tiles alone: 64 x 64 to 192, 64 x 128 to 384."""
    t = B.planned_tile
    assert [t(2048, 1536, 1023), t(2048, 1537, 768), t(2048, 3072, 100), t(2048, 3073, 768)] == [11, 12, 12, 23]
    assert t(129, 768, 768) == 11 and t(2048, 1536, 1024) == 12


def test_planned_kernel_of_small_linears():
    """Where bwta_linear's one launch is the kernel of 16-token strips, by workgroups of 128 channels and K: the edges."""
    r = B.planned_rows
    assert [r(1, 768, 768), r(2, 768, 768), r(2, 1, 8), r(2, 1, 7)] == [0, 1, 1, 0]
    assert [r(128, 4096, 2048), r(128, 4097, 2048), r(64, 768, 2048), r(64, 768, 2049)] == [1, 0, 1, 0]          # 256, 264 workgroups
    assert [r(128, 6144, 1280), r(128, 6145, 1280), r(128, 6144, 1281)] == [1, 0, 0]                              # 384, 392
    assert [r(512, 2048, 1024), r(513, 2048, 1024), r(512, 2048, 1281)] == [1, 0, 0]                              # 512, 528
    assert [r(256, 2048, K) for K in (6144, 6145)] == [1, 0] and [r(128, 2048, K) for K in (3072, 6144)] == [0, 0]
    assert [r(129, 896, 8192), r(129, 897, 8192), r(129, 384, 12288), r(129, 385, 12288), r(129, 384, 12289)] == [1, 0, 1, 0, 0]
    for M, N, K in ((64, 768, 768), (64, 100, 768), (64, 768, 1025)):
        assert r(M, N, K) == 1 and B.planned_kernel(B.OPERAND_FP16, M, N, K) == B.KERNEL_LINEAR_ROWS and B.linear_launches(M, N, K) == 1
    try:
        B.set_tile(901)                                                                                             # tuning: the other kernel
        assert r(64, 768, 768) == 0 and B.planned_kernel(B.OPERAND_FP16, 64, 768, 768) == B.KERNEL_LINEAR_FUSED
    finally:
        B.set_tile(0)


def test_planned_kernel_of_long_products():
    """Where the kernel of 16 x 16 blocks takes a product, by pairs of slabs (512 k) and tiles of 64 x 128: the edges."""
    w = B.planned_wide
    assert [w(512, 4096, K) for K in (3072, 3073, 11008)] == [0, 611, 611]                 # 256 tiles
    assert [w(513, 4096, K) for K in (2560, 2561, 3073, 4096, 4097, 8192)] == [0, 521, 611, 611, 521, 611]
    assert w(1300, 3001, 3000) == 0 and w(777, 3001, 2999) == 521                           # 64 x 128 tiles just fill two rounds
    assert [w(2048, 4096, K) for K in (2560, 3072, 3500, 4096, 11008)] == [0, 521, 0, 521, 521]
    assert w(3072, 4096, 4096) == 521 and [w(2048, 11008, K) for K in (3584, 3585, 4096)] == [0, 422, 422]
    assert [w(652, 16384, 5504), w(652, 16385, 5504), w(652, 16385, 3000)] == [521, 422, 0]  # 768, 774 tiles of 128 x 128, half a row of them empty
    assert w(2048, (1 << 32) // (344 * 4) + 1, 11008) == 0 and w(0, 8, 8) == 0              # beyond 32-bit offsets
    # on an operand that was prepared by its own call: seven and nine pairs, the last one half full, are left to the
    # other tiles where these are few, and seven or eight where 128 x 96 tiles make one round
    p = lambda *s: w(*s, prepared=True)
    assert [(w(512, 2048, K), p(512, 2048, K)) for K in (3072, 3073, 3328, 3329, 4096, 4097, 4352, 4353, 5121)] == \
        [(0, 0), (611, 0), (611, 0), (611, 611), (611, 611), (611, 0), (611, 0), (611, 611), (611, 611)]
    assert p(512, 2049, 3073) == p(512, 2049, 4097) == 611                                   # 136 tiles
    assert [(w(513, 4096, K), p(513, 4096, K)) for K in (3073, 3584, 3585, 4096, 4097, 5633)] == \
        [(611, 0), (611, 0), (611, 521), (611, 521), (521, 521), (611, 611)]
    assert p(513, 4895, 3073) == 0 and p(513, 4897, 3073) == 611                             # 255, 260 tiles of 128 x 96
    # .. and, whoever reads it, where these divide N
    assert [(w(1397, 1536, K), p(1397, 1536, K)) for K in (2560, 2561, 3073, 4608, 4609)] == [(0, 0), (0, 0), (0, 0), (0, 0), (521, 521)]
    assert w(1397, 1535, 3073) == w(7680, 480, 4000) == 611 and w(7680, 384, 4000) == 0
    assert all(w(M, N, K) == p(M, N, K) for M, N, K in ((512, 4096, 3073), (300, 11007, 3073), (2048, 4096, 4096), (2048, 11008, 4096)))
    one = [B.planned_kernel(B.OPERAND_FP16, *s) == B.KERNEL_LINEAR_STRIP for s in
           ((256, 4096, 5120), (256, 4096, 5121), (641, 768, 7168), (640, 768, 7168), (641, 768, 7169), (1280, 512, 12288), (1280, 513, 12288),
            (1300, 1536, 4096), (1024, 2048, 4096), (2048, 768, 7168), (2048, 768, 7169), (4096, 512, 11008), (4096, 768, 11008),
            (2048, 1152, 11008), (2048, 1152, 8192))]
    assert one == [True, False, True, False, False, True, False, True, False, True, False, True, True, False, True]
    # .. an odd number of pairs of slabs (512 k) leaves more to the slab kernel where it has one channel block per wavefront
    odd = [B.planned_kernel(B.OPERAND_FP16, *s) == B.KERNEL_LINEAR_STRIP for s in
           ((513, 1900, 5632), (512, 1900, 5632), (600, 1100, 6144), (600, 1100, 6145), (600, 1100, 6656), (600, 1100, 6657), (769, 500, 7680),
            (768, 500, 7680), (769, 500, 7681), (897, 600, 8704), (896, 600, 8704), (897, 600, 8705), (1200, 600, 9728))]
    assert odd == [True, False, False, True, True, False, True, False, False, True, False, False, False]
    try:
        B.set_tile(243)
        assert w(2048, 11008, 4096) == 0 and B.planned_tile(2048, 11008, 4096) == 243
        B.set_tile(611)
        assert w(2048, 11008, 4096) == 611
    finally:
        B.set_tile(0)


def test_planned_decode_blocks():
    """How many blocks of channel tiles a decode workgroup walks: the shapes measured on both sides of the rule."""
    b = B.planned_decode_blocks
    assert [b(16, 2041, 4500, 24), b(2, 4090, 5000, 32), b(3, 4096, 4500, 64), b(40, 4096, 11008, 16), b(16, 4096, 11008, 64)] == [2, 4, 8, 4, 8]
    assert b(40, 4096, 8192, 64) == 8 and b(4, 5000, 8192, 1) == b(16, 4096, 4096, 64) == b(16, 4096, 16384, 64) == 1
    # 6 or 8 wavefronts in one and a half to two rounds of 4 or 8 blocks, 4 blocks of 2 tiles for 6: one block each (or 4 in more rounds)
    assert [b(44, 12160, 8432, 6), b(20, 6144, 12285, 17), b(75, 1394, 7273, 20), b(82, 12105, 14867, 2), b(35, 2313, 16193, 25)] == [1] * 5
    assert b(59, 3456, 9118, 29) == b(40, 4096, 11008, 16) == b(50, 1024, 16164, 39) == 4 and b(28, 8058, 15744, 41) == 8
    # 5, 7, 9 and 10 wavefronts, and two blocks, keep two rounds
    assert [b(28, 8064, 4864, 12), b(59, 1880, 12821, 28), b(42, 589, 12906, 37), b(28, 4089, 19466, 14)] == [4, 4, 2, 8]
    assert b(1, 4096, 11008, 64) == b(129, 4096, 11008, 1) == b(16, 0, 8, 1) == b(16, 8, 8, 0) == 0  # other kernels, nothing
    assert b(16, 4096, 11008, 200) == b(16, 4096, 11008, 64)                                          # at most 64 to a launch


def _code(fn, *a, **k):
    with pytest.raises(B.BwtaError) as e:
        fn(*a, **k)
    return e.value.code


def test_quantize_pack_rejects_bad_arguments():
    q = B.bwta_quantize_pack_act
    kw = dict(M=4, K=256, stream=0, scale_mode=B.SCALE_VECTOR)
    assert _code(q, None, FAKE, FAKE, FAKE, **kw) == B.ERR_NULL
    assert _code(q, FAKE, None, FAKE, FAKE, **kw) == B.ERR_NULL          # scale needed in VECTOR mode
    assert _code(q, FAKE, FAKE, FAKE + 4, FAKE, **kw) == B.ERR_ALIGN       # planes are 16-byte aligned
    assert _code(q, FAKE, FAKE, FAKE, FAKE, **dict(kw, lda=255)) == B.ERR_SHAPE
    assert _code(q, FAKE, FAKE, FAKE, FAKE, **dict(kw, M=-1)) == B.ERR_SHAPE
    assert _code(q, FAKE, FAKE, FAKE, FAKE, **dict(kw, K=0)) == B.ERR_SHAPE
    assert _code(q, FAKE, FAKE, FAKE, FAKE, **dict(kw, a_dtype=9)) == B.ERR_UNSUPPORTED
    assert _code(q, FAKE, FAKE, FAKE, FAKE, **dict(kw, scale_mode=5)) == B.ERR_UNSUPPORTED
    q(FAKE, FAKE, FAKE, FAKE, **dict(kw, M=0))                            # empty input is a no-op


def test_pack_weights_rejects_bad_arguments():
    p = B.bwta_pack_weights
    assert _code(p, None, FAKE, N=4, K=128, stream=0) == B.ERR_NULL
    assert _code(p, FAKE, FAKE + 8, N=4, K=128, stream=0) == B.ERR_ALIGN
    assert _code(p, FAKE, FAKE, N=4, K=128, ldw=64, stream=0) == B.ERR_SHAPE
    assert _code(p, FAKE, FAKE, N=4, K=128, w_dtype=3, stream=0) == B.ERR_UNSUPPORTED
    p(FAKE, FAKE, N=0, K=128, stream=0)


def test_gemm_and_linear_reject_bad_arguments():
    g = B.bwta_gemm
    ws = B.workspace_bytes(8, 8, 128)
    kw = dict(M=8, N=8, K=128, stream=0, workspace_bytes=ws, a_scale_mode=B.SCALE_VECTOR,
              w_scale_mode=B.SCALE_VECTOR)
    assert _code(g, FAKE, None, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, **kw) == B.ERR_NULL   # a NULL mask alone is legal (binary activations)
    assert _code(g, FAKE, FAKE, FAKE, FAKE, FAKE, None, None, FAKE, **kw) == B.ERR_NULL   # no output at all
    assert _code(g, FAKE, FAKE, FAKE + 4, FAKE, FAKE, FAKE, FAKE, FAKE, **kw) == B.ERR_ALIGN
    assert _code(g, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, **dict(kw, ldo=7)) == B.ERR_SHAPE
    assert _code(g, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, None, **kw) == B.ERR_WORKSPACE
    assert _code(g, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, **dict(kw, workspace_bytes=ws - 1)) == B.ERR_WORKSPACE
    assert _code(g, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE + 16, **kw) == B.ERR_ALIGN
    assert _code(g, FAKE, FAKE, FAKE, None, FAKE, FAKE, FAKE, FAKE, **kw) == B.ERR_NULL    # s_a missing
    g(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, **dict(kw, N=0))
    lin = B.bwta_linear
    assert _code(lin, FAKE, FAKE, FAKE, FAKE, None, FAKE, **kw) == B.ERR_NULL
    assert _code(lin, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, **dict(kw, lda=100)) == B.ERR_SHAPE
    assert _code(lin, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, **dict(kw, workspace_bytes=0)) == B.ERR_WORKSPACE
    lin(FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, **dict(kw, M=0))


def test_linear_converts_its_arguments_like_the_other_calls():
    """bwta_linear's arguments travel in one packed block; integers outside a field's range wrap and what is no integer
    is refused by ctypes, as in the calls that pass them one by one."""
    lin = B.bwta_linear
    kw = dict(M=8, N=8, K=128, stream=0, workspace_bytes=B.workspace_bytes(8, 8, 128), a_scale_mode=B.SCALE_VECTOR,
              w_scale_mode=B.SCALE_VECTOR)
    bad_ws = (FAKE, FAKE, FAKE, FAKE, FAKE, FAKE + 16)      # a workspace on no 256-byte boundary: the last check
    assert _code(lin, *bad_ws, **kw) == B.ERR_ALIGN
    assert _code(lin, *bad_ws, **dict(kw, workspace_bytes=-1)) == B.ERR_ALIGN        # the largest size_t
    assert _code(lin, *bad_ws, **dict(kw, M=2 ** 32 + 8)) == B.ERR_ALIGN
    assert _code(lin, *bad_ws, **dict(kw, M=2 ** 31)) == B.ERR_SHAPE                 # negative as an int
    assert _code(lin, -256, *bad_ws[1:], **kw) == B.ERR_ALIGN
    lin(*bad_ws, **dict(kw, M=2 ** 32))                                              # no rows: nothing to do
    for bad in (dict(K=128.0), dict(K="128"), dict(M=None), dict(lda=128.5), dict(workspace_bytes="x")):
        with pytest.raises(ctypes.ArgumentError):
            lin(*bad_ws, **dict(kw, **bad))
        if "lda" not in bad and "workspace_bytes" not in bad:
            with pytest.raises(ctypes.ArgumentError):
                B.bwta_linear_static(*bad_ws[:5], **{k: v for k, v in dict(kw, **bad).items() if k != "workspace_bytes"})


def test_the_block_of_linear_arguments_states_its_size():
    call = B.raw().bwta_linear_call
    good = B._linear_pack(*[0] * 15, B._LINEAR_ARGS_SIZE)
    assert len(good) == B._LINEAR_ARGS_SIZE == 104
    assert call(good) == B.OK                                                        # M = N = 0
    assert call(B._linear_pack(*[0] * 16)) == B.ERR_UNSUPPORTED and call(None) == B.ERR_NULL


def test_native_marshalling_knows_the_python_forms():
    """Every natively marshalled call has the Python form's parameters, in its order, and hands it whatever is not the
    ordinary form (here: host tensors, integers, wrong argument lists) as it came."""
    import inspect
    table = B._native.parameters()
    assert len(table) == 11
    for name, (positional, params) in table.items():
        sig = inspect.signature(getattr(B, name))
        assert [p.name for p in sig.parameters.values()] == params, name
        assert sum(p.kind is p.POSITIONAL_OR_KEYWORD for p in sig.parameters.values()) == positional, name
        seen = []
        f = B._native.bind(name, 0, lambda *a, **k: seen.append((a, k)))    # no address: it must not be called
        host = torch.zeros(4)
        required = {p.name: 1 for p in sig.parameters.values() if p.kind is p.KEYWORD_ONLY and p.default is p.empty}
        for args, kw in (((host,) * positional, required), ((FAKE,) * positional, required), ((), {}), ((None,) * (positional + 1), required),
                         ((None,) * positional, dict(required, M=1.5, K=1.5)), ((None,) * positional, dict(required, K=2 ** 70)),
                         ((None,) * positional, dict(required, stream=0)), ((None,) * positional, dict(required, nothing=1))):
            f(*args, **kw)
            assert len(seen) == 1 and len(seen[0][0]) == len(args) and all(x is y for x, y in zip(seen[0][0], args)) and seen[0][1] == kw
            seen.clear()
    with pytest.raises(KeyError):
        B._native.bind("bwta_nothing", 0, print)


def test_native_calls_are_used_like_python_functions():
    """What programs do with a function besides calling it: attributes, methods, weak references, pickles and copies,
    inspection."""
    import copy
    import functools
    import inspect
    import pickle
    import types
    import weakref
    calls = []

    def bwta_linear(A, s_a, wsign, s_w, out, workspace, *, M, N, K, lda=None):
        """a docstring"""
        calls.append((A, M))

    f = B._native.bind("bwta_linear", 0, bwta_linear)
    assert f.__name__ == "bwta_linear" and f.__doc__ == "a docstring" and f.__module__ == __name__ and repr(f) == repr(bwta_linear)
    assert isinstance(f, types.FunctionType) and inspect.isfunction(f) and inspect.signature(f) == inspect.signature(bwta_linear)
    f.note = 5
    assert f.note == 5 and getattr(functools.wraps(f)(lambda: 0), "note") == 5
    del f.note
    assert not hasattr(f, "note")

    class Layer:
        linear = f

    layer = Layer()
    layer.linear(None, None, None, None, None, M=1, N=2, K=3)
    Layer.linear(None, None, None, None, None, None, M=4, N=5, K=6)
    assert calls == [(layer, 1), (None, 4)]
    r = weakref.ref(f)
    assert r() is f
    for g in (copy.copy(B.bwta_linear), copy.deepcopy({"f": B.bwta_linear})["f"], pickle.loads(pickle.dumps(B.bwta_linear)), pickle.loads(pickle.dumps(B.bwta_linear, 0))):
        assert g is B.bwta_linear
    Layer.linear = None
    del f, layer
    assert r() is None


def _package_copy(tmp_path):
    """The package's Python files and built libraries in a folder of their own: what a child interpreter imports."""
    import shutil
    src = os.path.dirname(os.path.abspath(B.__file__))
    dst = tmp_path / os.path.basename(src)
    (dst / "csrc").mkdir(parents=True)
    for f in ("__init__.py", "binding.py"):
        shutil.copy(os.path.join(src, f), str(dst / f))
    for f in (B.LIB_PATH, B.NATIVE_PATH):
        shutil.copy(f, str(dst / "csrc" / os.path.basename(f)))
    return dst


_CHILD = """
import types, warnings
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    from paper_2604_03957_amd import binding as B
says = [str(w.message) for w in seen if issubclass(w.category, RuntimeWarning) and "marshalled in Python" in str(w.message)]
python = [type(getattr(B, n)) is types.FunctionType for n in ("bwta_linear", "bwta_gemm", "bwta_matmul_bool_prepared")]
try:
    B.bwta_linear(None, None, 0x1000, None, 0x1000, None, M=1, N=1, K=128, stream=0)
    code = 0
except B.BwtaError as e:
    code = e.code
print("RESULT", len(says), all(python), any(python), code)
"""


def _child_import(folder):
    import subprocess
    import sys
    env = {k: v for k, v in os.environ.items() if k != "BWTA_LIB"}
    r = subprocess.run([sys.executable, "-c", _CHILD], cwd=str(folder), env=dict(env, PYTHONPATH=str(folder)), stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True, timeout=300)
    lines = [l for l in r.stdout.splitlines() if l.startswith("RESULT")]
    assert r.returncode == 0 and len(lines) == 1, r.stdout[-2000:]
    return lines[0]


def test_native_marshalling_of_another_build_is_not_called(tmp_path):
    """The extension holds the C signatures it was compiled with.  One of other sources than the library's, or for another
    torch, is left alone, with a warning: the Python forms make the calls."""
    if os.environ.get("BWTA_LIB"):
        pytest.skip("a library built some other way is loaded")
    pkg = _package_copy(tmp_path)
    native = pkg / "csrc" / os.path.basename(B.NATIVE_PATH)
    assert _child_import(tmp_path) == "RESULT 0 False False %d" % B.ERR_NULL
    good, mine = native.read_bytes(), B._native.identity().encode()
    assert good.count(mine) == 1 and B._native.identity() == B._native_identity()
    for other in (b"0" * 12 + mine[12:], mine[:13] + b"1" * (len(mine) - 13)):
        native.write_bytes(good.replace(mine, other))
        assert _child_import(tmp_path) == "RESULT 1 True True %d" % B.ERR_NULL
    assert good.count(b"\0identity\0") == 1  # one that does not say what it was built from
    native.write_bytes(good.replace(b"\0identity\0", b"\0identitx\0"))
    assert _child_import(tmp_path) == "RESULT 1 True True %d" % B.ERR_NULL


def test_import_without_the_native_marshalling(tmp_path):
    """No extension, or one that does not load: the package imports, warns and makes every call in its Python form.  (The
    library itself has no such substitute.)"""
    if os.environ.get("BWTA_LIB"):
        pytest.skip("a library built some other way is loaded")
    pkg = _package_copy(tmp_path)
    native = pkg / "csrc" / os.path.basename(B.NATIVE_PATH)
    native.write_bytes(b"no shared object")
    assert _child_import(tmp_path) == "RESULT 1 True True %d" % B.ERR_NULL
    native.unlink()
    assert _child_import(tmp_path) == "RESULT 1 True True %d" % B.ERR_NULL


def test_build_without_what_the_native_marshalling_needs(tmp_path, monkeypatch, capsys):
    """No C++ compiler, or no headers of Python or torch: said, an older extension is taken away, and the build goes on."""
    from paper_2604_03957_amd import build
    for what in ("_binding_compiler", "_binding_headers"):
        files = [tmp_path / "_bwta_native.so", tmp_path / "binding_identity.txt"]
        for f in files:
            f.write_text("left from before")
        with monkeypatch.context() as m:
            m.setattr(build, "BINDING", str(files[0]))
            m.setattr(build, "BINDING_ID", str(files[1]))
            m.setattr(build, what, lambda: None)
            assert build.build_binding("0" * 12, verbose=False) is None
        assert "not built" in capsys.readouterr().out and not any(f.exists() for f in files)
    assert build._binding_compiler() and build._binding_headers()


def test_prepare_and_gemm_prepared_reject_bad_arguments():
    pb = B.prepared_bytes(8, 128)
    assert pb % 256 == 0 and pb > 0 and B.prepared_bytes(0, 128) == 0
    kw = dict(M=8, K=128, stream=0, a_scale_mode=B.SCALE_VECTOR, prepared_bytes=pb)
    assert _code(B.bwta_prepare_act, None, FAKE, FAKE, **kw) == B.ERR_NULL
    assert _code(B.bwta_prepare_act, FAKE, FAKE, FAKE, **dict(kw, prepared_bytes=pb - 1)) == B.ERR_WORKSPACE
    assert _code(B.bwta_prepare_act, FAKE, FAKE, FAKE + 32, **kw) == B.ERR_ALIGN
    assert _code(B.bwta_prepare_act, FAKE, FAKE, FAKE, **dict(kw, lda=64)) == B.ERR_SHAPE
    kw = dict(M=8, N=8, K=128, stream=0, a_scale_mode=B.SCALE_VECTOR, w_scale_mode=B.SCALE_VECTOR, prepared_bytes=pb,
              fmt=B.PREPARED_PLANES)
    g = B.bwta_gemm_prepared
    assert _code(g, None, FAKE, FAKE, FAKE, None, FAKE, **kw) == B.ERR_WORKSPACE
    assert _code(g, FAKE, None, FAKE, FAKE, None, FAKE, **kw) == B.ERR_NULL
    assert _code(g, FAKE, FAKE, FAKE, FAKE, None, None, **kw) == B.ERR_NULL
    assert _code(g, FAKE, FAKE, FAKE, FAKE, None, FAKE, **dict(kw, ldo=4)) == B.ERR_SHAPE
    # the operand's format travels with it: an id that names neither layout is refused before any launch
    for bad in (0, 3, -1, 77):
        assert _code(g, FAKE, FAKE, FAKE, FAKE, None, FAKE, **dict(kw, fmt=bad)) == B.ERR_UNSUPPORTED


def test_prepared_format_and_planned_kernel():
    """What bwta_prepare_act writes is decided once and reported; the consumer's kernel follows from
    that id and the shape, never from a second look at the path setting.  In particular prepared
    planes never resolve to the tiled FP4 kernel, which would need scratch the call does not have:
    that includes a decode-sized token count against a packed matrix too large for the decode
    kernel's 32-bit offsets (the shape that used to fall through to it)."""
    assert B.prepared_format(2048, 4096) == B.PREPARED_FP4 and B.prepared_format(16, 4096) == B.PREPARED_PLANES
    assert B.prepared_format(128, 11008) == B.PREPARED_PLANES and B.prepared_format(129, 11008) == B.PREPARED_FP4
    assert B.planned_kernel(B.PREPARED_FP4, 2048, 4096, 4096) == B.KERNEL_GEMM_FP4
    assert B.planned_kernel(B.PREPARED_PLANES, 16, 11008, 4096) == B.KERNEL_GEMV_FP4
    assert B.planned_kernel(0, 2048, 4096, 4096) == B.KERNEL_GEMM_FP4
    assert B.planned_kernel(0, 1, 4096, 4096) == B.KERNEL_GEMV_POPC
    huge_n = (1 << 32) // (344 * 4) + 1                       # (N + 4096) * row bytes no longer fits 32 bits
    for M in (2, 16, 128):
        assert B.planned_kernel(0, M, huge_n, 11008) == B.KERNEL_GEMM_FP4          # with a workspace: tiled kernel
        k = B.planned_kernel(B.PREPARED_PLANES, M, huge_n, 11008)
        assert k in (B.KERNEL_GEMM_MFMA_I8, B.KERNEL_GEMM_POPC, B.KERNEL_GEMV_POPC), k
    # prepared planes under every path setting, over a grid of shapes: never the kernel that needs scratch
    try:
        for path in (B.PATH_AUTO, B.PATH_POPC, B.PATH_MFMA, B.PATH_FP4):
            B.set_path(path)
            for M in (1, 2, 16, 128, 129, 2048):
                for N in (1, 128, 4096, huge_n):
                    for K in (32, 1024, 4096, 11008, 30000):
                        assert B.planned_kernel(B.PREPARED_PLANES, M, N, K) not in (0, B.KERNEL_GEMM_FP4)
                        assert B.planned_kernel(B.PREPARED_FP4, M, N, K) == B.KERNEL_GEMM_FP4
    finally:
        B.set_path(B.PATH_AUTO)
    assert B.planned_kernel(5, 8, 8, 8) == 0 and B.planned_kernel(0, 0, 8, 8) == 0


def test_attention_entry_points_reject_bad_arguments():
    qb = B.bwta_quantize_pack_bool
    kw = dict(M=4, K=256, stream=0, scale_mode=B.SCALE_SCALAR)
    assert _code(qb, None, FAKE, FAKE, **kw) == B.ERR_NULL
    assert _code(qb, FAKE, None, FAKE, **kw) == B.ERR_NULL
    assert _code(qb, FAKE, FAKE, FAKE + 8, **kw) == B.ERR_ALIGN
    assert _code(qb, FAKE, FAKE, FAKE, **dict(kw, lda=100)) == B.ERR_SHAPE
    qb(FAKE, FAKE, FAKE, **dict(kw, M=0))                                   # empty: nothing enqueued
    mm = B.bwta_matmul_tt
    kw = dict(batch=2, M=8, N=8, K=128, stream=0, a_scale_mode=B.SCALE_NONE, b_scale_mode=B.SCALE_NONE)
    assert _code(mm, None, FAKE, FAKE, FAKE, None, None, FAKE, FAKE, **kw) == B.ERR_NULL
    assert _code(mm, FAKE, None, FAKE, None, None, None, None, None, **kw) == B.ERR_NULL      # no output at all
    assert _code(mm, FAKE, FAKE + 4, FAKE, FAKE, None, None, FAKE, FAKE, **kw) == B.ERR_ALIGN
    assert _code(mm, FAKE, FAKE, FAKE, FAKE, None, None, FAKE, FAKE, **dict(kw, strideA=8)) == B.ERR_SHAPE
    assert _code(mm, FAKE, FAKE, FAKE, FAKE, None, None, FAKE, FAKE, **dict(kw, strideA=8 * 4 + 2)) == B.ERR_ALIGN
    assert _code(mm, FAKE, FAKE, FAKE, FAKE, None, None, FAKE, FAKE, **dict(kw, ldo=4)) == B.ERR_SHAPE
    assert _code(mm, FAKE, FAKE, FAKE, FAKE, None, None, FAKE, FAKE, **dict(kw, alpha=float("inf"))) == B.ERR_UNSUPPORTED
    assert _code(mm, FAKE, FAKE, FAKE, FAKE, None, None, FAKE, FAKE, **dict(kw, batch=-1)) == B.ERR_SHAPE
    mm(FAKE, FAKE, FAKE, FAKE, None, None, FAKE, FAKE, **dict(kw, batch=0))  # empty batch: nothing enqueued


def test_weight_preparation_entry_points_reject_bad_arguments():
    pw = B.bwta_prepare_weights
    kw = dict(N=4, K=256, stream=0)
    assert _code(pw, None, FAKE, FAKE, **kw) == B.ERR_NULL
    assert _code(pw, FAKE, FAKE, None, **kw) == B.ERR_NULL
    assert _code(pw, FAKE, FAKE + 4, FAKE, **kw) == B.ERR_ALIGN
    assert _code(pw, FAKE, FAKE, FAKE, **dict(kw, ldw=255)) == B.ERR_SHAPE
    assert _code(pw, FAKE, FAKE, FAKE, **dict(kw, K=32769)) == B.ERR_UNSUPPORTED
    pw(FAKE, FAKE, FAKE, **dict(kw, N=0))
    sc = B.bwta_act_scale
    kw = dict(M=4, K=256, stream=0)
    assert _code(sc, None, FAKE, **kw) == B.ERR_NULL
    assert _code(sc, FAKE, FAKE + 1, **kw) == B.ERR_ALIGN
    assert _code(sc, FAKE, FAKE, **dict(kw, lda=8)) == B.ERR_SHAPE
    assert _code(sc, FAKE, FAKE, **dict(kw, K=40000)) == B.ERR_UNSUPPORTED
    sc(FAKE, FAKE, **dict(kw, M=0))
    au = B.bwta_prepare_act_autoscale
    kw = dict(M=4, K=256, stream=0, prepared_bytes=B.prepared_bytes(4, 256))
    assert _code(au, None, FAKE, FAKE, **kw) == B.ERR_NULL
    assert _code(au, FAKE, None, FAKE, **kw) == B.ERR_NULL
    assert _code(au, FAKE, FAKE + 1, FAKE, **kw) == B.ERR_ALIGN
    assert _code(au, FAKE, FAKE, FAKE + 16, **kw) == B.ERR_ALIGN
    assert _code(au, FAKE, FAKE, FAKE, **dict(kw, lda=8)) == B.ERR_SHAPE
    assert _code(au, FAKE, FAKE, FAKE, **dict(kw, prepared_bytes=16)) == B.ERR_WORKSPACE
    assert _code(au, FAKE, FAKE, None, **kw) == B.ERR_WORKSPACE
    assert _code(au, FAKE, FAKE, FAKE, **dict(kw, K=40000, prepared_bytes=1 << 30)) == B.ERR_UNSUPPORTED
    au(FAKE, FAKE, FAKE, **dict(kw, M=0))


def test_prepared_attention_product_rejects_bad_arguments():
    f = B.bwta_matmul_bool_prepared
    kw = dict(batch=2, M=64, N=128, K=256, stream=0, prepared_bytes=B.prepared_bytes(256, 256), fmt=B.PREPARED_FP4)
    assert _code(f, None, FAKE, None, None, FAKE, **kw) == B.ERR_NULL
    assert _code(f, FAKE, FAKE, None, None, None, **kw) == B.ERR_NULL
    assert _code(f, FAKE, None, None, None, FAKE, **kw) == B.ERR_WORKSPACE
    assert _code(f, FAKE, FAKE, None, None, FAKE, **dict(kw, prepared_bytes=64)) == B.ERR_WORKSPACE
    assert _code(f, FAKE, FAKE + 16, None, None, FAKE, **kw) == B.ERR_ALIGN
    assert _code(f, FAKE + 4, FAKE, None, None, FAKE, **kw) == B.ERR_ALIGN
    assert _code(f, FAKE, FAKE, None, None, FAKE, **dict(kw, strideA=64 * 8 + 2)) == B.ERR_ALIGN
    assert _code(f, FAKE, FAKE, None, None, FAKE, **dict(kw, N=96)) == B.ERR_UNSUPPORTED      # not a multiple of 128
    assert _code(f, FAKE, FAKE, None, None, FAKE, **dict(kw, fmt=B.PREPARED_PLANES)) == B.ERR_UNSUPPORTED  # needs fragments
    assert _code(f, FAKE, FAKE, None, None, FAKE, **dict(kw, fmt=0)) == B.ERR_UNSUPPORTED
    assert _code(f, FAKE, FAKE, None, None, FAKE, **dict(kw, alpha=float("nan"))) == B.ERR_UNSUPPORTED
    assert _code(f, FAKE, FAKE, None, None, FAKE, **dict(kw, ldo=64)) == B.ERR_SHAPE
    assert _code(f, FAKE, FAKE, None, None, FAKE, **dict(kw, strideA=8)) == B.ERR_SHAPE
    f(FAKE, FAKE, None, None, FAKE, **dict(kw, batch=0))


def test_static_scratch_entry_point_refuses_oversized_shapes_on_the_host():
    assert B.static_scratch_bytes() == 32 << 20
    lin = B.bwta_linear_static
    kw = dict(stream=0, a_scale_mode=B.SCALE_VECTOR, w_scale_mode=B.SCALE_VECTOR)
    assert B.workspace_bytes(8192, 768, 11008) > B.static_scratch_bytes()
    assert _code(lin, FAKE, FAKE, FAKE, FAKE, FAKE, M=8192, N=768, K=11008, **kw) == B.ERR_TOO_LARGE
    assert _code(lin, None, None, None, None, None, M=8192, N=768, K=11008, **kw) == B.ERR_TOO_LARGE  # size first
    assert B.strerror(B.ERR_TOO_LARGE) != "unknown error code"
    lin(FAKE, FAKE, FAKE, FAKE, FAKE, M=0, N=768, K=11008, **kw)   # empty: a no-op, no device needed
