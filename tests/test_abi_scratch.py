"""Host-side validation of the calls with a scratch of the library's own layout and of lutnn_bias_gradient: everything here is
refused before anything is launched (no GPU needed)."""
import ctypes

import pytest

import paper_2302_03213_amd as lut

OK, NULL, SHAPE, UNSUPPORTED, ALIGN = 0, "LUTNN_E_NULL", "LUTNN_E_SHAPE", "LUTNN_E_UNSUPPORTED", "LUTNN_E_ALIGN"
X, Y, S = ctypes.c_void_p(0x10000), ctypes.c_void_p(0x20000), ctypes.c_void_p(0x30000)


def name(code):
    return lut.LIB.lutnn_status_string(code).decode()


def layer(C=100, K=16, V=4, M=1000, dtype=lut.TABLE_I8, packed=0x50000, table=0x40000):
    return ctypes.byref(lut.binding._CLayer(C, K, V, M, dtype, 0, 0x60000, table, packed, 0x70000, None))


def test_scratch_bytes():
    f = lut.LIB.lutnn_linear_scratch_bytes
    assert f(layer(), 5000, 0) == 5000 * 128 and f(layer(), 5000, 1) == 5000 * 128  # sparse lookup: rows padded to 32 bytes
    assert f(layer(C=64), 5000, 0) == 5000 * 64
    assert f(layer(K=40, packed=None), 5000, 0) == 5000 * 100  # no matrix form: dense rows
    assert f(layer(dtype=lut.TABLE_F32, packed=None), 5000, 0) == 5000 * 100
    assert f(layer(), 1, 0) == 0 and f(layer(M=37, C=20), 8, 0) == 0 and f(layer(dtype=lut.TABLE_I4), 1, 0) == 0  # one launch
    assert f(layer(), 0, 0) == 0 and f(layer(), -1, 0) == 0 and f(layer(C=0), 10, 0) == 0 and f(None, 10, 0) == 0
    assert lut.LIB.lutnn_conv2d_scratch_bytes(layer(), 5000) == 5000 * 128


def test_the_variant_that_runs():
    """... agrees with the scratch that is asked for: none for one launch, padded index rows for the sparse lookup."""
    f, bytes_of = lut.LIB.lutnn_scratch_variant, lut.LIB.lutnn_linear_scratch_bytes
    FUSED, SMFMAC, LDS = lut.binding.VARIANT_FUSED, lut.binding.VARIANT_SMFMAC, lut.binding.VARIANT_LDS
    assert f(layer(), 5000, 0) == f(layer(), 5000, 1) == f(layer(), 5000, 2) == SMFMAC  # any number of codebooks
    assert f(layer(M=37, C=20), 8, 0) == f(layer(dtype=lut.TABLE_I4), 1, 1) == FUSED  # any width, INT4
    assert f(layer(M=37, C=20), 8, 2) == f(layer(K=40, packed=None), 5000, 0) == LDS
    for C in (20, 75, 128, 700):
        for N in (1, 40, 1000, 9000):
            for tree in (0, 1):
                v, n = f(layer(C=C), N, tree), bytes_of(layer(C=C), N, tree)
                assert n == {FUSED: 0, SMFMAC: N * ((C + 31) // 32 * 32), LDS: N * C}[v]
    MFMA = lut.binding.VARIANT_MFMA
    assert [f(layer(C=C), 20000, call) for call in (0, 1, 2) for C in (1, 8, 9)] == [MFMA, MFMA, SMFMAC] * 3
    assert f(layer(), 0, 0) == f(None, 10, 0) == f(layer(C=0), 10, 0) == f(layer(), 10, 3) == -1


def test_one_launch_where_the_searches_are_few():
    """Every workgroup repeats the searches of its rows: thousands of workgroups and long searches take two launches."""
    f = lut.LIB.lutnn_scratch_variant
    FUSED, LDS = lut.binding.VARIANT_FUSED, lut.binding.VARIANT_LDS
    for C, K, V, M, N, want in [(1, 256, 32, 4096, 1369, LDS), (3, 256, 32, 4096, 1038, LDS), (1, 64, 2, 3072, 2847, LDS), (1, 256, 2, 256, 200, FUSED),
                                (6, 16, 8, 4096, 300, FUSED), (20, 100, 2, 128, 15, FUSED)]:
        assert f(layer(C=C, K=K, V=V, M=M, dtype=lut.TABLE_F32, packed=None), N, 0) == want, (C, K, V, M, N)


def test_few_codebooks_and_many_outputs_take_the_matrix_form():
    f, MFMA = lut.LIB.lutnn_scratch_variant, lut.binding.VARIANT_MFMA
    for C, M, N, dtype in [(2, 3436, 1311, lut.TABLE_I4), (1, 2368, 1323, lut.TABLE_I4), (4, 2944, 1282, lut.TABLE_I4), (3, 234, 17210, lut.TABLE_I4)]:
        assert f(layer(C=C, V=2, M=M, dtype=dtype), N, 2) == MFMA, (C, M, N)
    for C, M, N, dtype in [(64, 64, 3136, lut.TABLE_I8), (2, 300, 200, lut.TABLE_I4), (20, 128, 5000, lut.TABLE_I8)]:
        assert f(layer(C=C, V=2, M=M, dtype=dtype), N, 2) == lut.binding.VARIANT_LDS, (C, M, N)


def test_what_is_refused():
    call = lut.LIB.lutnn_linear_scratch
    n = 5000 * 128
    for args, want in [((layer(), X, 5000, 400, Y, 1000, None, n, None), NULL), ((layer(), X, 5000, 400, Y, 1000, S, n - 1, None), SHAPE),
                       ((layer(), X, 5000, 400, Y, 1000, ctypes.c_void_p(0x30004), n, None), ALIGN),
                       ((layer(), X, 5000, 399, Y, 1000, S, n, None), SHAPE), ((layer(), X, 5000, 400, Y, 999, S, n, None), SHAPE),
                       ((layer(), None, 5000, 400, Y, 1000, S, n, None), NULL), ((layer(), X, 5000, 400, None, 1000, S, n, None), NULL),
                       ((layer(packed=0x50004), X, 5000, 400, Y, 1000, S, n, None), ALIGN),
                       ((layer(), X, 1, 400, None, 1000, None, 0, None), NULL), ((None, X, 1, 400, Y, 1000, None, 0, None), NULL)]:
        assert name(call(*args)) == want, args
    assert call(layer(), None, 0, 400, None, 1000, None, 0, None) == OK  # an empty batch
    tree = lut.binding._CTree(100, 4, 3, 0, 0x80000, 0x90000)
    assert name(lut.LIB.lutnn_linear_tree_scratch(layer(), ctypes.byref(tree), X, 5000, 400, Y, 1000, S, n, None)) == SHAPE  # K != 2^3
    geom = lut.binding._CConvGeom(100, 20, 20, 2, 2, 1, 1, 0, 0, 0)
    conv = lut.LIB.lutnn_conv2d_scratch
    rows = 16 * 19 * 19
    assert name(conv(layer(), X, 16, ctypes.byref(geom), Y, 1000, S, rows * 128 - 1, None)) == SHAPE
    assert name(conv(layer(V=5, C=80), X, 16, ctypes.byref(geom), Y, 1000, S, rows * 128, None)) == UNSUPPORTED
    assert name(conv(layer(), None, 16, ctypes.byref(geom), Y, 1000, S, rows * 128, None)) == NULL


def test_one_launch_with_a_variant_takes_the_layers_it_took():
    """Long rows of indices for many narrow outputs: refused by the calls with a variant, run by those without."""
    linear, tree_call = lut.LIB.lutnn_linear, lut.LIB.lutnn_linear_tree
    FUSED, AUTO = lut.binding.VARIANT_FUSED, lut.binding.VARIANT_AUTO
    for C, M in [(2799, 64), (318, 4), (516, 16), (8193, 256), (16500, 768)]:
        l = layer(C=C, K=64, V=1, M=M, dtype=lut.TABLE_F32, packed=None)
        assert name(linear(l, X, 3, C, Y, M, FUSED, S, None)) == UNSUPPORTED
        assert name(linear(l, X, 3, C, Y, M, AUTO, None, None)) == NULL
        assert lut.LIB.lutnn_linear_auto_variant(l, None, 3) == lut.binding.VARIANT_LDS
        tree = lut.binding._CTree(C, 1, 6, 0, 0x80000, 0x90000)
        assert name(tree_call(l, ctypes.byref(tree), X, 3, C, Y, M, FUSED, S, None)) == UNSUPPORTED
    for C, M in [(2048, 64), (128, 4), (8192, 256), (16384, 768), (32768, 1024)]:
        l = layer(C=C, K=64, V=1, M=M, dtype=lut.TABLE_F32, packed=None)
        assert lut.LIB.lutnn_linear_auto_variant(l, None, 3) == FUSED


@pytest.mark.parametrize("args,want", [((X, 100, 7, 8, 1, Y, S, 1 << 20, None), SHAPE), ((X, 100, 8, 3, 1, Y, S, 1 << 20, None), UNSUPPORTED),
                                       ((X, 100, 8, 8, 0, Y, S, 1 << 20, None), SHAPE), ((X, -1, 8, 8, 1, Y, S, 1 << 20, None), SHAPE),
                                       ((None, 100, 8, 8, 1, Y, S, 1 << 20, None), NULL), ((X, 100, 8, 8, 1, None, S, 1 << 20, None), NULL),
                                       ((X, 100, 8, 8, 1, Y, None, 1 << 20, None), NULL), ((X, 100, 8, 8, 49, Y, S, 100 * 8 * 4 - 1, None), SHAPE),
                                       ((ctypes.c_void_p(0x10002), 100, 8, 8, 1, Y, S, 1 << 20, None), ALIGN)])
def test_bias_gradient_refuses(args, want):
    assert name(lut.LIB.lutnn_bias_gradient(*args)) == want
