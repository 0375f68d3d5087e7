"""GPU parity of the table reads straight from global memory (arXiv 2302.03213, Eq. 4) at widths, numbers of codebooks and
addresses that are multiples of nothing, for the stand-alone lookups and the one-launch form of lutnn_linear_scratch.
INT8 and INT4 tables bit-exact; an fp32 sum of C terms within C half ulps of the sum of magnitudes."""
import numpy as np
import pytest
import torch

import lutnn_workloads as wl
import oracle
from gpu_util import dev, host, near_tie_report

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lut():
    import paper_2302_03213_amd as lut_mod
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return lut_mod


def at_offset(a, offset):
    """A device copy of the array that starts `offset` elements after an aligned address and ends where its memory does."""
    flat = torch.empty(a.size + offset, dtype=torch.from_numpy(a[:0].copy()).dtype, device="cuda")
    flat[offset:] = torch.from_numpy(a.reshape(-1))
    return flat[offset:].view(a.shape)


def table_case(lut, dtype, C, K, M, offset, seed):
    rng = np.random.default_rng(seed)
    P = torch.zeros((C, K, 4), device="cuda")
    bias = rng.standard_normal(M).astype(np.float32)
    if dtype == "f32":
        T = rng.standard_normal((C, K, M)).astype(np.float32)
        layer = lut.LutLayer(P, at_offset(T, offset), lut.TABLE_F32, M, bias=dev(bias))
        return layer, bias, T, None
    top = 7 if dtype == "i4" else 127
    q = rng.integers(-top, top + 1, (C, K, M)).astype(np.int8)
    layer = lut.LutLayer(P, at_offset(oracle.pack_nibbles(q) if dtype == "i4" else q, offset),
                         lut.TABLE_I4 if dtype == "i4" else lut.TABLE_I8, M, scale=dev(np.array([0.37], np.float32)), bias=dev(bias))
    return layer, bias, q, np.float32(0.37)


def check(got, T, s, idx, bias):
    if s is None:
        ref = oracle.lookup_f32(T.astype(np.float32), idx, bias).astype(np.float64)
        picked = np.abs(np.take_along_axis(T[None], idx[:, :, None, None].astype(np.int64), axis=2)[:, :, 0]).sum(axis=1)
        assert (np.abs(got - ref) <= (T.shape[0] + 1) * 2.0 ** -24 * 2 * (picked + np.abs(bias))).all()
    else:
        np.testing.assert_array_equal(got, oracle.lookup_i8(T, s, idx, bias))


# N, C, K, M: one group of columns and a column more, rows of a wavefront less, just and more, the split form, batches of
# sixteen codebooks and what is left of them, K past the staged kernels
SHAPES = [(5, 1, 16, 4), (70, 3, 16, 5), (33, 15, 8, 7), (40, 16, 16, 9), (29, 17, 16, 63), (300, 31, 16, 131), (9, 66, 16, 255),
          (7, 67, 16, 257), (3, 130, 8, 1021), (2, 513, 16, 515), (150, 33, 200, 37), (1300, 5, 256, 301), (17, 9, 16, 3)]


@pytest.mark.parametrize("dtype", ["i8", "i4", "f32"])
@pytest.mark.parametrize("N,C,K,M", SHAPES)
def test_lookup(lut, dtype, N, C, K, M):
    for offset in (0, 1):
        layer, bias, T, s = table_case(lut, dtype, C, K, M, offset, seed=N + C + M)
        idx = np.random.default_rng(C).integers(0, K, (N, C)).astype(np.uint8)
        out = torch.full((N, M + 3), -3.5, device="cuda")
        lut.lookup(layer, at_offset(idx, offset), "lds", out=out[:, :M])
        check(host(out[:, :M]), T, s, idx, bias)
        assert (host(out[:, M:]) == -3.5).all()


@pytest.mark.parametrize("dtype", ["i8", "f32"])
@pytest.mark.parametrize("N,C,K,M", SHAPES)
def test_lookup16(lut, dtype, N, C, K, M):
    for offset in (0, 1):
        layer, bias, T, s = table_case(lut, dtype, C, K, M, offset, seed=N + C + M)
        idx = np.random.default_rng(C).integers(0, K, (N, C)).astype(np.uint8)
        got = host(lut.lookup16(layer, at_offset(idx.astype(np.int16), offset)))
        check(got, T, s, idx, bias)


@pytest.mark.parametrize("dtype", ["i8", "i4", "f32"])
@pytest.mark.parametrize("N,C,V,M", [(1, 5, 4, 7), (3, 33, 2, 143), (50, 13, 8, 238), (2, 70, 4, 259), (1, 300, 2, 1001), (33, 20, 4, 520)])
def test_one_launch(lut, dtype, N, C, V, M):
    w = wl.make_layer("t", N, C, 16, V, M, "f32", seed=N + C + M)
    code = {"i8": lut.TABLE_I8, "i4": lut.TABLE_I4, "f32": lut.TABLE_F32}[dtype]
    layer = lut.build_table(dev(w.P), dev(w.W), code, bias=dev(w.bias))
    assert lut.LIB.lutnn_linear_scratch_bytes(layer.ref, N, 0) == 0  # one launch
    got = host(lut.linear(layer, dev(w.X)))
    idx = host(lut.encode(layer, dev(w.X)))
    assert near_tie_report(w, idx, oracle.encode(w.P, w.X)) <= 1
    Tf = oracle.build_table_f32(w.P, w.W)
    if dtype == "f32":
        check(got, Tf, None, idx, w.bias)
    else:
        q, s = oracle.quantize(Tf, 8 if dtype == "i8" else 4)
        check(got, q, s, idx, w.bias)
