"""GPU parity of the table construction (Eq. 3, Sec. 3.3 of arXiv 2302.03213) at the edges of its kernels' shares: four
columns per thread from 1024 columns on, one below or where rows cannot be moved 16 bytes at a time."""
import numpy as np
import pytest
import torch

import lutnn_workloads as wl
import oracle
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,K,V,M,strided", [
    (3, 16, 1, 1024, False), (2, 5, 2, 1028, False), (2, 16, 4, 1023, False), (2, 16, 8, 1024, True), (1, 8, 9, 1300, False),
    (2, 17, 16, 1032, False), (1, 33, 32, 4100, False), (3, 16, 3, 1024, False), (2, 16, 16, 4096, False), (5, 7, 9, 63, False),
    # a run-time V: 16 sums a thread, blocks of centroids that are not full
    (2, 33, 12, 100, False), (1, 16, 64, 1000, True), (3, 5, 6, 70, False), (1, 17, 5, 65, False),
])
def test_table_shares(C, K, V, M, strided):
    import paper_2302_03213_amd as lut
    w = wl.make_layer("t", 1, C, K, V, M, "i8", seed=C + K + V + M)
    W = dev(w.W)
    if strided:  # a row stride that is no multiple of four floats
        wide = torch.zeros((C * V, M + 3), dtype=torch.float32, device="cuda")
        wide[:, :M] = W
        W = wide[:, :M]
    Tf = oracle.build_table_f32(w.P, w.W)
    q, s = oracle.quantize_i8(Tf)
    layer = lut.build_table(dev(w.P), W, lut.TABLE_I8)
    np.testing.assert_array_equal(host(layer.table), q)
    assert host(layer.scale)[0] == np.float32(s)
    packed = host(layer.packed).reshape(C, (K + 15) // 16, -1, 16)
    for c in range(C):  # [c][block of 16 centroids][column][centroid], zero outside K and M
        full = np.zeros((packed.shape[1] * 16, packed.shape[2]), np.int8)
        full[:K, :M] = q[c]
        np.testing.assert_array_equal(packed[c], full.reshape(packed.shape[1], 16, -1).transpose(0, 2, 1))
    np.testing.assert_array_equal(host(lut.build_table(dev(w.P), W, lut.TABLE_F32).table), Tf)
    # scale and table of a layer that is all zero, and INT4 with and without the packed copy
    zero = lut.build_table(dev(w.P) * 0, W, lut.TABLE_I8)
    assert host(zero.scale)[0] == 1.0 and not host(zero.table).any()
    scales = [host(lut.build_table(dev(w.P), W, lut.TABLE_I4, packed=p).scale)[0] for p in (True, False)]
    assert scales == [np.float32(np.abs(Tf).max() / np.float32(7))] * 2


@pytest.mark.parametrize("C,K,V,M", [(1, 2, 3, (1 << 24) - 512), (1, 3, 2, 4194305), (1, 2, 9, 4194239), (2, 2, 9, 4194241)])
def test_widest_tables(C, K, V, M):
    """One column per thread, at widths where workgroups of 64 would not fit the grid's second dimension."""
    import paper_2302_03213_amd as lut
    gen = torch.Generator(device="cuda").manual_seed(M)
    P = torch.randn(C, K, V, generator=gen, device="cuda")
    W = torch.randn(C * V, M, generator=gen, device="cuda")
    f32 = lut.build_table(P, W, lut.TABLE_F32).table
    for part in (slice(0, 1000), slice(M - 1000, M)):
        np.testing.assert_array_equal(host(f32[:, :, part]), oracle.build_table_f32(host(P), host(W[:, part].contiguous())))
    layer = lut.build_table(P, W, lut.TABLE_I8)
    q, s = oracle.quantize_i8(host(f32))
    assert host(layer.scale)[0] == np.float32(s)
    np.testing.assert_array_equal(host(layer.table), q)
    packed = host(layer.packed).reshape(C, -1, 16)
    np.testing.assert_array_equal(packed[:, :M, :K], q.transpose(0, 2, 1))
    assert not packed[:, :, K:].any() and not packed[:, M:].any()
