"""GPU parity of the unquantised lookup on the matrix cores (arXiv 2302.03213, Eq. 4) at the edges of its tiles and stages,
and with table entries whose parts need care.  Exact 64-bit sums: the error of C terms stays within C half ulps of the sum
of their magnitudes, as an fp32 chain's does."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lut():
    import paper_2302_03213_amd as lut_mod
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return lut_mod


def run(lut, T, idx, bias, offset=0, form="matrix"):
    C, K, M = T.shape
    flat = torch.empty(T.size + offset, device="cuda")
    flat[offset:] = torch.from_numpy(T.reshape(-1))
    layer = lut.LutLayer(torch.zeros((C, K, 4), device="cuda"), flat[offset:].view(T.shape), lut.TABLE_F32, M, bias=dev(bias))
    N = idx.shape[0]
    i8 = torch.empty(idx.size + offset, dtype=torch.uint8, device="cuda")
    i8[offset:] = torch.from_numpy(idx.reshape(-1))
    out = torch.full((N, M + 3), -3.5, device="cuda")
    with lut.tunables(LUTNN_LOOKUP_F32=form):
        lut.lookup(layer, i8[offset:].view(idx.shape), "lds", out=out[:, :M])
    assert (host(out[:, M:]) == -3.5).all()
    return host(out[:, :M])


def sums(T, idx, bias):
    """The 64-bit sums, their terms' magnitudes, and the fp32 chain."""
    total = np.zeros((idx.shape[0], T.shape[2]))
    size = np.zeros_like(total)
    chain = np.zeros(total.shape, np.float32)
    with np.errstate(over="ignore", invalid="ignore"):
        for c in range(T.shape[0]):
            term = T[c, np.minimum(idx[:, c], T.shape[1] - 1)]
            total += term
            size += np.abs(term.astype(np.float64))
            chain += term
        return (total, size, chain) if bias is None else (total + bias, size + np.abs(bias), chain + bias)


# stages of four codebooks with one, two and three left, rows past a tile and fewer than one, widths that end in a tile, one
# column tile as a convolution has
SHAPES = [(3001, 7, 16, 3001), (3100, 9, 8, 3017), (3000, 10, 16, 3072), (1500, 64, 16, 2049), (1100, 130, 7, 2190),
          (2000, 513, 16, 1200), (4097, 32, 16, 1100), (1, 16, 16, 1), (63, 17, 16, 65), (257, 18, 5, 63), (1000, 19, 16, 130),
          (255, 33, 1, 4), (20000, 64, 16, 64), (9000, 16, 8, 32), (300, 512, 16, 200)]


@pytest.mark.parametrize("N,C,K,M", SHAPES)
def test_edges(lut, N, C, K, M):
    rng = np.random.default_rng(N + C)
    T = rng.standard_normal((C, K, M)).astype(np.float32)
    bias = rng.standard_normal(M).astype(np.float32) if C != 64 else None
    idx = rng.integers(0, K + (C == 9), (N, C)).astype(np.uint8)  # with one past the table, which is its last row
    total, size, chain = sums(T, idx, bias)
    got = run(lut, T, idx, bias, offset=C % 2)
    assert (np.abs(got - total) <= (C + 1) * 2.0 ** -24 * size).all()
    if C >= 32:  # no less exact than the chain
        assert np.linalg.norm(got - total) <= 1.02 * np.linalg.norm(chain - total)


# shapes that the matrix form would be fast on, entries that its sums would lose bits of
@pytest.mark.parametrize("N,C,M", [(8192, 7, 3072), (5000, 4, 3000), (9000, 15, 1030)])
def test_few_codebooks_are_summed_as_an_fp32_chain(lut, N, C, M):
    rng = np.random.default_rng(C)
    T = (rng.standard_normal((C, 16, M)) * 2.0 ** rng.integers(-20, 20, (C, 16, M))).astype(np.float32)
    idx = rng.integers(0, 16, (N, C)).astype(np.uint8)
    for form in ("matrix", None):
        np.testing.assert_array_equal(run(lut, T, idx, None, form=form), sums(T, idx, None)[2])


@pytest.mark.parametrize("C", [16, 17, 22, 31, 64])
def test_entries_of_all_sizes_are_summed_no_less_exactly(lut, C):
    """Relative to the sum of the terms' magnitudes, over a million sums (the ratio itself: 0.93 at 16 codebooks)."""
    rng = np.random.default_rng(C)
    T = (rng.standard_normal((C, 16, 512)) * 2.0 ** rng.integers(-20, 20, (C, 16, 512))).astype(np.float32)
    idx = rng.integers(0, 16, (2048, C)).astype(np.uint8)
    total, size, chain = sums(T, idx, None)
    got = run(lut, T, idx, None)
    assert np.linalg.norm((got - total) / size) <= np.linalg.norm((chain - total) / size)


@pytest.mark.parametrize("scale", [1e-38, 1e-30, 1e28])
def test_small_and_large_entries(lut, scale):
    rng = np.random.default_rng(1)
    T = (rng.standard_normal((33, 16, 1500)) * scale).astype(np.float32)
    idx = rng.integers(0, 16, (2500, 33)).astype(np.uint8)
    total, size, _ = sums(T, idx, None)
    assert (np.abs(run(lut, T, idx, None) - total) <= 34 * (2.0 ** -24 * size + 2.0 ** -149)).all()


def test_entries_that_are_not_finite_and_overflow(lut):
    rng = np.random.default_rng(2)
    T = rng.standard_normal((40, 16, 1500)).astype(np.float32)
    T[3, 5, 7], T[4, 2, 70], T[11, 15, 199], T[12, 0, 100], T[13, 0, 100] = np.inf, -np.inf, np.nan, 3e38, 3e38
    idx = rng.integers(0, 16, (2500, 40)).astype(np.uint8)
    bias = rng.standard_normal(1500).astype(np.float32)
    total, size, chain = sums(T, idx, bias)
    got = run(lut, T, idx, bias)
    fine = np.isfinite(chain)
    np.testing.assert_array_equal(got[~fine], chain[~fine])
    assert (np.abs(got - total)[fine] <= 41 * 2.0 ** -24 * size[fine]).all()


def test_the_switch_pins_the_form(lut):
    """The three forms add in different orders; both chains give the same sums.  A form the shape cannot take is ignored."""
    rng = np.random.default_rng(3)
    T = rng.standard_normal((40, 16, 700)).astype(np.float32)
    idx = rng.integers(0, 16, (2500, 40)).astype(np.uint8)
    chain = sums(T, idx, None)[2]
    np.testing.assert_array_equal(run(lut, T, idx, None, form="rows"), chain)
    np.testing.assert_array_equal(run(lut, T, idx, None, form="gather"), chain)
    assert (run(lut, T, idx, None, form="matrix") != chain).any()
    T, idx = rng.standard_normal((5, 200, 3)).astype(np.float32), rng.integers(0, 200, (300, 5)).astype(np.uint8)
    for form in ("rows", "gather", "matrix"):
        np.testing.assert_array_equal(run(lut, T, idx, None, form=form), sums(T, idx, None)[2])
    with pytest.raises(lut.LutnnError):
        lut.set_tunable("LUTNN_LOOKUP_F32", "staged")
