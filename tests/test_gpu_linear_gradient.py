"""lutnn_linear_gradient (matmul_split.hip): Z = G . W^T from bf16 parts, against 64-bit sums.

Bar: |Z - ref| <= 2^-20 sum_m |G W| elementwise.  A product loses at most 3 * 2^-22 of itself to the parts left out (the
middle and low parts are below 2^-7 and 2^-15 of the value).  Each slice of 32 m ends in a few cut fp32 sums (2^-23 of the
slice's magnitude each, two of them at full size) and one rounded addition to the running sum (2^-24): together below
2^-20 of the sum of magnitudes.  Observed: 2-norm error 8e-8 to 1.6e-7 of the result (library fp32: 1.4e-7 to 1e-6)."""
import pytest
import torch

import paper_2302_03213_amd as lut

pytestmark = pytest.mark.gpu


def operands(N, D, M, ldg=0, ldw=0, shift=0, seed=0):
    gen = torch.Generator(device="cuda").manual_seed(seed + N * 7 + D * 3 + M)
    def one(rows, ld):
        flat = torch.full((rows * ld + shift,), float("nan"), device="cuda")  # what lies between the rows is not read
        view = flat[shift:].view(rows, ld)[:, :M]
        view.copy_(torch.randn(rows, M, generator=gen, device="cuda"))
        return view
    return one(N, max(ldg, M)), one(D, max(ldw, M))


def check(G, W, Z):
    ref = G.double() @ W.double().t()
    bound = G.double().abs() @ W.double().abs().t() * 2.0 ** -20
    assert bool(((Z.double() - ref).abs() <= bound).all())


def error(G, W, Z):
    ref = G.double() @ W.double().t()
    return float((Z.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("N,D,M,ldg,ldw,shift", [
    (1, 1, 1, 0, 0, 0), (64, 64, 64, 0, 0, 0), (65, 63, 4, 0, 0, 0), (33, 97, 65, 0, 0, 0), (200, 130, 1001, 0, 0, 0),
    (256, 256, 96, 100, 128, 0),             # strides; the second group's last slice is empty
    (300, 77, 64, 0, 0, 1),                  # not 16-byte aligned
    (4096, 768, 160, 0, 0, 0),               # 128 x 96 tiles
    (8192, 2048, 36, 0, 0, 0), (4090, 1999, 68, 0, 0, 0),  # 128 x 128, whole and not
    (1100, 1030, 132, 0, 0, 0), (600, 1800, 404, 0, 0, 0),  # 64 x 64 and 96 x 64
])
def test_against_64_bit_sums(N, D, M, ldg, ldw, shift):
    G, W = operands(N, D, M, ldg, ldw, shift)
    out = torch.full((N, D + 5), 7.0, device="cuda")
    check(G, W, lut.linear_gradient(G, W))
    check(G, W, lut.linear_gradient(G, W, out=out[:, :D]))
    assert bool((out[:, D:] == 7.0).all())


@pytest.mark.parametrize("scale_g,scale_w", [(1e-30, 1e20), (1e30, 1e-20), (3e37, 1e-3), (1e-25, 1.0)])
def test_the_range_of_the_exponent(scale_g, scale_w):
    G, W = operands(200, 100, 200)
    check(G * scale_g, W * scale_w, lut.linear_gradient(G * scale_g, W * scale_w))


def test_error_is_no_larger_than_the_librarys():
    for N, D, M, same_sign in [(4096, 768, 3072, False), (4096, 256, 256, False), (8192, 96, 64, False), (2048, 512, 2048, True)]:
        G, W = operands(N, D, M)
        if same_sign:
            G, W = G.abs(), W.abs()
        assert error(G, W, lut.linear_gradient(G, W)) <= error(G, W, G @ W.t())


def test_values_that_are_not_finite_stay_in_their_row_and_column():
    G, W = operands(300, 200, 128)
    G[17, 5], G[200, 100], W[33, 7] = float("inf"), float("nan"), float("-inf")
    Z = lut.linear_gradient(G, W)
    bad = ~torch.isfinite(Z)
    expect = torch.zeros_like(bad)
    expect[17], expect[200], expect[:, 33] = True, True, True
    assert torch.equal(bad, expect)


def test_refusals():
    G, W = operands(8, 8, 8)
    Z = torch.empty(8, 8, device="cuda")
    call = lut.LIB.lutnn_linear_gradient
    p = lambda t: t.data_ptr()  # noqa: E731
    assert call(p(G), 0, 8, p(W), 8, 8, 8, p(Z), 8, None) == 0
    for args in [(None, 8, 8, p(W), 8, 8, 8, p(Z), 8), (p(G), 8, 7, p(W), 8, 8, 8, p(Z), 8), (p(G), 8, 8, p(W), 8, 8, 8, p(Z), 7),
                 (p(G), 8, 8, p(W), 8, 0, 8, p(Z), 8), (p(G), 8, 8, p(W), (1 << 20) + 1, 8, 8, p(Z), 8),
                 (p(G) + 2, 8, 8, p(W), 8, 8, 8, p(Z), 8)]:
        assert call(*args, None) != 0
    assert not lut.LIB.lutnn_linear_gradient_preferred(p(G) + 4, 4096, 3072, p(W), 3072, 768, 3072)


@pytest.mark.parametrize("M", [1, 2, 4, 8, 12, 16, 20, 32, 48])
def test_short_sums_are_no_less_exact_than_an_fp32_chain(M):
    """What training forms Z with: for a linear layer where linear_gradient is preferred, for a convolution always.  With all
    centroids equal the soft encoding is 1/16 each and no other term is left: dL/dP of a single pixel is Z / 16."""
    def chain(G, W):
        sums = torch.zeros(G.shape[0], W.shape[0], device="cuda")
        for m in range(M):  # one rounding a term: the product of two fp32 values is exact in 64 bits
            sums = (sums.double() + G[:, m:m + 1].double() * W[:, m].double()).float()
        return sums
    G, W = operands(8192, 1024, M)
    if lut.linear_gradient_preferred(G, W):
        assert error(G, W, lut.linear_gradient(G, W)) <= error(G, W, chain(G, W))
    C, pixels = 1000, 200
    G, W = operands(pixels, 9 * C, M)
    layer = lut.LutLayer(torch.zeros(C, 16, 9, device="cuda"), None, lut.TABLE_F32, M)
    image = torch.ones(1, C, 3, 3, device="cuda")
    Z = [lut.softpq_backward_conv2d(layer, 1.0, image, W, G[n].reshape(1, M, 1, 1), 3)[0][:, 7].reshape(-1) * 16
         for n in range(pixels)]
    assert error(G, W, torch.stack(Z)) <= error(G, W, chain(G, W))


def test_infinite_values_and_overflow_as_in_an_fp32_product():
    """All terms of a sum have one sign: whether it is finite does not hang on the order of the sum."""
    G, W = operands(300, 200, 128)
    G, W = G.abs() + 0.1, W.abs() + 0.1
    W[50:60] *= -1
    G[17, 5], G[200, 100], W[33, 7], W[34, 9] = float("inf"), float("nan"), float("-inf"), 0.0
    G[34], W[34, 100] = G[34] * 3e38, 1.0  # sums beyond the largest value
    W[40, 5] = 0.0  # times an infinite value
    assert torch.equal(torch.isfinite(lut.linear_gradient(G, W)), torch.isfinite(G @ W.t()))
    bad = ~torch.isfinite(G @ W.t())
    torch.testing.assert_close(lut.linear_gradient(G, W)[bad], (G @ W.t())[bad], rtol=0, atol=0, equal_nan=True)
    assert bool((lut.linear_gradient(G, W)[17, 50:60] == float("-inf")).all())


@pytest.mark.parametrize("scale_g,scale_w", [(1e-34, 1.0), (1e-36, 1.0), (1e-37, 1e20), (1e-20, 1e-16), (1.0, 1e-36), (1e20, 1e-36),
                                             (1e19, 1e10), (1e37, 1e-36)])
def test_small_and_large_values_keep_their_bits(scale_g, scale_w):
    """Both kernels, at the ends of the range: the parts of small values, the fp32 chains of large ones (whose error is the
    library's but for the spread of an estimate)."""
    G, W = operands(300, 200, 128)
    G, W = G * scale_g, W * scale_w
    assert error(G, W, lut.linear_gradient(G, W)) <= 1.02 * error(G, W, G @ W.t())
    C = 1000
    G, W = operands(1, 9 * C, 128)
    G, W = G * scale_g, W * scale_w
    layer = lut.LutLayer(torch.zeros(C, 16, 9, device="cuda"), None, lut.TABLE_F32, 128)  # equal centroids: dL/dP = Z / 16
    dP, _, _ = lut.softpq_backward_conv2d(layer, 1.0, torch.ones(1, C, 3, 3, device="cuda"), W, G.reshape(1, 128, 1, 1), 3)
    assert error(G, W, dP[:, 7].reshape(1, -1) * 16) <= 2.5e-7  # 9e-8 from parts, 2e-7 from an fp32 chain of 128 terms
