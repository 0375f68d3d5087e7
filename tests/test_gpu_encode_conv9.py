"""The matrix-core filter of the 3x3 convolution's encoder (encode_conv9.hip): indices equal to the oracle's on the unfolded
rows, including where the filter must step aside - ties, near-ties, values beyond fp16's range, zeros, values that
are not finite.  Launches larger than a workgroup per CU, where the filter is taken."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


def unfolded(inp, kernel, stride, pad):
    cols = torch.nn.functional.unfold(torch.from_numpy(inp), kernel, padding=pad, stride=stride)
    return np.ascontiguousarray(cols.permute(0, 2, 1).reshape(-1, cols.shape[1]).numpy())


def tiles_per_chunk(rows_an_image, B, C, K):
    """Tiles of 64 pixels that a workgroup of the filter goes through, as encode_conv9_filter_chunks deals them out; fails
    where that rule takes the direct search."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    tiles, columns = B * -(-rows_an_image // 64), -(-C // 16)
    assert tiles * columns > units if K == 16 else tiles * columns >= 4 * units, "these sizes take the direct search"
    return -(-tiles // min(max(4 * units // columns, 1), tiles))


def check(P, inp, kernel, stride, pad, finite=True, tiles=1):
    import paper_2302_03213_amd as lut
    layer = lut.LutLayer(dev(P), None, lut.TABLE_F32, 8)
    got = host(lut.encode_conv2d(layer, dev(inp), kernel, stride, pad))
    X = unfolded(inp, kernel, stride, pad)
    assert tiles_per_chunk(X.shape[0] // inp.shape[0], *inp.shape[:2], P.shape[1]) == tiles
    if finite:
        np.testing.assert_array_equal(got, oracle.encode(P, X))
    else:  # what is not finite is the direct kernel's to decide: the same as on materialised rows
        np.testing.assert_array_equal(got, host(lut.encode(layer, dev(X))))
        assert got.max() < P.shape[1]
    return got


@pytest.mark.parametrize("B,C,H,W,kernel,stride,pad,K,tiles", [
    (6, 64, 56, 56, 3, 1, 1, 16, 2),      # five pieces of band, chunks of one and two tiles
    (9, 37, 28, 28, 3, 1, 1, 16, 1),      # three pieces; codebooks that fill neither a wavefront nor a dword
    (4, 18, 100, 90, 3, 1, 1, 8, 2),      # eight pieces, K = 8; the band's width changes from tile to tile of a chunk
    (80, 64, 7, 7, 3, 1, 1, 16, 1),       # images smaller than a tile
    (600, 64, 7, 7, 3, 1, 1, 16, 3),      # a chunk goes from image to image
    (9, 66, 57, 41, 3, 2, 1, 16, 1),      # stride 2
    (30, 66, 57, 41, 3, 2, 1, 16, 2),
    (30, 50, 9, 120, 3, 1, 0, 16, 2),     # tiles within one row and across two: the band's width changes
    (40, 30, 21, 13, (1, 9), 1, (0, 4), 16, 1),  # nine taps in a row
])
def test_indices_equal_the_oracles(B, C, H, W, kernel, stride, pad, K, tiles):
    rng = np.random.default_rng(B * C)
    inp = rng.standard_normal((B, C, H, W)).astype(np.float32)
    inp[rng.random(inp.shape) < 0.01] *= 10
    check(rng.standard_normal((C, K, 9)).astype(np.float32), inp, kernel, stride, pad, tiles=tiles)


def test_doubtful_rows():
    rng = np.random.default_rng(5)
    B, C = 8, 48
    P = rng.standard_normal((C, 16, 9)).astype(np.float32)
    P[0, 9] = P[0, 3]                       # equal centroids: the lower index
    P[1, 12] = np.nextafter(P[1, 4], 9)     # one unit in the last place apart
    P[2] = np.round(P[2])                   # small integers: exact ties between different centroids
    P[3] = 0                                # all equal
    P[4] *= 1e-5                            # too small for the parts
    P[5] *= 1e4                             # too large
    inp = rng.standard_normal((B, C, 30, 30)).astype(np.float32)
    inp[:, 2] = np.round(inp[:, 2])
    inp[:, 4] *= 1e-5
    inp[:, 5] *= 1e4
    inp[:, 6] *= 1e30                       # activations beyond fp16 against ordinary centroids
    inp[:, 7] *= 1e-30
    inp[:, 8] = np.maximum(inp[:, 8], 0)
    inp[0, 9] = 0
    inp[:, 10, ::7] *= 30000
    got = check(P, inp, 3, 1, 1)
    assert not (got[:, 0] == 9).any() and not got[:, 3].any()


@pytest.mark.parametrize("kind", ["small", "equal centroids", "nearly equal centroids", "no image in half the tiles", "all zero"])
@pytest.mark.parametrize("K", [8, 16])
def test_whole_tiles_without_the_filter(kind, K):
    """Codebooks outside its range, and tiles with more doubtful rows than are searched one by one: 64 rows at once, and the
    rest of the chunk, too; 37 codebooks end within a wavefront's four."""
    rng = np.random.default_rng(K)
    P = rng.standard_normal((37, K, 9)).astype(np.float32)
    inp = rng.standard_normal((120, 37, 30, 30)).astype(np.float32)
    if kind == "small":
        P, inp = P * np.float32(1e-5), inp * np.float32(1e-5)
    elif kind == "equal centroids":
        P[:, K // 2:] = P[:, :K // 2]
    elif kind == "nearly equal centroids":
        P[::2, K // 2:] = P[::2, :K // 2] * np.float32(1 + 1e-6)
    elif kind == "no image in half the tiles":
        P[::2, 3], P[1::2, 5] = -P[::2, 1], -P[1::2, 2]  # as far from zero as each other, and near it
        P[:, (1, 2, 3, 5)] *= np.float32(0.25)
        inp[:, :, 10:20] = 0
    else:
        P *= 0
    got = check(P, inp, 3, 1, 1, tiles=6)
    if kind == "equal centroids":
        assert got.max() < K // 2


def test_values_that_are_not_finite():
    rng = np.random.default_rng(6)
    inp = rng.standard_normal((40, 32, 30, 30)).astype(np.float32)
    inp[rng.random(inp.shape) < 0.01] = np.nan
    inp[rng.random(inp.shape) < 0.01] = np.inf
    inp[rng.random(inp.shape) < 0.01] = -np.inf
    check(rng.standard_normal((32, 16, 9)).astype(np.float32), inp, 3, 1, 1, finite=False, tiles=2)


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("k", [0, 5, 15])
def test_centroids_that_are_not_finite(value, k):
    """A distance that is not a number loses against any other but in centroid 0, which nothing is below then."""
    rng = np.random.default_rng(7)
    P = rng.standard_normal((32, 16, 9)).astype(np.float32)
    P[::3, k, 4] = value
    inp = rng.standard_normal((40, 32, 30, 30)).astype(np.float32)
    inp[rng.random(inp.shape) < 0.01] = np.inf
    inp[rng.random(inp.shape) < 0.01] = np.nan
    check(P, inp, 3, 1, 1, finite=False, tiles=2)


def test_channels_of_all_images_beyond_31_bits():
    """B * Cin above 2^31, with images of one pixel: the last images equal the oracle's indices on their rows."""
    B, C, last = (1 << 23) + 70, 256, 64
    P = np.random.default_rng(8).standard_normal((C, 16, 9)).astype(np.float32)
    inp = torch.randn(B, C, 1, 1, generator=torch.Generator(device="cuda").manual_seed(8), device="cuda")
    import paper_2302_03213_amd as lut
    got = lut.encode_conv2d(lut.LutLayer(dev(P), None, lut.TABLE_F32, 8), inp, 3, 1, 1)
    for part in (slice(0, last), slice(B - last, B)):
        np.testing.assert_array_equal(host(got[part]), oracle.encode(P, unfolded(host(inp[part]), 3, 1, 1)))
    del got, inp
    torch.cuda.empty_cache()
