"""The cell table where a pair lies on the edge between two cells, in the strips that the outermost cells reach to, and at their
end: device codebook training with the table against the distances to all points, the same points bit for bit."""
import ctypes as C
import sys

import numpy as np
import pytest
import torch

from paper_2605_26339_amd import qamw

pytestmark = pytest.mark.gpu


def _edges(cells, half):
    """Where s^2 (3 - 2s) of s = x / 2R + 1/2, R = 17/16 half, passes (i - 1/2) / (cells - 1); and the strips' ends, 5/4 R."""
    t = (np.arange(1, cells) - 0.5) / (cells - 1)
    s = 0.5 - np.sin(np.arcsin(1.0 - 2.0 * t) / 3.0)
    return np.concatenate([(2.0 * s - 1.0) * 1.0625 * half, [-1.328125 * half, -1.0625 * half, 1.0625 * half, 1.328125 * half]]).astype(np.float32)


# the smallest codebook that has a table, the largest of 64 x 64 cells, and the two of 128 x 128
@pytest.mark.parametrize("bits,cells", [(6, 64), (9, 64), (10, 128), (11, 128)])
@pytest.mark.parametrize("scale", [1.0, 0.25])
def test_samples_on_the_edges_of_cells(bits, cells, scale):
    print(f"[cells edges] B={bits} x {scale}", flush=True)
    sys.stdout.flush()
    init = torch.from_numpy(qamw.train_codebook(bits, 1 << 16, max_iters=20)[0]).cuda() * scale
    rng = np.random.default_rng(bits)
    e = _edges(cells, 4.0 * scale)
    near = np.concatenate([np.nextafter(e, np.float32(9e9)), e, np.nextafter(e, np.float32(-9e9)), e * np.float32(1 + 3e-6), e * np.float32(1 - 3e-6)])
    other = (rng.standard_normal((near.size, 24)) * 1.3 * scale).astype(np.float32)
    x = np.stack([np.broadcast_to(near[:, None], other.shape), other], -1).reshape(-1, 2)
    corners = near[rng.integers(0, near.size, (20000, 2))]
    strips = (rng.uniform(-6.0, 6.0, (20000, 2)) * scale).astype(np.float32)
    x = np.concatenate([x, x[:, ::-1], corners, strips]).astype(np.float32)
    samples = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    _same_points(samples, init, bits)


def _same_points(samples, init, bits):
    """Two iterations with the table and with the least scratch, which computes all distances."""
    got, _, it = qamw.lloyd_device(samples, init, bits, max_iters=2, tol=0.0)
    want, least = init.clone(), torch.empty((1 << bits) * 40 + 64, dtype=torch.uint8, device="cuda")
    assert qamw.lib().qamw_lloyd_device(C.c_void_p(samples.data_ptr()), samples.shape[0], bits, C.c_void_p(want.data_ptr()), 2, 0.0,
                                        C.c_void_p(least.data_ptr()), least.numel(), None, None, None) == qamw.OK
    assert it == 2 and torch.equal(got, want)


@pytest.mark.parametrize("bits", [6, 11])
def test_samples_that_are_no_points(bits):
    """One coordinate infinite or a NaN, the other anywhere in the table's range or on its edge."""
    print(f"[cells edges] not finite, B={bits}", flush=True)
    init = torch.from_numpy(qamw.train_codebook(bits, 1 << 16, max_iters=20)[0]).cuda()
    good = torch.randn(20000, 2, generator=torch.Generator().manual_seed(bits))
    good[::7] *= 1.6
    for bad in (float("nan"), -float("nan"), float("inf"), -float("inf")):
        for coordinate in (0, 1):
            samples = good.clone()
            samples[::5, coordinate] = bad
            _same_points(samples.cuda(), init, bits)


def _nearest_fields(x, cb):
    """The lowest index of the least fp32 distance (fma(e1, e1, e0 * e0)); one that is a NaN is never the least."""
    best = []
    for part in x.reshape(-1, 2).split(4096):
        e = part[:, None, :] - cb[None]
        d = (e[..., 1].double() ** 2 + (e[..., 0] * e[..., 0]).double()).float()
        best.append(torch.where(d.isnan(), torch.inf, d).argmin(1))
    return torch.cat(best).view(x.shape[:-1])


def _fields(packed, bits, n):
    stream = (packed[..., None] >> torch.arange(8, device="cuda", dtype=torch.uint8)) & 1
    return (stream.reshape(packed.shape[0], -1)[:, : n * bits].view(packed.shape[0], n, bits).long() << torch.arange(bits, device="cuda")).sum(-1)


# 4200 x 4: the table in LDS; at 11 bits also 40 x 4, its records from memory
@pytest.mark.parametrize("bits,rows", [(4, 4200), (9, 4200), (10, 4200), (11, 4200), (11, 40)])
def test_codewords_that_are_no_points(bits, rows):
    """A codeword with a NaN, of either sign and in either coordinate, is nearest to no pair: every cell lists it."""
    print(f"[cells edges] codewords not finite, B={bits} rows {rows}", flush=True)
    good = torch.from_numpy(qamw.train_codebook(bits, 1 << 15, max_iters=20)[0]).cuda()
    W = torch.randn(20, 4096, device="cuda", generator=torch.Generator("cuda").manual_seed(bits))
    pairs, _ = qamw.normalised_pairs(W, 64)
    for bad in (float("nan"), -float("nan")):
        for coordinate in (0, 1):
            cb = good.clone()
            cb[(1 << bits) - 2, coordinate] = torch.tensor(bad).cuda()
            packed, _ = qamw.encode(W.repeat(rows // 20, 1), cb, bits, 64)
            torch.cuda.synchronize()
            got, want = _fields(packed, bits, 2048), _nearest_fields(pairs, cb)
            assert torch.equal(got.view(-1, 20, 2048), want.expand(rows // 20, -1, -1)), (bad, coordinate)


# the encoder's three tables
@pytest.mark.parametrize("bits,cells", [(9, 64), (10, 96), (11, 128)])
@pytest.mark.parametrize("scale", [1.0, 0.25])
def test_pairs_on_the_edges_of_cells(bits, cells, scale):
    """Pairs +-(1, r) g and +-(r, 1) g: weights so small beside the row's first that its norm is 1, gains on the edges and beside them."""
    print(f"[cells edges] pairs, B={bits} x {scale}", flush=True)
    cb = torch.from_numpy(qamw.train_codebook(bits, 1 << 16, max_iters=20)[0]).cuda() * scale
    rng = np.random.default_rng(bits)
    e = _edges(cells, 4.0 * scale)
    e = e[e > 0]
    inverse = (1.0 / (e.astype(np.float64) * 2.0 ** 23)).astype(np.float32)
    sigma = np.concatenate([inverse, np.nextafter(inverse, np.float32(0)), np.nextafter(inverse, np.float32(1)), inverse * np.float32(1 + 3e-6),
                            inverse * np.float32(1 - 3e-6)])
    d_in = 4096
    r = rng.integers(-1200, 1201, 42) / 1024.0
    r[::6] *= 4
    a, b = (1 + r) / 2, (1 - r) / 2
    b[::2] *= -1                                                # a + b and a - b the other way round
    W = np.zeros((42, d_in))
    W[:, 2::64], W[:, 3::64] = a[:, None] * 2.0 ** -20, b[:, None] * 2.0 ** -20
    W[:, :64] = 0
    W[:, 0] = 1.0
    W = torch.from_numpy(W.astype(np.float32)).cuda()
    sg = torch.from_numpy(np.resize(sigma, d_in // 2)).cuda()
    x, _ = qamw.normalised_pairs(W, 64, pair_sigma=sg)
    own = x[:, 32:]
    assert torch.isin(own.abs(), torch.from_numpy(e).cuda()).any(-1).float().mean() > 0.05
    packed, _ = qamw.encode(W.repeat(100, 1), cb, bits, 64, pair_sigma=sg)
    torch.cuda.synchronize()
    assert torch.equal(_fields(packed, bits, d_in // 2).view(100, 42, -1), _nearest_fields(x, cb).expand(100, -1, -1))
