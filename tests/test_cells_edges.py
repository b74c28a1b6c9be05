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
