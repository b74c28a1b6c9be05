"""Device codebook training with a cell table per iteration (64 to 2048 points, the workspace the library asks for) against
the same call with the least workspace, which computes the distances to all points: the same points, bit for bit."""
import ctypes as C
import sys

import numpy as np
import pytest
import torch

from paper_2605_26339_amd import qamw

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _both(x, init, bits, iters, tol):
    L = qamw.lib()
    cb, mse, it = qamw.lloyd_device(x, init, bits, max_iters=iters, tol=tol)
    want, w_mse, w_it = init.clone(), C.c_double(), C.c_int()
    ws = torch.empty((1 << bits) * 40 + 64, dtype=torch.uint8, device="cuda")
    assert L.qamw_lloyd_device(C.c_void_p(x.data_ptr()), x.shape[0], bits, C.c_void_p(want.data_ptr()), iters, tol,
                               C.c_void_p(ws.data_ptr()), ws.numel(), C.byref(w_mse), C.byref(w_it), None) == qamw.OK
    assert L.qamw_lloyd_device(C.c_void_p(x.data_ptr()), x.shape[0], bits, C.c_void_p(want.clone().data_ptr()), iters, tol,
                               C.c_void_p(ws.data_ptr()), ws.numel() - 1, None, None, None) == qamw.ERR_INVALID_ARG
    assert torch.equal(cb, want) and it == w_it.value
    # the error: fp64 sums of 32-bit distances, rounded to 2^-30 once per wave, of which there are n / 64 at most
    assert abs(mse - w_mse.value) <= 1e-12 * w_mse.value + 2.0 ** -31
    return it


# sample counts around a wave, a workgroup's share and the largest grid; one to several looks of the host at the stop
@pytest.mark.parametrize("bits,n,iters,tol", [(6, 64, 3, 0.0), (6, 1 << 19, 5, 0.0), (7, 2047, 40, 1e-3), (8, 2049, 16, 0.0),
                                              (9, 70001, 60, 1e-4), (10, 300000, 17, 0.0), (11, 2048, 2, 0.0), (11, (1 << 20) + 77, 4, 0.0)])
def test_table_gives_the_points_of_the_whole_search(bits, n, iters, tol):
    say(f"[lloyd cells] B={bits} n={n} iterations<={iters} tol={tol}")
    g = torch.Generator("cuda").manual_seed(n)
    x = torch.randn(n, 2, device="cuda", generator=g)
    init = torch.randn(1 << bits, 2, device="cuda", generator=g)
    it = _both(x, init, bits, iters, tol)
    assert it == iters if tol == 0.0 else 1 < it <= iters


@pytest.mark.parametrize("kind", ["far_samples", "one_cell", "duplicate_points", "far_points"])
def test_samples_and_points_that_strain_the_table(kind):
    say(f"[lloyd cells] {kind}")
    bits, n = 8, 5000
    rng = np.random.default_rng(3)
    x = rng.standard_normal((n, 2)).astype(np.float32)
    c = rng.standard_normal((1 << bits, 2)).astype(np.float32)
    if kind == "far_samples":
        x[::3] *= 300.0                                       # beyond the table, and beyond the sums' clamp
    elif kind == "one_cell":
        x, c = x * 1e-3, c * 1e-3                             # more points in a cell than a record lists
    elif kind == "duplicate_points":
        c[128:] = c[:128]                                     # the upper half never wins: empty cells keep their points
    else:
        c *= 1000.0
    _both(torch.from_numpy(x).cuda(), torch.from_numpy(c).cuda(), bits, 6, 0.0)
