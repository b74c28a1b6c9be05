"""Device codebook training, where the sums of all workgroups meet in one copy per iteration: the same points as the call with
the least workspace, bit for bit, with iterations that end just before, at and after the host looks (every 16), and with
any number of workgroups."""
import ctypes as C
import sys

import pytest
import torch

from paper_2605_26339_amd import qamw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,n,iters", [(6, 64, 1), (6, 5000, 15), (7, 5000, 16), (8, 5000, 17), (11, 9000, 32), (10, 5000, 33),
                                          (6, 1 << 20, 3), (6, (1 << 20) + 1, 3), (11, (1 << 20) - 1, 2)])
def test_one_copy_of_the_sums(bits, n, iters):
    print(f"[lloyd sums] B={bits} n={n} iterations={iters}", flush=True)
    sys.stdout.flush()
    g = torch.Generator("cuda").manual_seed(n + iters)
    x = torch.randn(n, 2, device="cuda", generator=g)
    init = torch.randn(1 << bits, 2, device="cuda", generator=g)
    least = torch.empty((1 << bits) * 40 + 64, dtype=torch.uint8, device="cuda")
    want, w_mse, w_it = init.clone(), C.c_double(), C.c_int()
    assert qamw.lib().qamw_lloyd_device(C.c_void_p(x.data_ptr()), n, bits, C.c_void_p(want.data_ptr()), iters, 0.0,
                                        C.c_void_p(least.data_ptr()), least.numel(), C.byref(w_mse), C.byref(w_it), None) == qamw.OK
    for _ in range(2):                                        # the second on memory that the first has used
        cb, mse, it = qamw.lloyd_device(x, init, bits, max_iters=iters, tol=0.0)
        assert torch.equal(cb, want) and it == w_it.value
        # the error: fp64 sums of 32-bit distances, rounded to 2^-30 once per wave, of which there are n / 64 and one at most
        assert abs(mse - w_mse.value) <= 1e-12 * w_mse.value + 2.0 ** -30


# workgroups of the assignment from half of the chip (128) on: as many as a pass of 4096 samples each needs, of 8192 with 2048
# points; on either side of both ends, and between
@pytest.mark.parametrize("bits,n", [(6, 128 * 4096 - 1), (6, 128 * 4096 + 1), (8, 700001), (10, 255 * 4096 + 1), (10, 256 * 4096 + 1),
                                    (11, 128 * 8192 + 1), (11, 1500001), (11, 256 * 8192 + 1), (7, 127 * 1024 + 1), (7, 129 * 1024)])
def test_any_number_of_workgroups(bits, n):
    test_one_copy_of_the_sums(bits, n, 3)
