"""The fused product for one activation row where no wave has a second step (a workgroup's slabs times its groups of eight rows are
at most its four waves), on either side of that line and in one launch with matrices beyond it: the bits of the kernel after a
rotation launch, and X times the decoder's fp32 output in fp64 (bar 1e-5 ||x|| ||w_i||, a hundred times the rounding of an fp32
sum over the row)."""
import sys

import numpy as np
import pytest
import torch

from paper_2605_26339_amd import qamw

pytestmark = pytest.mark.gpu


def _matrix(g, d_out, d_in, bits):
    pk = torch.randint(0, 256, (d_out, qamw.packed_row_bytes(d_in, bits)), dtype=torch.uint8, device="cuda", generator=g)
    return (pk, torch.rand(d_out, device="cuda", generator=g) + 0.5, torch.exp(0.5 * torch.randn(d_in, device="cuda", generator=g)),
            (torch.randint(0, 2, (d_in,), device="cuda", generator=g) * 2 - 1).to(torch.int8),
            (torch.rand(d_in // 2, device="cuda", generator=g) + 0.5) / np.sqrt(d_in))


@pytest.mark.parametrize("bits,block,xdtype", [(7, 64, torch.float32), (8, 256, torch.bfloat16), (11, 1024, torch.bfloat16), (11, 128, torch.float32)])
def test_one_step_a_wave(bits, block, xdtype):
    g = torch.Generator("cuda").manual_seed(bits)
    cb = torch.randn(1 << bits, 2, device="cuda", generator=g)
    # one slab: a step in one wave alone; four slabs or two groups of rows: one each; five slabs, four groups: two for some
    shapes = [(5, 1024), (2047, 4096), (4097, 2048), (33, 5120), (8200, 1024), (8200, 2048)]
    X = {d_in: torch.randn(1, d_in, device="cuda", generator=g).to(xdtype) for _, d_in in shapes}
    mats, alone = [], []
    for d_out, d_in in shapes:
        print(f"[matmul one step] {d_out}x{d_in} B={bits} b={block} {xdtype}", flush=True)
        sys.stdout.flush()
        pk, nr, s, sg, sigma = _matrix(g, d_out, d_in, bits)
        kw = dict(chan_scale=s, signs=sg, pair_sigma=sigma)
        Y = qamw.matmul(X[d_in], pk, nr, cb, bits, block, **kw)
        prev = qamw.set_kernel_path(1)                          # a rotation launch, then the product
        try:
            two = qamw.matmul(X[d_in], pk, nr, cb, bits, block, **kw)
            torch.cuda.synchronize()
        finally:
            qamw.set_kernel_path(prev)
        assert torch.equal(Y, two)
        W = qamw.decode(pk, nr, d_in, cb, bits, block, f32=True, **kw).double()
        bar = 1e-5 * X[d_in].double().norm(dim=1)[:, None] * W.norm(dim=1)[None, :] + 1e-30
        assert float(((Y.double() - X[d_in].double() @ W.t().contiguous()).abs() / bar).max()) <= 1.0
        mats.append((X[d_in], pk, nr, s, sg, sigma))
        alone.append(Y)
    for pick in ([0, 1], [1, 3], [2, 0, 4]):
        Ys = [torch.zeros_like(alone[i]) for i in pick]
        items = qamw.make_matmul_items([mats[i] + (y,) for i, y in zip(pick, Ys)])
        qamw.matmul_batch(items, cb, bits, block, torch.empty(items[4], dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        assert all(torch.equal(y, alone[i]) for i, y in zip(pick, Ys)), pick
