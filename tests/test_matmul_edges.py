"""The fused product for up to 8 activation rows where a workgroup's rows or a row's columns end: groups of eight rows that reach
the matrix's last row (their packed words are taken from further to the front), slabs that are not full, waves with steps of one
slab, of several and of none; rows of X that begin anywhere.  Against X times the decoder's fp32 output in fp64 (bar 1e-5
||x|| ||w_i||, a hundred times the rounding of an fp32 sum over the row), and bit-identical whichever kernel rotates."""
import sys

import numpy as np
import pytest
import torch

from paper_2605_26339_amd import qamw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [7, 8, 11])
@pytest.mark.parametrize("d_out,d_in,block", [(1, 64, 64), (7, 192, 64), (8, 1024, 128), (9, 1088, 64), (17, 5632, 512), (40, 3072, 1024)])
@pytest.mark.parametrize("m,xdtype,plain", [(1, torch.bfloat16, False), (1, torch.float32, True), (2, torch.float32, False),
                                            (3, torch.bfloat16, True), (8, torch.bfloat16, False)])
def test_few_rows_at_the_edges(bits, d_out, d_in, block, m, xdtype, plain):
    print(f"[matmul edges] {d_out}x{d_in} B={bits} b={block} m={m} {xdtype} plain={plain}", flush=True)
    sys.stdout.flush()
    g = torch.Generator("cuda").manual_seed(1000 * bits + d_out + m)
    cb = torch.randn(1 << bits, 2, device="cuda", generator=g)
    pk = torch.randint(0, 256, (d_out, qamw.packed_row_bytes(d_in, bits)), dtype=torch.uint8, device="cuda", generator=g)
    nr = torch.rand(d_out, device="cuda", generator=g) + 0.5
    kw = {}
    if not plain:
        kw = dict(chan_scale=torch.exp(0.5 * torch.randn(d_in, device="cuda", generator=g)),
                  signs=(torch.randint(0, 2, (d_in,), device="cuda", generator=g) * 2 - 1).to(torch.int8),
                  pair_sigma=(torch.rand(d_in // 2, device="cuda", generator=g) + 0.5) / np.sqrt(d_in))
    X = torch.randn(m * d_in + 1, device="cuda", generator=g).to(xdtype)[1:].view(m, d_in)   # one element off any alignment
    Y = qamw.matmul(X, pk, nr, cb, bits, block, **kw)
    W = qamw.decode(pk, nr, d_in, cb, bits, block, f32=True, **kw).double()
    bar = 1e-5 * X.double().norm(dim=1)[:, None] * W.norm(dim=1)[None, :] + 1e-30
    assert float(((Y.double() - X.double() @ W.t().contiguous()).abs() / bar).max()) <= 1.0
    if m <= 2:
        for path in (1, 2):
            prev = qamw.set_kernel_path(path)
            try:
                Yp = qamw.matmul(X, pk, nr, cb, bits, block, **kw)
                torch.cuda.synchronize()
            finally:
                qamw.set_kernel_path(prev)
            assert torch.equal(Yp, Y), f"kernel path {path}"
