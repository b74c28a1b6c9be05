"""Row norms are the same to the bit with scratch and without, alone and in a batch: fp64 sums whose fp32 square root depends on
the order of the addends."""
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


def _row(d_in, dtype):
    """1 + 2^-23 + 2^-48, whose root lies half way between two fp32 numbers, and eight times 2^-54: lost one by one beside the 1,
    2^-51 when added up first, which rounds the root up.  The eight stand where a lane that takes every 256th (fp32) or 512th
    (bf16) columns' worth of 16 bytes meets them after the 1, and a lane that takes 16 columns in a run does not."""
    row = np.zeros(d_in, dtype=np.float32)
    row[:4] = 1.0, 2.0 ** -12, 2.0 ** -12, 2.0 ** -24
    for at in (512, 768) if dtype == torch.float32 else (512, 516):
        row[at:at + 4] = 2.0 ** -27
    return row


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("bits,d_out,d_in", [(11, 3, 2048), (11, 8195, 2048), (7, 300, 4096), (6, 9000, 1024), (5, 5, 1024), (5, 5000, 1024),
                                             (4, 4100, 1088), (3, 4100, 1024), (11, 2, 66560)])
def test_with_scratch_and_without(dtype, bits, d_out, d_in):
    say(f"[norm order] B={bits} {d_out}x{d_in} {dtype}")
    block = 64
    row = _row(d_in, dtype)
    up, down = np.float32(1 + 2.0 ** -23), np.float32(1)
    squares = row.astype(np.float64) ** 2
    assert np.float32(np.sqrt(squares[:4].sum())) == down and np.float32(np.sqrt(squares[:4].sum() + squares[4:].sum())) == up
    W = torch.from_numpy(np.tile(row, (d_out, 1))).cuda().to(dtype)
    cb = torch.randn(1 << bits, 2, device="cuda", generator=torch.Generator("cuda").manual_seed(bits))
    want = qamw.encode(W, cb, bits, block, full_scans=torch.zeros(1, dtype=torch.int64, device="cuda"))
    if bits > 3 and d_in <= 65536:                            # slab by slab, 16 columns a lane
        assert bool((want[1] == float(up)).all())
    outs = [tuple(torch.empty_like(t) for t in want) for _ in range(2)]
    qamw.encode_batch(qamw.make_encode_items([(W, None, None, None, p, r) for p, r in outs]), cb, bits, block)
    for got in (qamw.encode(W, cb, bits, block), *outs):
        torch.cuda.synchronize()
        assert torch.equal(got[1], want[1]) and torch.equal(got[0], want[0])
    assert torch.equal(qamw.normalised_pairs(W, block)[1], want[1]) or bits <= 3
    # the pruned search, whose norms come from a launch of their own
    grid = torch.from_numpy(qamw.search_grid(cb.cpu().numpy(), bits)[0]).cuda()
    got = qamw.encode_pruned(W, cb, grid, bits, block)
    packed, norms = torch.empty_like(got[0]), torch.empty_like(got[1])
    assert qamw.lib().qamw_encode_pruned(W.data_ptr(), 0 if dtype == torch.float32 else 1, d_out, d_in, d_in, None, None, None, cb.data_ptr(),
                                         bits, block, grid.data_ptr(), packed.data_ptr(), norms.data_ptr(), None, None) == qamw.OK
    torch.cuda.synchronize()
    assert torch.equal(got[1], norms) and torch.equal(got[0], packed)


def test_codebook_at_eight_bytes():
    # the whole-codebook kernels need 16; the general kernels serve such a call without scratch, and their norms are what it gets
    say("[norm order] codebook at 8 bytes")
    bits, d_out, d_in, block = 11, 40, 2048, 128
    W = torch.from_numpy(np.tile(_row(d_in, torch.float32), (d_out, 1))).cuda()
    cb = torch.randn((1 << bits) + 1, 2, device="cuda")[1:]
    want = (torch.empty((d_out, qamw.packed_row_bytes(d_in, bits)), dtype=torch.uint8, device="cuda"), torch.empty(d_out, device="cuda"))
    assert qamw.lib().qamw_encode(W.data_ptr(), 0, d_out, d_in, d_in, None, None, None, C.c_void_p(cb.data_ptr()), bits, block,
                                  want[0].data_ptr(), want[1].data_ptr(), None) == qamw.OK
    got = qamw.encode(W, cb, bits, block)
    torch.cuda.synchronize()
    assert torch.equal(got[1], want[1]) and torch.equal(got[0], want[0])
