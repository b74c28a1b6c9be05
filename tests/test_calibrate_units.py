"""Pair scales of rows whose slabs of 1024 columns do not divide evenly among a workgroup's eight waves: each count of slabs left
over after eight at a time, with all and with few of a chunk's eight rows; and the same bits alone and beside longer rows."""
import sys

import pytest
import torch

from paper_2605_26339_amd import qamw, synth

from .test_calibrate_split import test_pair_scales_against_float64 as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_in,block", [(6144, 256), (7168, 1024), (10240, 512), (12224, 64), (13824, 128), (16384, 1024)])
@pytest.mark.parametrize("d_out,dtype", [(3, "bf16"), (21, "f32"), (64, "bf16")])
def test_slabs_left_over(d_in, block, d_out, dtype):
    check(d_in, block, d_out, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_alone_and_in_a_batch(dtype):
    print(f"[calibrate] batch {dtype}", flush=True)
    sys.stdout.flush()
    items, alone = [], []
    for i, (d_out, d_in) in enumerate([(70, 2048), (33, 11008), (9, 10240), (100, 512)]):
        W = synth.weight_device(i, d_out, d_in, 1.0, dtype)
        items.append((W, None, None, torch.empty(d_in // 2, device="cuda")))
        alone.append(qamw.calibrate_sigma(W, 128))
    cal = qamw.make_calibrate_items(items)
    qamw.calibrate_sigma_batch(cal, 128, torch.empty(cal[3], dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    for (_, _, _, got), want in zip(items, alone):
        assert torch.equal(got, want)


# a unit of one, two, four and more rows of a chunk, and what a chunk at the matrix's end leaves of it
@pytest.mark.parametrize("d_in,block", [(64, 64), (512, 512), (1024, 128), (1152, 128), (2048, 1024), (3072, 256), (5120, 64)])
@pytest.mark.parametrize("d_out,dtype", [(1, "bf16"), (6, "bf16"), (11, "f32"), (27, "bf16")])
def test_rows_of_a_unit(d_in, block, d_out, dtype):
    check(d_in, block, d_out, dtype)
