"""Pair scales where the calibration kernel deals a chunk's rows or slabs differently to its waves: one to four slabs (rows
shared by 8, 4 and 2 waves), more slabs than waves, ragged slabs, chunks of fewer than 8 rows, zero and tiny rows."""
import math
import sys

import pytest
import torch

from paper_2605_26339_amd import qamw, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_in,block", [(64, 64), (1024, 1024), (1152, 128), (2048, 256), (2560, 512), (4096, 128), (4160, 64),
                                        (8192, 1024), (9216, 512), (11008, 256)])
@pytest.mark.parametrize("d_out,dtype", [(1, "f32"), (7, "bf16"), (9, "f32"), (300, "bf16"), (1100, "f32")])
def test_pair_scales_against_float64(d_in, block, d_out, dtype):
    print(f"[calibrate] {d_out}x{d_in} b={block} {dtype}", flush=True)
    sys.stdout.flush()
    W = synth.weight_device(d_in + d_out, d_out, d_in, 1.0, dtype)
    if d_out > 1:
        W[1] = 0                                               # contributes zeros to every pair's mean
    if d_out > 8:
        W[8] *= 1e-30                                          # normalised like any other row
    s = torch.from_numpy(qamw.channel_scales(synth.act_rms_host(1, d_in), 0.3)).cuda()
    sg = torch.from_numpy(qamw.sign_mask(2, d_in)).cuda()
    got = qamw.calibrate_sigma(W, block, chan_scale=s, signs=sg)
    torch.cuda.synchronize()
    ws = W[:1024].double() * s.double()
    norm = ws.norm(dim=1, keepdim=True)
    y = (torch.where(norm > 0, ws / norm.clamp(min=1e-300), 0.0) * sg.double()).view(-1, block)
    h = 1
    while h < block:
        y = y.view(-1, block // (2 * h), 2, h)
        y = torch.stack((y[:, :, 0] + y[:, :, 1], y[:, :, 0] - y[:, :, 1]), 2).reshape(-1, block)
        h *= 2
    z = (y / math.sqrt(block)).view(len(ws), -1, 2)
    want = z.norm(dim=2).mean(0) / math.sqrt(math.pi / 2)
    # fp32 coefficients: the unit row, up to 10 butterflies and two products, each half a unit of a value no larger than the
    # row's largest partial sum; the mean of |z| over few rows may hit a small |z|, hence the absolute part
    assert torch.allclose(got.double(), want, rtol=2e-6, atol=2e-6 / math.sqrt(d_in)), (got.double() / want - 1).abs().max()
