"""The polar encoder's workgroups that stay for several steps of rows, with lookup tables, give each row what it gets alone (a
workgroup of its own, binary searches): last steps and last workgroups of fewer rows, rows and pairs of zeros, the fewest and the most
bins that have tables."""
import math

import pytest
import torch

from paper_2605_26339_amd import qamw, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_out,d_in,bits_a,bits_p,block,dtype", [
    (3584, 11008, 5, 6, 256, "bf16"),       # seven rows a workgroup: steps of four and three
    (3585, 11008, 4, 3, 128, "f32"),        # eight, the last workgroup one; eight bins
    (18433, 1024, 3, 8, 64, "bf16"),   # 37 rows of one slab, 256 bins, the last workgroup seven
    (9000, 2112, 5, 5, 64, "f32"),          # three slabs, the last of one block
    (20000, 2048, 0, 9, 1024, "bf16"),      # more bins than have tables
    (20000, 2048, 6, 0, 512, "bf16"),       # no bins
    (1001, 66560, 5, 6, 1024, "bf16")])     # norms from a launch ahead; steps of one row, the last workgroup one step
def test_a_row_in_any_step(d_out, d_in, bits_a, bits_p, block, dtype):
    print(f"[polar steps] {d_out}x{d_in} {bits_a}+{bits_p} b={block} {dtype}", flush=True)
    levels = torch.from_numpy(qamw.polar_codebook(bits_a, bits_p)[0]).cuda()
    W = synth.weight_device(d_out, d_out, d_in, 1.0, dtype)
    W[7] = 0
    W[9, : d_in // 2 // block * block] = 0  # whole blocks: pairs of zeros
    s = torch.from_numpy(qamw.channel_scales(synth.act_rms_host(1, d_in), 0.3)).cuda()
    sg = torch.from_numpy(qamw.sign_mask(2, d_in)).cuda()
    g = torch.Generator("cuda").manual_seed(3)
    sigma = (0.5 + torch.rand(d_in // 2, device="cuda", generator=g)) / math.sqrt(d_in)
    kw = dict(chan_scale=s, signs=sg, pair_sigma=sigma)
    packed, norms = qamw.encode_polar(W, levels, bits_a, bits_p, block, **kw)
    torch.cuda.synchronize()
    for r in [*range(24), *range(24, d_out, d_out // 16), *range(d_out - 12, d_out)]:
        p1, n1 = qamw.encode_polar(W[r:r + 1], levels, bits_a, bits_p, block, **kw)
        torch.cuda.synchronize()
        assert torch.equal(p1[0], packed[r]) and torch.equal(n1[0], norms[r]), r
