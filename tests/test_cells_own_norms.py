"""Launches in which the encoder computes row norms itself (large matrices whose rows a workgroup's waves can share: with bf16 weights
rows of 2, 4 or 8 full slabs of 1024 columns, with fp32 of one too) give the bytes and norms of the same rows in small launches, whose
norms come from a launch ahead of it: slab counts of every kind in one call, each first and last in turn, rows of zeros, rows that the
table does not decide (put off until the others are done)."""
import pytest
import torch

from paper_2605_26339_amd import qamw, synth

pytestmark = pytest.mark.gpu

SHAPES = [(8000, 4096), (301, 11008), (9001, 1024), (2003, 8192), (7, 512), (3000, 2048), (1001, 3072), (600, 16384), (4100, 4032)]


@pytest.mark.parametrize("bits,block,dtype,turn", [(11, 64, "bf16", 0), (11, 64, "f32", 4), (10, 64, "bf16", 7), (7, 64, "f32", 2), (6, 64, "bf16", 5),
                                                   (11, 128, "bf16", 1), (11, 1024, "f32", 3), (10, 256, "f32", 6), (9, 512, "bf16", 8), (7, 256, "bf16", 0)])
def test_norms_of_the_encoder_itself(bits, block, dtype, turn):
    print(f"[own norms] {bits} bits block {block} {dtype} turn {turn}", flush=True)
    cb = torch.from_numpy(qamw.train_codebook(bits, 1 << 16, seed=0, max_iters=20)[0]).cuda()
    mats = []
    for i, (d_out, d_in) in enumerate(SHAPES[turn:] + SHAPES[:turn]):
        d_in = max(block, d_in // block * block)
        W = synth.weight_device(11 * turn + i, d_out, d_in, 0.5, dtype)
        W[d_out // 3] = 0
        s = torch.from_numpy(qamw.channel_scales(synth.act_rms_host(i, d_in), 0.3)).cuda()
        sg = torch.from_numpy(qamw.sign_mask(i, d_in)).cuda()
        sigma = torch.full((d_in // 2,), d_in ** -0.5, device="cuda")
        if i % 3 == 1:
            sigma *= 0.05                   # pairs far outside the table
        out = (torch.empty((d_out, qamw.packed_row_bytes(d_in, bits)), dtype=torch.uint8, device="cuda"), torch.full((d_out,), -1.0, device="cuda"))
        mats.append((W, s, sg, sigma, *out))
    parts = {2048: 2, 4096: 3, 8192: 4}     # 64 MiB of rows of two slabs, 96 of four or 128 of eight
    assert sum(W.numel() * W.element_size() / parts[W.shape[1]] for W, *_ in mats if W.shape[1] in parts) >= 32 << 20
    for _ in range(2):
        qamw.encode_batch(qamw.make_encode_items(mats), cb, bits, block)
    torch.cuda.synchronize()
    for W, s, sg, sigma, packed, norms in mats:
        step = max(1, (16 << 20) // (W.shape[1] * W.element_size()))
        for r in range(0, W.shape[0], step):
            p1, n1 = qamw.encode(W[r:r + step], cb, bits, block, chan_scale=s, signs=sg, pair_sigma=sigma)
            torch.cuda.synchronize()
            assert torch.equal(n1, norms[r:r + step]) and torch.equal(p1, packed[r:r + step]), (tuple(W.shape), r)
