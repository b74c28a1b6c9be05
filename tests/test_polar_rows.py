"""The polar encoder's workgroups own several whole rows; how many depends on the matrix.  Rows encoded alone (one row per
workgroup) and in matrices whose workgroups hold many, with a remainder, give the same bytes and norms; and the bytes are
those of the definition in float64 away from the decisions' boundaries."""
import math
import sys

import pytest
import torch

from paper_2605_26339_amd import qamw, synth

pytestmark = pytest.mark.gpu


# one slab (48 rows cut to 32 per workgroup), a ragged slab, 11 slabs, more slabs than a workgroup's item count allows for
# two rows; few and many thresholds, none at all
@pytest.mark.parametrize("d_out,d_in,bits_a,bits_p,block,dtype", [
    (20003, 1024, 5, 6, 128, "bf16"), (20003, 64, 3, 4, 64, "f32"), (9001, 2176, 0, 1, 128, "bf16"), (2051, 11008, 4, 4, 256, "f32"),
    (700, 33792, 6, 0, 1024, "bf16"), (515, 4096, 0, 0, 512, "f32"), (515, 5632, 1, 12 - 1, 512, "bf16"), (3, 65536, 2, 5, 64, "f32")])
def test_rows_are_the_same_in_any_workgroup(d_out, d_in, bits_a, bits_p, block, dtype):
    print(f"[polar rows] {d_out}x{d_in} {bits_a}+{bits_p} b={block} {dtype}", flush=True)
    sys.stdout.flush()
    bits = bits_a + bits_p
    if bits < 1:
        bits_a = bits = 1
    levels = torch.from_numpy(qamw.polar_codebook(bits_a, bits_p)[0]).cuda()
    W = synth.weight_device(d_out, d_out, d_in, 1.0, dtype)
    W[d_out // 2] = 0
    s = torch.from_numpy(qamw.channel_scales(synth.act_rms_host(1, d_in), 0.3)).cuda()
    sg = torch.from_numpy(qamw.sign_mask(2, d_in)).cuda()
    g = torch.Generator("cuda").manual_seed(3)
    sigma = (0.5 + torch.rand(d_in // 2, device="cuda", generator=g)) / math.sqrt(d_in)
    kw = dict(chan_scale=s, signs=sg, pair_sigma=sigma)
    packed, norms = qamw.encode_polar(W, levels, bits_a, bits_p, block, **kw)
    torch.cuda.synchronize()
    for r in sorted({0, 1, 2, d_out // 2, d_out - 2, d_out - 1}):
        p1, n1 = qamw.encode_polar(W[r:r + 1], levels, bits_a, bits_p, block, **kw)
        torch.cuda.synchronize()
        assert torch.equal(p1[0], packed[r]) and torch.equal(n1[0], norms[r]), r
    # a sample of rows against float64
    rows = torch.arange(0, d_out, max(1, d_out // 64), device="cuda")
    ws = W[rows].double() * s.double()
    norm = ws.norm(dim=1, keepdim=True)
    assert torch.allclose(norm[:, 0], norms[rows].double(), rtol=1.3e-7, atol=0)
    y = torch.where(norm > 0, ws / norm.clamp(min=1e-300), 0.0) * sg.double()
    y = y.view(-1, block)
    h = 1
    while h < block:
        y = y.view(-1, block // (2 * h), 2, h)
        y = torch.stack((y[:, :, 0] + y[:, :, 1], y[:, :, 0] - y[:, :, 1]), 2).reshape(-1, block)
        h *= 2
    x = (y / math.sqrt(block)).view(len(rows), -1, 2) / sigma.double()[None, :, None]
    a, ph = x.norm(dim=2), torch.remainder(torch.atan2(x[..., 1], x[..., 0]), 2 * math.pi) * (1 << bits_p) / (2 * math.pi)
    mids = 0.5 * (levels[1:] + levels[:-1]).double()
    ia = torch.bucketize(a, mids)
    ip = torch.where(a == 0, 0.0, ph).floor().long() % (1 << bits_p)
    stream = (packed[rows][:, :, None] >> torch.arange(8, device="cuda", dtype=torch.uint8)) & 1
    used = d_in // 2 * bits
    assert not stream.reshape(len(rows), -1)[:, used:].any()
    got = (stream.reshape(len(rows), -1)[:, :used].view(len(rows), -1, bits).long() << torch.arange(bits, device="cuda")).sum(-1)
    # fp32 points are within 1e-5 (1 + |x|) of the exact ones (a norm, 10 butterflies, three products)
    eps = 1e-5 * (1 + a)
    clear_a = torch.full_like(a, True, dtype=torch.bool) if len(mids) == 0 else ((a[..., None] - mids).abs().amin(-1) > eps)
    clear_p = ((ph - ph.round()).abs() * a * (2 * math.pi / (1 << bits_p)) > eps) | (a == 0) | (bits_p == 0)
    assert torch.equal((got >> bits_p)[clear_a], ia[clear_a])
    assert torch.equal((got & ((1 << bits_p) - 1))[clear_p], ip[clear_p])
    assert clear_a.double().mean() > 0.99 and clear_p.double().mean() > 0.8


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_a_long_row_shared_by_workgroups(dtype):
    # one row is shared by as many workgroups as it has eight slabs; 600 such rows are not shared: the same bytes and norms, and no
    # more time for few rows than the matrix-at-once kernel's share (4-wave workgroups of four items took 14.4 us for 16 x 40960,
    # one workgroup a row 23)
    block, bits_a, bits_p = 64, 5, 6
    levels = torch.from_numpy(qamw.polar_codebook(bits_a, bits_p)[0]).cuda()
    for d_in in (8192, 9216, 40960, 66560):
        print(f"[polar rows] shared 600x{d_in} {dtype}", flush=True)
        W = synth.weight_device(d_in, 600, d_in, 1.0, dtype)
        want = qamw.encode_polar(W, levels, bits_a, bits_p, block)
        for lo, n in ((0, 1), (17, 16), (300, 100), (0, 300)):
            got = qamw.encode_polar(W[lo:lo + n], levels, bits_a, bits_p, block)
            torch.cuda.synchronize()
            assert torch.equal(got[0], want[0][lo:lo + n]) and torch.equal(got[1], want[1][lo:lo + n]), (d_in, lo, n)
    W = synth.weight_device(1, 16, 40960, 1.0, dtype)
    out = qamw.encode_polar(W, levels, bits_a, bits_p, block)
    best = 1e9
    for _ in range(20):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            qamw.encode_polar(W, levels, bits_a, bits_p, block, out=out)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / 20 * 1e3)
    print(f"[polar rows] 16x40960: {best:.1f} us", flush=True)
    assert best < 19.0
