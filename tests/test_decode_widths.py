"""The fast decoder at every bit width it takes (4 to 12) and at each length of a wave's unit of rows, against the general
decoder: within two roundings of it in fp32, one unit in the last place in bf16, nothing written outside the output."""
import sys

import pytest
import torch

from paper_2605_26339_amd import qamw

def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _case(bits, d_out, d_in, seed):
    g = torch.Generator("cuda").manual_seed(seed)
    rb = qamw.packed_row_bytes(d_in, bits)
    packed = torch.randint(0, 256, (d_out, rb), dtype=torch.uint8, device="cuda", generator=g)
    rest = d_in // 2 * bits % 8
    if rest:
        packed[:, d_in // 2 * bits // 8] &= (1 << rest) - 1
    cb = torch.randn(1 << bits, 2, device="cuda", generator=g)
    norms = torch.rand(d_out, device="cuda", generator=g) + 0.5
    s = torch.rand(d_in, device="cuda", generator=g) + 0.5
    sg = (torch.randint(0, 2, (d_in,), device="cuda", generator=g) * 2 - 1).to(torch.int8)
    sigma = torch.rand(d_in // 2, device="cuda", generator=g) + 0.5
    return packed, norms, cb, dict(chan_scale=s, signs=sg, pair_sigma=sigma)


def _general(*a, **kw):
    prev = qamw.set_kernel_path(1)
    try:
        return qamw.decode(*a, **kw)
    finally:
        qamw.set_kernel_path(prev)


def _order(t):                                                # bf16 bits as integers that are monotone in the value
    b = t.view(torch.int16).int()
    return torch.where(b < 0, -(b & 0x7FFF), b)


@pytest.mark.parametrize("bits", range(4, 13))
def test_loads_stay_inside_the_packed_rows(bits):
    """The loads of the fast decoder, as its fetch() makes them: 16 bytes from the dword that a lane's 16 columns begin in, in the
    last row dword by dword and none past its end.  (No allocation on the GPU is sized to the byte, so a run cannot show it.)"""
    for d_in in [64 * k for k in range(1, 40)] + [1024 * 16 + 64, 65536]:
        rb = qamw.packed_row_bytes(d_in, bits)
        assert rb % 4 == 0 and rb >= 4 * bits
        for c in range(0, d_in, 16):                          # a lane's first column; lanes past the row read as the first does
            off = c // 16 * bits
            b0 = off & ~3
            assert off + bits <= b0 + 16 <= 2 * rb            # the fields are among the bytes; a row that is not the last has a next
            last = [min(b0 // 4 + k, rb // 4 - 1) for k in range(4)]
            covered = {4 * w + i for w in last for i in range(4)}
            assert max(last) < rb // 4 and set(range(off, off + bits)) <= covered
            # a clamped word stands where no field is
            assert all(4 * (b0 // 4 + k) >= off + bits for k in range(4) if b0 // 4 + k > rb // 4 - 1)


# shortest rows (64 columns), ragged last slabs, row counts around the units of 2, 4, 8 and 16 rows; the last three launches
# have 2, 4 and full rows per unit
@pytest.mark.gpu
@pytest.mark.parametrize("bits", range(4, 13))
def test_every_width(bits):
    for d_out, d_in, block in [(1, 64, 64), (3, 64, 64), (17, 192, 64), (5, 5632, 512), (33, 2048, 1024), (4095, 2048, 128),
                               (8191, 1088, 64), (8192, 4096, 256)]:
        say(f"[decode widths] B={bits} {d_out}x{d_in} b={block}")
        packed, norms, cb, kw = _case(bits, d_out, d_in, bits * 1000 + d_out)
        full = torch.full((d_out, d_in + 8), -7.0, dtype=torch.bfloat16, device="cuda")
        got = qamw.decode(packed, norms, d_in, cb, bits, block, out=full[:, :d_in], **kw)
        want = _general(packed, norms, d_in, cb, bits, block, **kw)
        assert bool((full[:, d_in:] == -7.0).all())
        assert int((_order(got.contiguous()) - _order(want)).abs().max()) <= 1
        got32 = qamw.decode(packed, norms, d_in, cb, bits, block, f32=True, **kw)
        want32 = _general(packed, norms, d_in, cb, bits, block, f32=True, **kw)
        # the row factor, the column factor and its reciprocal: each rounded once, in another order (2^-24 each)
        assert float(((got32 - want32).abs() / want32.abs().clamp_min(1e-30)).max()) <= 6 * 2.0 ** -24


# The widths that the general kernel served before: its bits, in fp32 and in bf16, at every block and launch size (at the paper's
# three rates the trailing factors are fused).  Column scales over 60 orders of magnitude: the reciprocal is rounded correctly.
@pytest.mark.gpu
@pytest.mark.parametrize("bits", [4, 5, 6, 9, 10, 12])
def test_widths_between_the_papers_round_as_the_general_kernel(bits):
    for d_out, d_in, block in [(3, 64, 64), (700, 2048, 128), (1100, 8192, 128), (40, 5632, 512), (8200, 4096, 512), (65, 3072, 256),
                               (33, 2048, 1024)]:
        say(f"[decode widths] exact B={bits} {d_out}x{d_in} b={block}")
        packed, norms, cb, kw = _case(bits, d_out, d_in, bits * 7 + d_out)
        kw["chan_scale"] = 10.0 ** (torch.rand(d_in, device="cuda", generator=torch.Generator("cuda").manual_seed(d_in)) * 60 - 30)
        for form in (kw, {}):
            assert torch.equal(qamw.decode(packed, norms, d_in, cb, bits, block, f32=True, **form),
                               _general(packed, norms, d_in, cb, bits, block, f32=True, **form))
            assert torch.equal(qamw.decode(packed, norms, d_in, cb, bits, block, **form),
                               _general(packed, norms, d_in, cb, bits, block, **form))   # (a zero's sign aside)


@pytest.mark.gpu
def test_unaligned_codebook_and_other_optional_forms():
    say("[decode widths] codebook at 8 bytes, no side vectors")
    bits, d_out, d_in, block = 10, 40, 2048, 128
    packed, norms, cb, kw = _case(bits, d_out, d_in, 5)
    shifted = torch.empty(2 * (1 << bits) + 2, device="cuda")[2:].view(-1, 2)
    shifted.copy_(cb)
    assert torch.equal(qamw.decode(packed, norms, d_in, shifted, bits, block, **kw), _general(packed, norms, d_in, cb, bits, block, **kw))
    got, want = qamw.decode(packed, norms, d_in, cb, bits, block), _general(packed, norms, d_in, cb, bits, block)
    assert int((_order(got) - _order(want)).abs().max()) <= 1
    items = qamw.make_decode_items([(packed, norms, d_in, None, None, None, torch.empty_like(got))])
    with pytest.raises(qamw.QamwError) as e:                  # the traffic probe stays with the paper's three rates
        qamw.decode_traffic_probe(items, cb, bits, block)
    assert e.value.status == qamw.ERR_UNSUPPORTED
