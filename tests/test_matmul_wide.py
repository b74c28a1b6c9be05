"""The fused product for many activation rows (a workspace that holds all of them) against the same product in tiles of at
most 64 rows (the least workspace): a row of Y has the same bits whichever kernel computes it."""
import ctypes as C
import sys

import pytest
import torch

from paper_2605_26339_amd import qamw

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _product(seed, d_out, d_in, m, bits, xdtype):
    g = torch.Generator("cuda").manual_seed(seed)
    cb = torch.randn(1 << bits, 2, device="cuda", generator=g)
    rb = qamw.packed_row_bytes(d_in, bits)
    packed = torch.randint(0, 256, (d_out, rb), dtype=torch.uint8, device="cuda", generator=g)
    norms = torch.rand(d_out, device="cuda", generator=g) + 0.5
    s = torch.rand(d_in, device="cuda", generator=g) + 0.5
    sg = (torch.randint(0, 2, (d_in,), device="cuda", generator=g) * 2 - 1).to(torch.int8)
    sigma = torch.rand(d_in // 2, device="cuda", generator=g) + 0.5
    X = torch.randn(m, d_in, device="cuda", generator=g).to(xdtype)
    return X, packed, norms, s, sg, sigma, cb


# edges: one chunk, fewer than eight chunks, segments of unequal length; rows and activation rows on either side of the
# tiles' (128, 256 / 128) and instructions' (32) edges; both tile widths; the split into a full and a partial round
@pytest.mark.parametrize("d_out,d_in,m,bits,block", [(1, 256, 193, 11, 64), (128, 768, 256, 7, 128), (129, 2304, 257, 8, 256),
                                                     (333, 4096, 300, 11, 1024), (130, 5632, 512, 11, 512), (4100, 1024, 1153, 7, 128),
                                                     (8193, 512, 1025, 11, 128), (11008, 256, 1000, 8, 64)])
@pytest.mark.parametrize("xdtype", [torch.bfloat16, torch.float32])
def test_wide_rows_have_the_bits_of_the_tiles(d_out, d_in, m, bits, block, xdtype):
    say(f"[wide] {d_out}x{d_in} m={m} B={bits} b={block} {xdtype}")
    X, packed, norms, s, sg, sigma, cb = _product(d_out + m, d_out, d_in, m, bits, xdtype)
    kw = dict(chan_scale=s, signs=sg, pair_sigma=sigma)
    least = torch.empty(qamw.matmul_workspace_bytes(d_in, d_out, m), dtype=torch.uint8, device="cuda")
    want = qamw.matmul(X, packed, norms, cb, bits, block, workspace=least, **kw)
    ldy = d_out + 5                                           # rows of Y at any alignment; nothing written beyond them
    full = torch.full((m, ldy), -3.0, device="cuda")
    got = qamw.matmul(X, packed, norms, cb, bits, block, out=full[:, :d_out], **kw)
    torch.cuda.synchronize()
    assert torch.equal(got, want) and bool((full[:, d_out:] == -3.0).all())
    # workspaces in between: fewer rows at a time
    for rows in (192, 224, 608):
        ws = torch.empty(rows * d_in * 2, dtype=torch.uint8, device="cuda")
        if ws.numel() >= least.numel():
            assert torch.equal(qamw.matmul(X, packed, norms, cb, bits, block, workspace=ws, **kw), want), rows


def test_wide_batch_equals_single_products():
    say("[wide] batch")
    m, bits, block = 260, 11, 128
    shapes = [(200, 1024), (1000, 4096), (64, 2560)]
    parts = [_product(i, d_out, d_in, m, bits, torch.bfloat16) for i, (d_out, d_in) in enumerate(shapes)]
    cb = parts[0][6]
    Y = [torch.empty(m, d_out, device="cuda") for d_out, _ in shapes]
    items = qamw.make_matmul_items([(X, p, r, s, sg, sigma, y) for (X, p, r, s, sg, sigma, _), y in zip(parts, Y)])
    ws = torch.empty(items[4], dtype=torch.uint8, device="cuda")
    qamw.matmul_batch(items, cb, bits, block, ws)
    for (X, p, r, s, sg, sigma, _), y, (d_out, d_in) in zip(parts, Y, shapes):
        least = torch.empty(qamw.matmul_workspace_bytes(d_in, d_out, m), dtype=torch.uint8, device="cuda")
        assert torch.equal(y, qamw.matmul(X, p, r, cb, bits, block, workspace=least, chan_scale=s, signs=sg, pair_sigma=sigma))
    need = sum(qamw.matmul_workspace_bytes(d_in, d_out, m) for d_out, d_in in shapes)
    before = [y.clone() for y in Y]
    for y in Y:
        y.zero_()
    qamw.matmul_batch(items, cb, bits, block, ws[:need])      # the least that is accepted: in tiles
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(Y, before))
    assert qamw.lib().qamw_matmul_batch(items[0], len(shapes), items[3], m, C.c_void_p(cb.data_ptr()), bits, block,
                                        C.c_void_p(ws.data_ptr()), need - 1, None) == qamw.ERR_INVALID_ARG


# 193 to 256 rows: in tiles of 64 where the rows are long and the wide tiles few, wide otherwise; both sides of the three lines
@pytest.mark.parametrize("d_out,d_in,m", [(130, 4096, 193), (130, 3840, 193), (8192, 4096, 200), (8193, 4096, 200), (4096, 4352, 256), (4096, 4352, 257)])
def test_either_kernel_around_four_tiles(d_out, d_in, m):
    say(f"[wide] four tiles {d_out}x{d_in} m={m}")
    X, packed, norms, s, sg, sigma, cb = _product(m, d_out, d_in, m, 7, torch.bfloat16)
    kw = dict(chan_scale=s, signs=sg, pair_sigma=sigma)
    least = torch.empty(qamw.matmul_workspace_bytes(d_in, d_out, m), dtype=torch.uint8, device="cuda")
    assert torch.equal(qamw.matmul(X, packed, norms, cb, 7, 128, **kw), qamw.matmul(X, packed, norms, cb, 7, 128, workspace=least, **kw))


# 256-row tiles over rows of several chunks a segment (the ring of three activation buffers goes round many times, and its requests
# cross from one chunk and segment into the next): all three widths, a chunk count that eight does and does not divide, d_out and m
# that end inside a tile; the second pair's last round goes into 128-row tiles of the same launch
@pytest.mark.parametrize("bits,d_out,d_in,m", [(11, 8193, 2304, 1025), (7, 8193, 4096, 1025), (8, 8320, 2560, 1000),
                                               (11, 11008, 4352, 1000), (7, 11008, 4352, 1000), (8, 11001, 4096, 993)])
def test_deep_rows_of_the_larger_tiles(bits, d_out, d_in, m):
    tiles256, tiles = (d_out + 127) // 128 * ((m + 255) // 256), (d_out + 127) // 128
    assert tiles256 >= 256 and d_in > 8 * 256
    first = tiles256 // 256 * 256 // ((m + 255) // 256)
    say(f"[wide] larger tiles {d_out}x{d_in} m={m} B={bits}, {tiles - first} of {tiles} in a last round")
    X, packed, norms, s, sg, sigma, cb = _product(d_out + m, d_out, d_in, m, bits, torch.bfloat16)
    kw = dict(chan_scale=s, signs=sg, pair_sigma=sigma)
    least = torch.empty(qamw.matmul_workspace_bytes(d_in, d_out, m), dtype=torch.uint8, device="cuda")
    want = qamw.matmul(X, packed, norms, cb, bits, 128 if d_in % 1024 else 1024, workspace=least, **kw)
    for _ in range(2):
        got = qamw.matmul(X, packed, norms, cb, bits, 128 if d_in % 1024 else 1024, **kw)
        torch.cuda.synchronize()
        assert torch.equal(got, want)


# 129 to 256 rows: either side of each line of the choice between the wide kernel and tiles of 64 (the rows' length, how many of the
# chip's CUs the wide tiles reach, how well they fill a last round)
@pytest.mark.parametrize("d_out,d_in,m", [(200, 512, 128), (200, 512, 129), (300, 2560, 130), (300, 2816, 192), (4992, 2816, 129), (5000, 2816, 129),
                                          (16385, 2816, 140), (24577, 2816, 140), (300, 5120, 193), (300, 5376, 256), (4096, 5376, 256),
                                          (4097, 5376, 193)])
def test_either_kernel_for_three_and_four_tiles(d_out, d_in, m):
    say(f"[wide] three and four tiles {d_out}x{d_in} m={m}")
    X, packed, norms, s, sg, sigma, cb = _product(m, d_out, d_in, m, 8, torch.float32)
    kw = dict(chan_scale=s, signs=sg, pair_sigma=sigma)
    least = torch.empty(qamw.matmul_workspace_bytes(d_in, d_out, m), dtype=torch.uint8, device="cuda")
    assert torch.equal(qamw.matmul(X, packed, norms, cb, 8, 256, **kw), qamw.matmul(X, packed, norms, cb, 8, 256, workspace=least, **kw))
