"""The encoder with a cell table made on the device (qamw_encode_ws / qamw_encode_batch_ws) against the search over the
whole codebook (qamw_encode_stats, which never uses a table): the same bytes and the same norms."""
import ctypes as C
import sys

import numpy as np
import pytest
import torch

from paper_2605_26339_amd import qamw, synth


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def test_workspace_sizes_and_errors():
    L = qamw.lib()
    assert [qamw.encode_workspace_bytes(b) for b in (1, 9, 10, 11, 12)] == [64 * 64 * 8, 64 * 64 * 8, 96 * 96 * 8, 128 * 128 * 8, 0]
    out = C.c_size_t()
    for bits in (0, 13):
        assert L.qamw_encode_workspace_bytes(bits, C.byref(out)) == qamw.ERR_INVALID_ARG
    assert L.qamw_encode_workspace_bytes(11, None) == qamw.ERR_INVALID_ARG
    p = C.c_void_p(4096)                                      # checked on the host before any launch
    args = dict(W=p, cb=p, packed=p, norms=p)

    def call(ws, **kw):
        a = {**args, **kw}
        return L.qamw_encode_ws(a["W"], 1, 8, kw.get("d_in", 256), 256, None, None, None, a["cb"], 11, kw.get("block", 128),
                                C.c_void_p(ws), 1 << 20, a["packed"], a["norms"], None)
    assert call(4096 + 8) == qamw.ERR_INVALID_ARG             # misaligned workspace
    assert call(4096, W=None) == qamw.ERR_INVALID_ARG
    assert call(4096, packed=C.c_void_p(4098)) == qamw.ERR_INVALID_ARG
    assert call(4096, block=96) == qamw.ERR_SHAPE
    assert call(4096, d_in=512) == qamw.ERR_SHAPE             # leading dimension below the row
    assert L.qamw_encode_batch_ws(None, 1, 1, p, 11, 128, p, 1 << 20, None) == qamw.ERR_INVALID_ARG


def _codebook(bits, kind):
    rng = np.random.default_rng(bits)
    cb = qamw.train_codebook(bits, 1 << 14, max_iters=10)[0] if kind != "random" else rng.standard_normal((1 << bits, 2)).astype(np.float32)
    if kind == "far":
        cb = cb * np.float32(64.0)
    elif kind == "small":
        cb = cb * np.float32(1 / 16)
    elif kind == "clustered":
        cb[cb.shape[0] // 4:] = (0.5 + 1e-4 * rng.standard_normal((cb.shape[0] - cb.shape[0] // 4, 2))).astype(np.float32)
    elif kind == "duplicates":
        cb[cb.shape[0] // 2:] = cb[:cb.shape[0] // 2]
    elif kind == "lattice":                                   # exact ties along the cells' edges
        n = int(round(len(cb) ** 0.5))
        g = (np.arange(n) - n / 2).astype(np.float32) * np.float32(0.25)
        cb[:n * n] = np.stack(np.meshgrid(g, g), -1).reshape(-1, 2)
    return np.ascontiguousarray(cb, dtype=np.float32)


def _both(W, cb, bits, block, **kw):
    scans = torch.zeros(1, dtype=torch.int64, device="cuda")
    want = qamw.encode(W, cb, bits, block, full_scans=scans, **kw)
    got = qamw.encode(W, cb, bits, block, **kw)
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.gpu
@pytest.mark.parametrize("bits", range(1, 12))
def test_every_bit_width_and_shape_of_item(bits):
    # rows of one slab, of a ragged last slab (16 columns; half a slab), one row, more rows than waves of a slab
    for seed, (d_out, d_in, block, dtype) in enumerate([(1, 64, 64, "f32"), (7, 1040 if bits % 2 else 1088, 16 if bits % 2 else 64, "bf16"),
                                                        (333, 5632, 512, "bf16"), (129, 2048, 1024, "f32"), (2100, 1152, 128, "bf16"),
                                                        (40, 11008, 256, "f32")]):
        say(f"[cells] B={bits} {d_out}x{d_in} b={block} {dtype}")
        cb = torch.from_numpy(_codebook(bits, "lloyd")).cuda()
        W = synth.weight_device(seed + 10 * bits, d_out, d_in, 1.0, dtype)
        s = torch.from_numpy(qamw.channel_scales(synth.act_rms_host(seed, d_in), 0.3)).cuda()
        sg = torch.from_numpy(qamw.sign_mask(seed, d_in)).cuda()
        W[d_out // 2] = 0
        sigma = qamw.calibrate_sigma(W, block, chan_scale=s, signs=sg) if d_out > 8 else None
        _both(W, cb, bits, block, chan_scale=s, signs=sg, pair_sigma=sigma)
        _both(W, cb, bits, block)


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["far", "small", "clustered", "duplicates", "lattice", "random"])
@pytest.mark.parametrize("bits", [4, 8, 10, 11])
def test_codebooks_that_strain_the_table(bits, kind):
    say(f"[cells] B={bits} codebook {kind}")
    cb = torch.from_numpy(_codebook(bits, kind)).cuda()
    g = torch.Generator("cuda").manual_seed(bits)
    W = torch.randn(48, 2048, device="cuda", generator=g)
    wild = (10.0 ** (torch.rand(1024, device="cuda", generator=g) * 6 - 4.5) / 45).contiguous()
    for sigma in (None, wild):                                # wild: pairs far outside the table, and all in one cell
        _both(W, cb, bits, 128, pair_sigma=sigma)
    heavy = torch.from_numpy(np.random.default_rng(1).standard_t(1.5, (16, 2048)).astype(np.float32)).cuda()
    _both(heavy, cb, bits, 64)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_batches_strides_streams_and_workspaces(dtype):
    say(f"[cells] batch, padded rows, second stream, workspace forms {dtype}")
    bits, block = 11, 128
    cb = torch.from_numpy(_codebook(bits, "lloyd")).cuda()
    shapes = [(300, 4096), (5, 1024), (64, 11008), (1, 640), (777, 5120)]
    Ws, outs = [], []
    for i, (d_out, d_in) in enumerate(shapes):
        full = synth.weight_device(i, d_out, d_in + 16 * i, 0.5, dtype)
        Ws.append(full[:, :d_in])
        outs.append((torch.full((d_out, qamw.packed_row_bytes(d_in, bits)), 0xAA, dtype=torch.uint8, device="cuda"),
                     torch.zeros(d_out, device="cuda")))
    items = qamw.make_encode_items([(W, None, None, None, p, r) for W, (p, r) in zip(Ws, outs)])
    scans = torch.zeros(1, dtype=torch.int64, device="cuda")
    want = [qamw.encode(W, cb, bits, block, full_scans=scans) for W in Ws]
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())

    def check(what):
        torch.cuda.synchronize()
        for (p, r), (wp, wr) in zip(outs, want):
            assert torch.equal(p, wp) and torch.equal(r, wr), what
            p.fill_(0xAA)
            r.zero_()
        torch.cuda.synchronize()
    qamw.encode_batch(items, cb, bits, block)
    check("batch")
    qamw.encode_batch(items, cb, bits, block, stream=st)
    check("another stream")
    L = qamw.lib()
    n = qamw.encode_workspace_bytes(bits)
    ws = torch.empty(n + 16, dtype=torch.uint8, device="cuda")
    for off, size in ((0, n), (16, n), (0, n - 1), (0, 0)):   # enough (two alignments); too small: the whole-codebook encoder
        assert L.qamw_encode_batch_ws(items[0], len(shapes), items[2], C.c_void_p(cb.data_ptr()), bits, block,
                                      C.c_void_p(ws.data_ptr() + off), size, None) == qamw.OK
        check((off, size))
    assert L.qamw_encode_batch_ws(items[0], len(shapes), items[2], C.c_void_p(cb.data_ptr()), bits, block, None, n, None) == qamw.OK
    check("no workspace")
    one = qamw.encode(Ws[0], cb, bits, block, stream=st)      # outputs and scratch allocated here, used on the other stream
    torch.cuda.synchronize()
    assert torch.equal(one[0], want[0][0])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_records_from_memory_and_from_lds(dtype):
    # at 11 bits the launch's item count decides where the records are read from: both sides of the line, a slab count that
    # does not divide the waves, and a batch whose matrices share a launch
    bits, block = 11, 128
    cb = torch.from_numpy(_codebook(bits, "lloyd")).cuda()
    for d_out, d_in in [(1, 128), (1024, 3072), (1025, 3072), (279, 11008), (280, 11008), (3, 14336)]:
        say(f"[cells] records {d_out}x{d_in} {dtype}")
        W = synth.weight_device(d_out, d_out, d_in, 0.5, dtype)
        _both(W, cb, bits, block)
    Ws = [synth.weight_device(i, d_out, d_in, 0.5, dtype) for i, (d_out, d_in) in enumerate([(5, 11008), (1, 1024), (64, 3072), (40, 14336)])]
    outs = [(torch.full((W.shape[0], qamw.packed_row_bytes(W.shape[1], bits)), 0xAA, dtype=torch.uint8, device="cuda"),
             torch.zeros(W.shape[0], device="cuda")) for W in Ws]
    qamw.encode_batch(qamw.make_encode_items([(W, None, None, None, p, r) for W, (p, r) in zip(Ws, outs)]), cb, bits, block)
    torch.cuda.synchronize()
    scans = torch.zeros(1, dtype=torch.int64, device="cuda")
    for W, (p, r) in zip(Ws, outs):
        wp, wr = qamw.encode(W, cb, bits, block, full_scans=scans)
        assert torch.equal(p, wp) and torch.equal(r, wr)


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [3, 7, 11, 12])
def test_pruned_call_with_scratch(bits):
    # the pruned entry point: with scratch, from the caller's table (which counts its scans), and over the whole codebook
    say(f"[cells] pruned B={bits}")
    host = _codebook(bits, "lloyd")
    cb, grid = torch.from_numpy(host).cuda(), torch.from_numpy(qamw.search_grid(host, bits)[0]).cuda()
    L = qamw.lib()
    for d_out, d_in, block, dtype in [(37, 1152, 128, "bf16"), (1200, 4096, 256, "f32"), (3, 192, 64, "bf16")]:
        W = synth.weight_device(d_in, d_out, d_in, 0.5, dtype)
        scans = torch.zeros(1, dtype=torch.int64, device="cuda")
        want = qamw.encode(W, cb, bits, block, full_scans=scans)
        for kw in ({}, {"full_scans": scans}):
            got = qamw.encode_pruned(W, cb, grid, bits, block, **kw)
            torch.cuda.synchronize()
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), kw
    # what was refused stays refused, with scratch or without
    W = synth.weight_device(1, 8, 96, 0.5, "f32")
    with pytest.raises(qamw.QamwError) as e:
        qamw.encode_pruned(W, cb, grid, bits, 32)
    assert e.value.status == qamw.ERR_UNSUPPORTED
    ptr = lambda t: C.c_void_p(t.data_ptr())
    args = (ptr(W), 0, 8, 96, 96, None, None, None, ptr(cb), bits, 32, ptr(grid))
    assert L.qamw_encode_pruned_ws(*args, C.c_void_p(cb.data_ptr() + 8), 1 << 20, ptr(W), ptr(W), None, None) != qamw.OK
