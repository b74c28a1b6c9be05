"""Calls that name a stream: the memory the binding makes for them belongs to that stream."""
import contextlib
import sys
import types

import pytest
import torch

from paper_2605_26339_amd import qamw, synth

D_IN, D_OUT, BITS, BLOCK, M = 512, 24, 11, 128, 100


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _calls(dev, out):
    """name -> call(stream): every entry point of the binding that allocates, with and without the caller's outputs."""
    W = torch.randn(D_OUT, D_IN, device=dev)
    cb = torch.randn(1 << BITS, 2, device=dev)
    grid = torch.zeros(qamw.search_grid_size(BITS)[1], dtype=torch.uint8, device=dev) if dev == "cpu" else \
        torch.from_numpy(qamw.search_grid(cb.cpu().numpy(), BITS)[0]).to(dev)
    levels = torch.from_numpy(qamw.polar_codebook(5, 6)[0]).to(dev)
    X = torch.randn(M, D_IN, device=dev)
    packed, norms = out
    code = torch.randint(0, 256, (D_OUT, qamw.packed_row_bytes(D_IN, BITS)), dtype=torch.uint8, device=dev)
    rows = torch.rand(D_OUT, device=dev) + 0.5
    enc = qamw.make_encode_items([(W, None, None, None, packed, norms)])
    samples = torch.randn(4096, 2, device=dev)
    return {
        "encode": lambda st: qamw.encode(W, cb, BITS, BLOCK, stream=st),
        "encode, outputs given": lambda st: qamw.encode(W, cb, BITS, BLOCK, out=out, stream=st),
        "encode_batch": lambda st: (qamw.encode_batch(enc, cb, BITS, BLOCK, stream=st), out)[1],
        "encode_pruned, outputs given": lambda st: qamw.encode_pruned(W, cb, grid, BITS, BLOCK, out=out, stream=st),
        "encode_polar": lambda st: qamw.encode_polar(W, levels, 5, 6, BLOCK, stream=st),
        "normalised_pairs": lambda st: qamw.normalised_pairs(W, BLOCK, stream=st),
        "calibrate_sigma": lambda st: qamw.calibrate_sigma(W, BLOCK, stream=st),
        "decode": lambda st: qamw.decode(code, rows, D_IN, cb, BITS, BLOCK, stream=st),
        "matmul": lambda st: qamw.matmul(X, code, rows, cb, BITS, BLOCK, stream=st),
        "lloyd_device": lambda st: qamw.lloyd_device(samples, cb, BITS, max_iters=2, tol=0.0, stream=st)[0],
    }


def _outputs(dev):
    return (torch.empty((D_OUT, qamw.packed_row_bytes(D_IN, BITS)), dtype=torch.uint8, device=dev), torch.empty(D_OUT, device=dev))


def test_memory_is_allocated_and_copied_on_the_stream_of_the_call(monkeypatch):
    """Without a GPU: torch's stream functions replaced by ones that keep note of the current stream, the library's device
    entry points by ones that accept everything."""
    L = qamw.lib()
    monkeypatch.setattr(qamw, "_require_cuda", lambda *t: None)
    calls = _calls("cpu", _outputs("cpu"))
    main, side = types.SimpleNamespace(cuda_stream=1), types.SimpleNamespace(cuda_stream=2)
    current, made, copied, recorded = [main], [], [], []

    @contextlib.contextmanager
    def use(stream):
        current.append(stream if stream is not None else current[-1])
        yield
        current.pop()
    real_empty, real_copy = torch.empty, torch.Tensor.copy_

    def empty(*a, **kw):
        made.append(current[-1])
        return real_empty(*a, **kw)

    def copy_(self, src):
        copied.append(current[-1])
        return real_copy(self, src)
    fake = types.SimpleNamespace(**{n: getattr(L, n) if n.endswith(("_bytes", "_size")) else (lambda *a: qamw.OK) for n in qamw.EXPORTS})
    monkeypatch.setattr(qamw, "lib", lambda: fake)
    monkeypatch.setattr(torch, "empty", empty)
    monkeypatch.setattr(torch.cuda, "stream", use)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: current[-1])
    monkeypatch.setattr(torch.cuda, "ExternalStream", lambda ptr, device=None: side if ptr == 2 else main)
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda self, s: recorded.append(s), raising=False)
    monkeypatch.setattr(torch.Tensor, "copy_", copy_)
    for name, call in calls.items():
        made.clear(), copied.clear(), recorded.clear()
        call(side)
        assert made and all(s is side for s in made), name
        assert all(s is side for s in copied) and (name != "lloyd_device" or copied), name
        assert len(recorded) == len(made) and all(s is main for s in recorded), name
        made.clear(), recorded.clear()
        call(main)                                             # the current stream, named: nothing to record
        assert made and all(s is main for s in made) and not recorded, name


def test_calls_make_do_with_the_least_scratch(monkeypatch):
    """Where the card has no room for the scratch that makes a call fast it takes the least, as it always did; what the least does
    not fit either is refused."""
    L = qamw.lib()
    monkeypatch.setattr(qamw, "_require_cuda", lambda *t: None)
    calls = _calls("cpu", _outputs("cpu"))
    asked, room, real_empty = [], 0, torch.empty

    def empty(shape, **kw):
        if kw.get("dtype") == torch.uint8 and isinstance(shape, int):
            if shape > room:
                raise torch.cuda.OutOfMemoryError("no room")
            asked.append(shape)
        return real_empty(shape, **kw)
    given = {}
    fake = types.SimpleNamespace(**{n: getattr(L, n) if n.endswith(("_bytes", "_size")) else
                                    (lambda *a, n=n: (given.__setitem__(n, a), qamw.OK)[1]) for n in qamw.EXPORTS})
    monkeypatch.setattr(qamw, "lib", lambda: fake)
    monkeypatch.setattr(torch, "empty", empty)
    monkeypatch.setattr(qamw, "_stream", lambda s: 0)
    calls["encode, outputs given"](None)
    calls["encode_pruned, outputs given"](None)
    calls["encode_batch"](None)
    assert not asked and given["qamw_encode_ws"][11:13] == (None, 0) and given["qamw_encode_pruned_ws"][12:14] == (None, 0)
    assert given["qamw_encode_batch_ws"][6:8] == (None, 0)
    for name, entry, at, least in (("matmul", "qamw_matmul", 15, qamw.matmul_workspace_bytes(D_IN, D_OUT, M)),
                                   ("lloyd_device", "qamw_lloyd_device", 7, (40 << BITS) + 64)):
        asked.clear()
        room = least - 1
        with pytest.raises(torch.cuda.OutOfMemoryError):
            calls[name](None)
        room = least
        calls[name](None)
        assert asked == [least] and given[entry][at] == least, name
        room = 1 << 40
        asked.clear()
        calls[name](None)
        assert asked[0] > least and given[entry][at] == asked[0], name


@pytest.mark.gpu
def test_scratch_is_not_memory_that_the_current_stream_still_writes():
    """Blocks of the sizes the calls ask for, freed on the current stream behind long work that ends by writing them, must not
    reach a call on another stream."""
    out = _outputs("cuda")
    calls = _calls("cuda", out)
    want = {}
    for name, call in calls.items():
        got = call(None)
        torch.cuda.synchronize()
        want[name] = [t.clone() for t in (got if isinstance(got, tuple) else (got,))]
    big = torch.randn(4096, 4096, device="cuda")
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    for name, call in calls.items():
        say(f"[streams] {name}")
        sizes = [qamw.encode_workspace_bytes(BITS), qamw.calibrate_workspace_bytes(D_IN, D_OUT), (M + 31) // 32 * 32 * D_IN * 2,
                 D_OUT * D_IN * 4, D_OUT * D_IN * 2, D_OUT * 4, (8 << BITS), M * D_OUT * 4, D_OUT * qamw.packed_row_bytes(D_IN, BITS)]
        blocks = [torch.zeros(n, dtype=torch.uint8, device="cuda") for n in sizes for _ in range(2)]
        torch.cuda.synchronize()
        for _ in range(20):
            big = torch.mm(big, big).mul_(1e-2)
        for b in blocks:
            b.fill_(0x5A)
        del b, blocks
        got = call(st)
        torch.cuda.synchronize()
        for g, w in zip(got if isinstance(got, tuple) else (got,), want[name]):
            assert torch.equal(g, w), name
