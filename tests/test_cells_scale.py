"""The cell table at other scales, and rows that it does not help: the bytes of the search over the whole codebook, and no
more time than at the unit scale where the table follows the codebook."""
import sys

import numpy as np
import pytest
import torch

from paper_2605_26339_amd import qamw

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _book(bits, scale=1.0):
    return torch.from_numpy(qamw.train_codebook(bits, 1 << 14, max_iters=10)[0]).cuda() * scale


def _matrix(d_out, d_in, dtype=torch.bfloat16, seed=0):
    g = torch.Generator("cuda").manual_seed(seed)
    return torch.randn(d_out, d_in, device="cuda", generator=g).to(dtype)


def _sigma(d_in, scale):
    """Pair scales that give pairs of `scale` times the unit variance."""
    return torch.full((d_in // 2,), 1.0 / (d_in ** 0.5 * scale), device="cuda")


def _check(W, cb, bits, block, sigma, grid=None):
    scans = torch.zeros(1, dtype=torch.int64, device="cuda")
    want = qamw.encode(W, cb, bits, block, pair_sigma=sigma, full_scans=scans)
    got = qamw.encode(W, cb, bits, block, pair_sigma=sigma)
    torch.cuda.synchronize()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    if grid is not None:
        got = qamw.encode_pruned(W, cb, grid, bits, block, pair_sigma=sigma)
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0])


# codebook and pairs together from the smallest normal numbers to beyond the range of a squared distance
@pytest.mark.parametrize("bits", [1, 3, 5, 6, 9, 10, 11])
def test_codebook_and_pairs_at_every_scale(bits):
    W = _matrix(520, 2048)
    for scale in (1e-25, 1e-12, 1e-4, 1 / 16, 0.5, 0.7, 1.5, 4.0, 64.0, 1e5, 1e12, 1e19, 1e25):
        say(f"[cells scale] B={bits} x {scale}")
        _check(W, _book(bits, scale), bits, 128, _sigma(2048, scale))


# The half-width that the table's first record holds: 4 for Lloyd codebooks of the unit Gaussian however they were trained (with
# 3.75 the pairs of weights with outlier channels stand outside the square half as often again), in proportion for others.
@pytest.mark.parametrize("bits", [7, 8, 9, 10, 11])
@pytest.mark.parametrize("samples,iters", [(1 << 14, 10), (1 << 17, 30), (1 << 20, 40)])
def test_the_square_of_a_trained_codebook(bits, samples, iters):
    cb = torch.from_numpy(qamw.train_codebook(bits, max(samples, 8 << bits), max_iters=iters)[0]).cuda()
    W = _matrix(1024, 1024)
    ws = torch.zeros(qamw.encode_workspace_bytes(bits), dtype=torch.uint8, device="cuda")
    packed = torch.empty((1024, qamw.packed_row_bytes(1024, bits)), dtype=torch.uint8, device="cuda")
    norms = torch.empty(1024, device="cuda")
    for scale in (1.0, 8.0):
        book = cb * scale
        qamw._check(qamw.lib().qamw_encode_ws(W.data_ptr(), qamw._dtype_code(W), 1024, 1024, 1024, None, None, None, book.data_ptr(),
                                              bits, 128, ws.data_ptr(), ws.numel(), packed.data_ptr(), norms.data_ptr(),
                                              qamw._stream(None)), "qamw_encode_ws")
        torch.cuda.synchronize()
        first = int(ws[:4].cpu().numpy().view(np.uint32)[0])
        assert np.array([(first >> 3) << 20], dtype=np.uint32).view(np.float32)[0] == 4.0 * scale


# pairs wider or narrower than the codebook, so that anything from none to all of a row's pairs is undecided by the table; both
# sides of "a few are scanned one by one"; the two element types, blocks that need more registers, ragged slabs, few lanes
@pytest.mark.parametrize("bits", [3, 5, 6, 7, 9, 10, 11])
@pytest.mark.parametrize("d_out,d_in,block,dtype", [(4200, 1024, 128, torch.bfloat16), (530, 5632, 512, torch.float32),
                                                    (1030, 2048, 1024, torch.bfloat16), (300, 11008, 256, torch.bfloat16),
                                                    (2000, 192, 64, torch.float32), (3, 1088, 64, torch.bfloat16)])
def test_pairs_that_the_table_does_not_decide(bits, d_out, d_in, block, dtype):
    host = _book(bits)
    grid = torch.from_numpy(qamw.search_grid(host.cpu().numpy(), bits)[0]).cuda()
    W = _matrix(d_out, d_in, dtype, seed=bits)
    W[d_out // 3] = 0
    for width in (0.02, 1.3, 1.6, 2.0, 3.0, 8.0):
        say(f"[cells wide] B={bits} {d_out}x{d_in} b={block} {dtype} pairs x {width}")
        _check(W, host, bits, block, _sigma(d_in, width), grid)
    # some columns wide, the others not; rows of each kind among the others
    sigma = _sigma(d_in, 1.0)
    sigma[: max(8, d_in // 16)] *= 0.1
    heavy = torch.from_numpy(np.random.default_rng(bits).standard_t(1.2, (40, d_in)).astype(np.float32)).cuda().to(dtype)
    W[5:45][: max(0, min(40, d_out - 5))] = heavy[: max(0, min(40, d_out - 5))]
    _check(W, host, bits, block, sigma, grid)
    rnd = torch.randn(1 << bits, 2, device="cuda", generator=torch.Generator("cuda").manual_seed(bits))
    _check(W, rnd, bits, block, _sigma(d_in, 1.0), torch.from_numpy(qamw.search_grid(rnd.cpu().numpy(), bits)[0]).cuda())


def test_more_rows_than_a_wave_can_put_off():
    # 256 items per wave can be put off; one more of each is scanned in place
    say("[cells] 1060000 x 1024, all pairs beyond the table")
    bits, d_in, d_out = 6, 1024, 1060000
    W = torch.cat([_matrix(106000, d_in, seed=i) for i in range(10)])
    cb, sigma = _book(bits), _sigma(d_in, 4.0)
    a = qamw.encode(W, cb, bits, 128, pair_sigma=sigma)
    for lo in (0, d_out - 70000):                             # the first rows, and the last, which exceed what a wave notes
        b = qamw.encode(W[lo:lo + 70000], cb, bits, 128, pair_sigma=sigma, full_scans=torch.zeros(1, dtype=torch.int64, device="cuda"))
        torch.cuda.synchronize()
        assert torch.equal(a[0][lo:lo + 70000], b[0]) and torch.equal(a[1][lo:lo + 70000], b[1])


def _time(f):
    f()
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(5):
            f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


# Five codebooks of one shape are five equal pieces of work.  With a square that does not follow them a codebook 16 times smaller
# took 6 to 70 times as long (it falls into a few cells, every pair is scanned).
@pytest.mark.parametrize("what", ["encode", "encode_pruned", "lloyd_device"])
def test_no_scale_is_slow(what):
    bits = 11
    W = _matrix(2048, 4096)
    took = {}
    for scale in (1.0, 0.003, 1 / 16, 3.0, 40.0):             # (the trainer's sums clamp coordinates beyond 256)
        cb, sigma = _book(bits, scale), _sigma(4096, scale)
        if what == "lloyd_device":
            x = torch.randn(1 << 18, 2, device="cuda") * scale
            took[scale] = _time(lambda: qamw.lloyd_device(x, cb, bits, max_iters=8, tol=0.0))
        elif what == "encode":
            took[scale] = _time(lambda: qamw.encode(W, cb, bits, 128, pair_sigma=sigma))
        else:
            grid = torch.from_numpy(qamw.search_grid(cb.cpu().numpy(), bits)[0]).cuda()
            took[scale] = _time(lambda: qamw.encode_pruned(W, cb, grid, bits, 128, pair_sigma=sigma))
        say(f"[cells scale] {what} x {scale}: {took[scale]:.2f}")
    assert max(took.values()) < 2.0 * took[1.0]


# Pairs that no table helps cost about what the search over the whole codebook does (1.0 to 1.3 times; 15 times and more when
# they are scanned one after the other at few codewords).
@pytest.mark.parametrize("bits", [5, 7, 11])
def test_undecided_pairs_cost_no_more_than_the_whole_search(bits):
    W, cb, sigma = _matrix(4096, 4096), _book(bits), _sigma(4096, 3.0)
    scans = torch.zeros(1, dtype=torch.int64, device="cuda")
    table = _time(lambda: qamw.encode(W, cb, bits, 128, pair_sigma=sigma))
    whole = _time(lambda: qamw.encode(W, cb, bits, 128, pair_sigma=sigma, full_scans=scans))
    say(f"[cells wide] B={bits}: table {table:.2f}, whole codebook {whole:.2f}")
    assert table < 1.6 * whole


# Codewords that no Lloyd iteration has spread: the caller's table, with smaller cells and more candidates, decides most of what
# the device's does not, so scratch makes the pruned call no slower (1.7 and 5.1 times as long when that table was not read).
@pytest.mark.parametrize("kind", ["as_drawn", "clustered"])
def test_pruned_call_reads_the_callers_table(kind):
    bits, d_out, d_in, block = 11, 4096, 4096, 128
    rng = np.random.default_rng(3)
    host = rng.standard_normal((1 << bits, 2)).astype(np.float32)
    if kind == "clustered":
        host[512:] = 0.5 + 1e-4 * host[512:]
    cb, grid = torch.from_numpy(host).cuda(), torch.from_numpy(qamw.search_grid(host, bits)[0]).cuda()
    W, sigma = _matrix(d_out, d_in), _sigma(d_in, 1.0)
    packed, norms = qamw.encode_pruned(W, cb, grid, bits, block, pair_sigma=sigma)
    other = torch.empty_like(packed)

    def without_scratch():
        assert qamw.lib().qamw_encode_pruned(W.data_ptr(), 1, d_out, d_in, d_in, None, None, sigma.data_ptr(), cb.data_ptr(), bits, block,
                                             grid.data_ptr(), other.data_ptr(), norms.data_ptr(), None, None) == qamw.OK
    without = _time(without_scratch)
    with_it = _time(lambda: qamw.encode_pruned(W, cb, grid, bits, block, pair_sigma=sigma, out=(packed, norms)))
    say(f"[pruned] {kind}: with scratch {with_it:.2f}, without {without:.2f}")
    assert torch.equal(packed, other) and with_it < 1.3 * without


# samples and points of different scales, as an iteration's points drift
@pytest.mark.parametrize("bits,n", [(6, 5000), (9, 20000), (11, 30000)])
def test_lloyd_with_samples_of_another_scale(bits, n):
    say(f"[lloyd scale] B={bits} n={n}")
    import ctypes as C
    for width, scale in ((4.0, 1.0), (0.02, 1.0), (1.0, 1e-6), (1.0, 1e6), (100.0, 1.0)):
        x = torch.randn(n, 2, device="cuda", generator=torch.Generator("cuda").manual_seed(n)) * (width * scale)
        init = _book(bits, scale)
        got, mse, it = qamw.lloyd_device(x, init, bits, max_iters=5, tol=0.0)
        want, ws = init.clone(), torch.empty((1 << bits) * 40 + 64, dtype=torch.uint8, device="cuda")
        w_mse = C.c_double()
        assert qamw.lib().qamw_lloyd_device(x.data_ptr(), n, bits, want.data_ptr(), 5, 0.0, ws.data_ptr(), ws.numel(), C.byref(w_mse),
                                            None, None) == qamw.OK
        assert torch.equal(got, want) and it == 5
