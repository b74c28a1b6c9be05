"""Pairs whose y = t / sqrt(block) is below the smallest normal number and is rounded there before the gain multiplies it: where
1 / sqrt(block) is a power of two, one multiplication by its product with the gain would leave that rounding out.  Weights so small
beside their row's norm, and pair scales that make up for it."""
import pytest
import torch

from paper_2605_26339_amd import qamw

pytestmark = pytest.mark.gpu


def _row(block, d_in, a, b):
    """A row of norm 1 whose second block's pairs rotate to (a + b, a - b) and (-(a + b), b - a)."""
    W = torch.zeros((1, d_in), dtype=torch.float64)
    W[0, 0] = 1.0
    W[0, block + 2], W[0, block + 3] = a, b
    return W.float().cuda()


def _fields(packed, bits, n):
    stream = (packed[..., None] >> torch.arange(8, device="cuda", dtype=torch.uint8)) & 1
    return (stream.reshape(packed.shape[0], -1)[:, : n * bits].view(packed.shape[0], n, bits).long() << torch.arange(bits, device="cuda")).sum(-1)


# workgroups of one row (binary searches) and of twelve (lookup tables)
@pytest.mark.parametrize("block", [64, 256, 1024])
@pytest.mark.parametrize("rows", [1, 6000])
def test_polar_phase_of_a_rounded_pair(block, rows):
    print(f"[unit gains] polar {block} rows {rows}", flush=True)
    d_in, bits_a, bits_p = 4096, 3, 6
    # t = +-(sqrt(block) 2^-130, -2 units in the last place): the y of the latter rounds to 0, the pair lies on the axis
    W = _row(block, d_in, block ** 0.5 * 2.0 ** -131 - 2.0 ** -149, block ** 0.5 * 2.0 ** -131 + 2.0 ** -149)
    sigma = torch.full((d_in // 2,), 2.0 ** -126, device="cuda")
    levels = torch.from_numpy(qamw.polar_codebook(bits_a, bits_p)[0]).cuda()
    pairs, _ = qamw.normalised_pairs(W, block, pair_sigma=sigma)
    packed, _ = qamw.encode_polar(W.repeat(rows, 1), levels, bits_a, bits_p, block, pair_sigma=sigma)
    torch.cuda.synchronize()
    own = slice(block // 2, block)
    x = pairs[:, own]
    assert bool((x[..., 0].abs() == 2.0 ** -4).all()) and bool((x[..., 1] == 0).all())
    assert bool((x[..., 0] < 0).any()) and bool((x[..., 0] > 0).any())
    want = torch.where(x[..., 0] > 0, 0, 1 << (bits_p - 1)).expand(rows, -1)
    assert torch.equal(_fields(packed, bits_a + bits_p, d_in // 2)[:, own] & ((1 << bits_p) - 1), want)


@pytest.mark.parametrize("block", [64, 256, 1024])
@pytest.mark.parametrize("rows", [1, 6000])
def test_polar_phase_of_a_pair_rounded_to_an_axis(block, rows):
    """One coordinate far above the smallest normal number, the y of the other rounded to 0: with gains as usual, the pair is on the axis."""
    print(f"[unit gains] polar axis {block} rows {rows}", flush=True)
    d_in, bits_a, bits_p = 4096, 3, 6
    levels = torch.from_numpy(qamw.polar_codebook(bits_a, bits_p)[0]).cuda()
    own = slice(block // 2, block)
    for tiny in (2.0 ** -149, -2.0 ** -149):
        W = _row(block, d_in, tiny, -tiny)                      # (0, 2 tiny) after the first butterfly, y at most 2^-151
        W[0, block + 4:block + 6] = 2.0 ** -30                  # (2^-29, 0)
        pairs, _ = qamw.normalised_pairs(W, block)
        packed, _ = qamw.encode_polar(W.repeat(rows, 1), levels, bits_a, bits_p, block)
        torch.cuda.synchronize()
        x = pairs[:, own]
        assert bool((x[..., 0].abs() == 2.0 ** -29 * (d_in / block) ** 0.5).all()) and bool((x[..., 1] == 0).all())
        assert bool((x[..., 0] < 0).any()) and bool((x[..., 0] > 0).any())
        want = torch.where(x[..., 0] > 0, 0, 1 << (bits_p - 1)).expand(rows, -1)
        assert torch.equal(_fields(packed, bits_a + bits_p, d_in // 2)[:, own] & ((1 << bits_p) - 1), want)


# records from memory and from LDS, norms from a launch ahead and inside the search
@pytest.mark.parametrize("block", [64, 256, 1024])
@pytest.mark.parametrize("bits", [7, 10, 11])
@pytest.mark.parametrize("rows", [300, 6000, 13000])
def test_nearest_codeword_of_a_rounded_pair(block, bits, rows):
    """The pairs lie half way between a codeword and its mirror image, where the lower index counts, or beside that by what is rounded."""
    print(f"[unit gains] cells {block} bits {bits} rows {rows}", flush=True)
    d_in = 4096
    W = _row(block, d_in, block ** 0.5 * 2.0 ** -131 - 2.0 ** -149, block ** 0.5 * 2.0 ** -131 + 2.0 ** -149).repeat(rows, 1)
    sigma = torch.full((d_in // 2,), 2.0 ** -126, device="cuda")
    cb = torch.from_numpy(qamw.train_codebook(bits, 1 << 15, max_iters=20)[0]).cuda()
    cb[::2, 1] = cb[::2, 1].abs()
    cb[1::2] = cb[::2] * torch.tensor([1.0, -1.0], device="cuda")
    scans = torch.zeros(1, dtype=torch.int64, device="cuda")
    want, _ = qamw.encode(W, cb, bits, block, pair_sigma=sigma, full_scans=scans)
    got, _ = qamw.encode(W, cb, bits, block, pair_sigma=sigma)
    torch.cuda.synchronize()
    assert not bool((_fields(want, bits, d_in // 2)[:, block // 2:block] & 1).any())
    assert torch.equal(got, want)
