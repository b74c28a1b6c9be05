"""The polar encoder's lookup tables (large launches) against its binary searches (small ones): the same packed bytes for the same
rows, over numbers of levels and bins on either side of what the tables take, levels that are crowded, unsorted, tiny or huge,
and pairs that are zero, on an axis or beyond the tables' range."""
import pytest
import torch

from paper_2605_26339_amd import qamw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits_a,bits_p", [(0, 3), (1, 2), (3, 3), (5, 6), (6, 5), (2, 8), (3, 9), (4, 0), (4, 1)])
@pytest.mark.parametrize("kind", ["lloyd", "crowded", "unsorted", "tiny", "huge"])
def test_tables_and_searches_agree(bits_a, bits_p, kind):
    print(f"[polar lookup] {bits_a}+{bits_p} {kind}", flush=True)
    levels = torch.from_numpy(qamw.polar_codebook(bits_a, bits_p)[0]).cuda()
    if kind == "crowded":
        levels = 1.0 + 1e-3 * levels                            # several thresholds in a cell
    elif kind == "unsorted":
        levels = levels.flip(0).contiguous()
    elif kind != "lloyd":
        levels = levels * (1e-6 if kind == "tiny" else 1e4)
    d_out, d_in, block = 9000, 1024, 64                         # 16 rows of one slab per workgroup
    g = torch.Generator("cuda").manual_seed(bits_a * 16 + bits_p)
    W = torch.randn(d_out, d_in, device="cuda", generator=g)
    W[1] = 0
    W[2, :] = 0
    W[2, 5] = 1.0                                               # every coefficient of one block the same magnitude: on the diagonals
    W[3, 64:] = 0
    W[3, 1:64] = 0                                              # a constant block and zero blocks
    sigma = torch.full((d_in // 2,), 1.0 / 32, device="cuda")
    sigma[:32] = 1e-20                                          # squares beyond the tables' range
    sigma[32:64] = 1e20
    full, norms = qamw.encode_polar(W, levels, bits_a, bits_p, block, pair_sigma=sigma)
    for r in range(0, d_out, 500):                              # 8 rows per workgroup
        part, n = qamw.encode_polar(W[r:r + 500], levels, bits_a, bits_p, block, pair_sigma=sigma)
        assert torch.equal(full[r:r + 500], part) and torch.equal(norms[r:r + 500], n)


@pytest.mark.parametrize("bits_a,bits_p,dtype", [(5, 6, torch.bfloat16), (3, 8, torch.float32)])
def test_shared_rows_with_and_without_tables(bits_a, bits_p, dtype):
    # 65 slabs: 128 rows are shared by four workgroups each, 16 or 17 items and tables; 100 rows by five, 13 and searches; 16 rows by
    # nine, 7 or 8; 600 rows are not shared, 65 items and tables
    print(f"[polar lookup] shared rows {bits_a}+{bits_p} {dtype}", flush=True)
    levels = torch.from_numpy(qamw.polar_codebook(bits_a, bits_p)[0]).cuda()
    W = torch.randn(600, 65 * 1024, device="cuda", generator=torch.Generator("cuda").manual_seed(bits_p)).to(dtype)
    W[3, :2048] = 0
    want, norms = qamw.encode_polar(W, levels, bits_a, bits_p, 1024)
    for lo, n in ((0, 128), (0, 100), (1, 16), (472, 128)):
        got, r = qamw.encode_polar(W[lo:lo + n], levels, bits_a, bits_p, 1024)
        torch.cuda.synchronize()
        assert torch.equal(got, want[lo:lo + n]) and torch.equal(r, norms[lo:lo + n]), (lo, n)
