"""da_csr_transpose at the edges of its tiles and passes, bit for bit against the oracle's stable sort."""
import numpy as np
import pytest
import torch

from oracle import reference as orc

pytestmark = pytest.mark.gpu


def matrix(m, k, nnz, kind, seed):
    """Row pointers and unsorted, repeating columns: 'even' rows, 'gaps' (nearly all rows empty, in long
    runs), or 'column' (nine tenths of the entries in one column)."""
    rng = np.random.default_rng(seed)
    if kind == "gaps":
        rows = np.sort(rng.choice(m, size=max(1, m // 5000), replace=False))
        r = np.sort(rng.choice(rows, size=nnz))
    else:
        r = np.sort(rng.integers(0, m, size=nnz))
    rowptr = np.zeros(m + 1, dtype=np.int32)
    rowptr[1:] = np.cumsum(np.bincount(r, minlength=m))
    colind = rng.integers(0, k, size=nnz).astype(np.int32)
    if kind == "column":
        colind[rng.random(nnz) < 0.9] = k - 1
    return rowptr, colind, rng.standard_normal(nnz).astype(np.float32)


CASES = [  # around the tile sizes 1024 and 2048, ranges of several tiles; one pass, two passes, general sort
    (7, 1, 1, "even"), (50, 16, 1023, "even"), (50, 1024, 1024, "even"), (60, 1025, 1025, "column"),
    (3000, 65536, 20001, "even"), (40000, 5000, 12345, "gaps"), (1, 300000, 5000, "even"),
    (1000, 1 << 20, 1024 * 1024 - 1, "even"), (70001, 262144, 1024 * 1024 + 1, "column"),
    (5000, 3000, 4096 * 1024 - 1, "even"), (2_000_000, 1000, 4096 * 1024, "gaps"), (100_000, 262145, 4_300_000, "even"),
    (1 << 22, 1 << 20, 30_000, "even"), ((1 << 22) + 1, 1 << 20, 30_000, "even"), (500, (1 << 20) + 1, 30_000, "even"),
]


@pytest.mark.parametrize("m,k,nnz,kind", CASES)
def test_transpose_edges(m, k, nnz, kind):
    from paper_2202_08556_amd import binding as da
    print(f"transpose m={m} k={k} nnz={nnz} {kind}", flush=True)
    rowptr, colind, vals = matrix(m, k, nnz, kind, seed=nnz)
    dev = torch.device("cuda:0")
    rp, ci, va = (torch.from_numpy(x).to(dev) for x in (rowptr, colind, vals))
    size = da.da_csr_transpose_workspace(m, k, nnz)
    ws = torch.full((size,), 0xA5, dtype=torch.uint8, device=dev)
    want = orc.csr_transpose(rowptr, colind, vals, k)
    for _ in range(2):                                       # again on the used workspace
        out = (torch.full((k + 1,), -7, dtype=torch.int32, device=dev), torch.full((nnz,), -7, dtype=torch.int32, device=dev),
               torch.full((nnz,), float("nan"), device=dev))
        da.da_csr_transpose(m, k, nnz, rp, ci, va, *out, ws, size)
        torch.cuda.synchronize()
        for g, w in zip(out, want):
            assert np.array_equal(g.cpu().numpy().view(np.uint32), np.ascontiguousarray(w).view(np.uint32))


def test_entries_beyond_32_bit_offsets():
    """2^30 entries and a few: byte offsets of entries no longer fit 32 bits."""
    from paper_2202_08556_amd import binding as da
    m, each, dev = (1 << 20) + 5, 1024, torch.device("cuda:0")
    k, nnz = each * 1024, m * each
    print(f"transpose m={m} k={k} nnz={nnz}", flush=True)
    r, i = torch.arange(m, dtype=torch.int32, device=dev)[:, None], torch.arange(each, dtype=torch.int32, device=dev)[None, :]
    rp = torch.arange(m + 1, dtype=torch.int32, device=dev) * each
    ci = (i * 1024 + r * 7 % 1024).view(-1)                  # entry i of row r: column 1024 i + 7 r mod 1024
    va = ((r * 31 + i) % 1000).to(torch.float32).view(-1)
    size = da.da_csr_transpose_workspace(m, k, nnz)
    ws = torch.empty(size, dtype=torch.uint8, device=dev)
    out = (torch.empty(k + 1, dtype=torch.int32, device=dev), torch.empty_like(ci), torch.empty_like(va))
    da.da_csr_transpose(m, k, nnz, rp, ci, va, *out, ws, size)
    del ws
    # every 1024 neighbouring columns hold all rows once, ordered by 7 r mod 1024 and then by r
    rows = torch.arange(m, dtype=torch.int64, device=dev)
    order = torch.sort(rows * 7 % 1024 * m + rows)[1]
    first = torch.cumsum(torch.bincount(rows * 7 % 1024, minlength=1024), 0)
    assert int(out[0][0]) == 0
    for i in range(each):
        part = slice(i * m, (i + 1) * m)
        assert torch.equal(out[0][i * 1024 + 1:(i + 1) * 1024 + 1].long(), first + i * m)
        assert torch.equal(out[1][part].long(), order)
        assert torch.equal(out[2][part], ((order * 31 + i) % 1000).float())
