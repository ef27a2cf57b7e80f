"""RB+RM+PR in tiles of 32 columns: long rows, uneven or of a wide matrix, with tiles on XCDs of their own and without."""
import numpy as np
import pytest
import torch

from oracle import reference as orc
from tests.gpu_util import kernels_of

pytestmark = pytest.mark.gpu


def matrix(m, k, even, seed):
    rng = np.random.default_rng(seed)
    lens = np.full(m, even) if even else np.where(np.arange(m) % 3 == 0, 300, 60)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    colind = rng.integers(0, k, size=int(rowptr[-1])).astype(np.int32)
    return rowptr, colind, rng.choice(np.array([-2, -1, 1, 2], np.float32), colind.size)


# two tiles, as many as XCDs, and numbers that are not pinned; B inside an L2 and beyond; even rows only of a wide matrix, and not
# where tiles of 64 are pinned
@pytest.mark.parametrize("m,k,even,N,narrow", [
    (301, 900, False, 64, True), (301, 900, False, 96, True), (301, 900, False, 256, True), (1000, 60_000, False, 128, True),
    (1000, 60_000, 130, 64, True), (1000, 20_000, 130, 192, True), (1000, 60_000, 60, 128, True), (301, 900, 130, 64, False),
    (1000, 20_000, 60, 64, False), (301, 900, False, 72, False), (301, 12_000, False, 128, False),
])
def test_tiles_of_32_columns(m, k, even, N, narrow):
    from paper_2202_08556_amd import binding as da
    rowptr, colind, vals = matrix(m, k, even, seed=N)
    B = np.random.default_rng(1).integers(-4, 5, (k, N)).astype(np.float32)
    want, _ = orc.spmm(rowptr, colind, vals, B)
    dev = [torch.from_numpy(x).cuda() for x in (rowptr, colind, vals, B)]
    print(f"tiles of 32 columns m={m} k={k} N={N} rows={even}", flush=True)
    da.da_spmm_features(m, N, dev[0])
    C = torch.full((m, N), float("nan"), device="cuda")
    names = kernels_of(lambda: da.da_spmm(m, k, N, *dev, C, da.DA_RB_RM_PR))
    assert np.array_equal(C.cpu().numpy(), want.astype(np.float32) + 0.0)
    assert any("rb_pr_kernel<4, 8," in n for n in names) == narrow, names


# a launch holds 65 535 tiles of columns: beyond 32 columns each, tiles of 64
@pytest.mark.parametrize("N,narrow", [(32 * 65535, True), (32 * 65537, False), (64 * 65535, False)])
def test_more_columns_than_tiles_of_32_reach(N, narrow):
    from paper_2202_08556_amd import binding as da
    m, k = 3, 16
    rowptr, colind, vals = matrix(m, k, False, seed=3)
    B = torch.from_numpy(np.random.default_rng(1).integers(-4, 5, (k, N)).astype(np.float32))
    a = torch.zeros((m, k), dtype=torch.float64)
    a.index_put_((torch.from_numpy(np.repeat(np.arange(m), np.diff(rowptr))), torch.from_numpy(colind).long()),
                 torch.from_numpy(vals).double(), accumulate=True)
    dev = [torch.from_numpy(x).cuda() for x in (rowptr, colind, vals)]
    print(f"tiles of 32 columns N={N}", flush=True)
    da.da_spmm_features(m, N, dev[0])
    C = torch.full((m, N), float("nan"), device="cuda")
    names = kernels_of(lambda: da.da_spmm(m, k, N, *dev, B.cuda(), C, da.DA_RB_RM_PR))
    assert torch.equal(C.cpu(), (a @ B.double()).float() + 0.0)
    assert any("rb_pr_kernel<4, 8," in n for n in names) == narrow, names


# many rows of a B that an L2 holds take tiles of 64, however uneven, and few rows tiles of 32; beyond an L2 the length of the rows decides
@pytest.mark.parametrize("m,k,lens,N,narrow", [
    (9000, 5000, (10, 100), 64, True), (60_000, 5000, (10, 100), 64, False), (60_000, 14_000, (10, 100), 64, False),
    (60_000, 14_000, (10, 100), 128, False), (60_000, 70_000, (20, 100), 64, True), (60_000, 20_000, (10, 100), 64, False),
    (2000, 170_000, (60, 80), 96, False), (2000, 170_000, (60, 80), 64, True), (2000, 240_000, (60, 80), 64, False),
])
def test_tiles_by_rows_and_columns(m, k, lens, N, narrow):
    from paper_2202_08556_amd import binding as da
    dev = torch.device("cuda:0")
    lens = torch.where(torch.arange(m, device=dev) % 3 == 0, lens[1], lens[0])
    rowptr = torch.zeros(m + 1, dtype=torch.int32, device=dev)
    torch.cumsum(lens, 0, out=rowptr[1:])
    at = torch.arange(int(rowptr[-1]), device=dev)
    colind, vals = (at * 7919 % k).to(torch.int32), (at % 5 - 2).float()
    B = (torch.arange(k * N, device=dev) % 9 - 4).float().view(k, N)
    print(f"tiles m={m} k={k} N={N}", flush=True)
    da.da_spmm_features(m, N, rowptr)
    C = torch.full((m, N), float("nan"), device=dev)
    names = kernels_of(lambda: da.da_spmm(m, k, N, rowptr, colind, vals, B, C, da.DA_RB_RM_PR))
    assert any("rb_pr_kernel<4, 8," in n for n in names) == narrow, names
    for n in (0, 31, 32, N - 1):                              # whole numbers: running sums are exact
        sums = torch.zeros(at.numel() + 1, dtype=torch.int64, device=dev)
        torch.cumsum((vals * B[:, n][colind.long()]).long(), 0, out=sums[1:])
        assert torch.equal(C[:, n], (sums[rowptr[1:].long()] - sums[rowptr[:-1].long()]).float())
    assert not torch.isnan(C.sum(1)).any()
