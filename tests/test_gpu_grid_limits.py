"""Row counts at which a launch geometry would need 2^32 threads and more in one dimension, which no launch takes: the
product goes another way.  Whole numbers, so that differences of running sums are exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def matrix(m, k, short, long, every):
    """Rows of `short` entries, every `every`-th one of `long`; columns and values follow from the position."""
    lens = torch.full((m,), short, dtype=torch.int32, device="cuda")
    lens[every // 2::every] = long
    rowptr = torch.zeros(m + 1, dtype=torch.int32, device="cuda")
    torch.cumsum(lens, 0, out=rowptr[1:])
    at = torch.arange(int(rowptr[-1]), device="cuda")
    return rowptr, (at * 7919 % k).to(torch.int32), (at % 5 - 2).float()


def product(rowptr, colind, vals, b):
    """A.b for one column of whole numbers."""
    sums = torch.zeros(colind.numel() + 1, dtype=torch.int64, device="cuda")
    torch.cumsum((vals * b[colind.long()]).long(), 0, out=sums[1:])
    return (sums[rowptr[1:].long()] - sums[rowptr[:-1].long()]).float()


# one wave to a row (PR; 64 lanes where an average entry lies in a row of more than 200): 2^26 rows are too many for one launch
@pytest.mark.parametrize("algo", ["RB+RM+SR", "RB+RM+PR", "RB+CM+SR", "RB+CM+PR", "EB+RM+SR", "EB+CM+PR"])
def test_rows_of_a_wave_each(algo):
    from paper_2202_08556_amd import binding as da
    m, k = (1 << 26) + 9, 5003
    rowptr, colind, vals = matrix(m, k, 2, 4000, 1 << 12)
    b = (torch.arange(k, device="cuda") % 9 - 4).float()
    da.da_spmm_features(m, 1, rowptr)
    C = torch.full((m,), float("nan"), device="cuda")
    print("rows", m, algo, flush=True)
    da.da_spmm(m, k, 1, rowptr, colind, vals, b, C, da.ALGO_NAMES.index(algo))
    assert torch.equal(C, product(rowptr, colind, vals, b))


# tiles on XCDs of their own put the blocks of both tiles into one dimension; with a layer's bias
@pytest.mark.parametrize("algo", ["RB+RM+PR"])
def test_rows_of_two_tiles(algo):
    from paper_2202_08556_amd import binding as da
    m, k, N = (1 << 25) + 9, 10007, 128
    rowptr, colind, vals = matrix(m, k, 0, 3, 1 << 12)
    B = (torch.arange(k * N, device="cuda") % 9 - 4).float().view(k, N)
    bias = (torch.arange(N, device="cuda") % 7 - 3).float()
    C = torch.full((m, N), float("nan"), device="cuda")
    print("rows", m, algo, flush=True)
    da.da_spmm_layer(m, k, N, rowptr, colind, vals, B, N, C, bias, False, da.ALGO_NAMES.index(algo))
    for n in (0, 63, 64, 127):
        assert torch.equal(C[:, n], product(rowptr, colind, vals, B[:, n].contiguous()) + bias[n])
    assert not torch.isnan(C.sum(1)).any()


# heavy rows on both sides of the first part's end: the other rows' kernel leaves them to the kernel of their own
def test_heavy_rows_of_both_parts():
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import kernels_of
    m, k, N, each = (1 << 27) + 4097, 20011, 17, 18000
    heavy = torch.cat([torch.arange(20) * 1000 + 3, m - 4 - torch.arange(20) * 100]).sort()[0].cuda()
    lens = torch.zeros(m, dtype=torch.int32, device="cuda")
    lens[heavy] = each
    rowptr = torch.zeros(m + 1, dtype=torch.int32, device="cuda")
    torch.cumsum(lens, 0, out=rowptr[1:])
    colind = (torch.arange(each, device="cuda")[None, :] + 50 * torch.arange(40, device="cuda")[:, None]).reshape(-1).to(torch.int32)
    vals = (torch.arange(40 * each, device="cuda") % 5 - 2).float()
    B = (torch.arange(k * N, device="cuda") % 9 - 4).float().view(k, N)
    da.da_spmm_prepare(m, k, colind.numel(), rowptr, colind)
    C = torch.full((m, N), float("nan"), device="cuda")
    print("rows", m, flush=True)
    names = kernels_of(lambda: da.da_spmm(m, k, N, rowptr, colind, vals, B, C, da.DA_EB_RM_SR))
    da.da_spmm_release(rowptr)
    assert any("heavy_rows_kernel" in n for n in names)
    want = torch.stack([(vals[i * each:(i + 1) * each, None] * B[colind[i * each:(i + 1) * each].long()]).sum(0) for i in range(40)])
    assert torch.equal(C[heavy], want)
    C[heavy] = 0.0
    assert not torch.isnan(C.sum(1)).any() and not C.any()
