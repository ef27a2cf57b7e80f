"""Column-major B under the RB ids (rb_columns_kernel): lanes per row by what is known of the matrix, column tiles, last
rows, and values that must not leak from lanes without an entry.  Integer values: any order gives the same bits."""
import numpy as np
import pytest
import torch

from oracle import reference as orc
from paper_2202_08556_amd import generators as gen

pytestmark = pytest.mark.gpu

MATRICES = {"short": lambda: gen.uniform_csr(m=1003, k=777, mean_len=3.0, seed=1),               # 4 lanes
            "stencil": lambda: gen.stencil27_csr(nx=9, ny=7, nz=5, seed=2),                      # 8
            "longer": lambda: gen.lognormal_csr(m=211, mean_len=90.0, cv=0.4, seed=3, k=900),    # 16
            "uneven": lambda: gen.skewed_csr(m=700, heavy_frac=0.01, heavy_lo=300, heavy_hi=650, seed=4)}   # 64


@pytest.mark.parametrize("name", MATRICES)
@pytest.mark.parametrize("known", [False, True])
@pytest.mark.parametrize("c_col", [False, True])
def test_column_major_products(name, known, c_col):
    from paper_2202_08556_amd import binding as da
    a = gen.integer_twin(MATRICES[name](), seed=8)
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (a.rowptr, a.colind, a.vals)]
    if known:
        da.da_spmm_features(a.m, 8, dev[0])
    for N in (1, 2, 3, 4, 5, 7, 8, 9, 16, 21, 24, 33):
        ldb, ldc = a.k + 3, (a.m + 2 if c_col else N + 2)
        B = np.full((N, ldb), np.nan, np.float32)
        B[:, :a.k] = gen.dense_int(a.k, N, seed=N).T
        want = orc.spmm(a.rowptr, a.colind, a.vals, np.ascontiguousarray(B[:, :a.k].T))[0].astype(np.float32) + 0.0
        Bd = torch.from_numpy(B).cuda()
        for algo in (da.DA_RB_RM_SR, da.DA_RB_CM_SR, da.DA_RB_RM_PR):
            C = torch.full((N, ldc) if c_col else (a.m, ldc), -7.0, device="cuda")
            da.da_spmm_ex(a.m, a.k, N, *dev, Bd, ldb, da.DA_COL_MAJOR, C, ldc, da.DA_COL_MAJOR if c_col else da.DA_ROW_MAJOR, algo)
            got = C.cpu().numpy()
            assert (got[:, a.m:] == -7.0).all() if c_col else (got[:, N:] == -7.0).all()
            got = got[:, :a.m].T if c_col else got[:, :N]
            assert np.array_equal(got, want), (N, algo)


def test_infinities_stay_in_their_rows():
    from paper_2202_08556_amd import binding as da
    a = gen.integer_twin(gen.uniform_csr(m=500, k=400, mean_len=6.0, seed=9), seed=9)
    B = gen.dense_int(a.k, 6, seed=1)
    B[0], B[17] = np.inf, np.nan                      # column 0 is what lanes without an entry would read
    want = orc.spmm(a.rowptr, a.colind, a.vals, B)[0].astype(np.float32) + 0.0
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (a.rowptr, a.colind, a.vals, B.T)]
    C = torch.empty((6, a.m), device="cuda")
    da.da_spmm_ex(a.m, a.k, 6, *dev, a.k, da.DA_COL_MAJOR, C, a.m, da.DA_COL_MAJOR, da.DA_RB_RM_SR)
    assert np.isfinite(want).any() and np.array_equal(C.t().cpu().numpy(), want, equal_nan=True)


# known: the lanes follow the rows; unknown: only where no sparsity law was slower for it
@pytest.mark.parametrize("name,known,N,algo,here", [
    ("stencil", True, 8, 0, True), ("stencil", True, 8, 1, True), ("stencil", True, 8, 2, True), ("uneven", True, 8, 1, True),
    ("short", True, 1, 0, True), ("longer", True, 8, 1, False), ("longer", True, 16, 0, True),
    ("stencil", False, 8, 0, False), ("stencil", False, 8, 1, False), ("short", False, 1, 2, False), ("uneven", False, 23, 0, False), ("uneven", False, 24, 0, True)])
def test_which_calls_take_the_kernel(name, known, N, algo, here):
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import kernels_of
    a = MATRICES[name]()
    dev = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (a.rowptr, a.colind, a.vals)]
    others = [torch.zeros(10, dtype=torch.int32, device="cuda") for _ in range(16)]
    for rowptr in others:                             # push out what is known of a matrix that lay here before
        da.da_spmm_features(9, 1, rowptr)
    if known:
        da.da_spmm_features(a.m, N, dev[0])
    B, C = torch.ones((N, a.k), device="cuda"), torch.empty((N, a.m), device="cuda")
    names = kernels_of(lambda: da.da_spmm_ex(a.m, a.k, N, *dev, B, a.k, da.DA_COL_MAJOR, C, a.m, da.DA_COL_MAJOR, algo))
    assert any("rb_columns_kernel" in n for n in names) == here, names


def test_positions_next_to_2_to_the_31():
    """2^31 - 1 entries in rows of 512: the last steps of the last rows pass 2^31."""
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import kernels_of
    m, k, each = 1 << 22, 1 << 20, 512
    rowptr = (torch.arange(m + 1, device="cuda") * each).clamp_(max=(1 << 31) - 1).to(torch.int32)
    colind = torch.empty(m * each, dtype=torch.int32, device="cuda")
    vals = torch.empty(m * each, device="cuda")
    b = (torch.arange(k, device="cuda") % 9 - 4).float()
    want = torch.empty(m, device="cuda")
    for r in range(0, m, 1 << 17):                    # in parts of 64 M entries
        at = torch.arange(r * each, (r + (1 << 17)) * each, device="cuda")
        c, v = (at * 7919) % k, (at % 5 - 2).float()
        if r + (1 << 17) == m:
            v[-1] = 0.0                               # the entry that the last row does not have
        colind[at[0]:at[-1] + 1], vals[at[0]:at[-1] + 1] = c.to(torch.int32), v
        want[r:r + (1 << 17)] = (v * b[c]).view(-1, each).sum(1)
        del at, c, v
    vals[-1] = float("nan")
    assert int(da.da_spmm_features(m, 1, rowptr)["nnz"]) == (1 << 31) - 1
    C = torch.full((m,), float("nan"), device="cuda")
    print("2^31 - 1 entries", flush=True)
    names = kernels_of(lambda: da.da_spmm(m, k, 1, rowptr, colind, vals, b, C, da.DA_RB_RM_SR))
    assert any("rb_columns_kernel" in n for n in names) and torch.equal(C, want)
