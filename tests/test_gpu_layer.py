"""da_spmm_layer (bias and rectification where the sums leave the product kernel) against da_spmm_ex and da_spmm_bias_relu:
whole numbers, so that additions in any order give the same bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def matrix(kind):
    g = torch.Generator().manual_seed(7)
    m, k = 700, 900
    if kind == "mixed":                                           # empty rows, short ones, rows of several chunks
        lens = torch.randint(0, 9, (m,), generator=g)
        lens[::7] = 0
        lens[3:700:50] = 64
        lens[5:700:90] = 130
        lens[[0, 350, 699]] = 880
    else:                                                         # every row longer than any chunk but PR's
        m = 40
        lens = torch.randint(300, 800, (m,), generator=g)
    rowptr = torch.zeros(m + 1, dtype=torch.int32)
    rowptr[1:] = lens.cumsum(0)
    colind = torch.cat([torch.randperm(k, generator=g)[:n].sort()[0] for n in lens.tolist()]).to(torch.int32)
    vals = torch.randint(1, 4, (colind.numel(),), generator=g).float() * (1 - 2 * torch.randint(0, 2, (colind.numel(),), generator=g))
    return m, k, rowptr.cuda(), colind.cuda(), vals.cuda()


# lane groups of one column (8 ... 16, ragged below 64) and of four, widths around a tile of 128, several tiles
@pytest.mark.parametrize("N", [1, 3, 4, 7, 8, 12, 16, 17, 30, 32, 41, 64, 67, 100, 128, 130, 257])
@pytest.mark.parametrize("kind", ["mixed", "long"])
@pytest.mark.parametrize("prepared", [False, True])
def test_layer_is_product_and_pass(N, kind, prepared):
    from paper_2202_08556_amd import binding as da
    m, k, rowptr, colind, vals = matrix(kind)
    g = torch.Generator().manual_seed(N)
    ldb = N + N % 5
    B = torch.randint(-4, 5, (k, ldb), generator=g).float().cuda()
    bias = torch.randint(-9, 10, (N + 1,), generator=g).float().cuda()[1:]       # not on a 16-byte address
    try:
        if prepared:
            da.da_spmm_features(m, N, rowptr)
            da.da_spmm_prepare(m, k, colind.numel(), rowptr, colind)
        for algo in range(da.DA_NUM_ALGOS):
            want = torch.empty((m, N), device="cuda")
            da.da_spmm_ex(m, k, N, rowptr, colind, vals, B, ldb, da.DA_ROW_MAJOR, want, N, da.DA_ROW_MAJOR, algo)
            for b, relu in ((bias, True), (bias, False), (None, True), (None, False)):
                print(f"layer N={N} {kind} prepared={prepared} algo={algo} bias={b is not None} relu={relu}", flush=True)
                full = want.clone()
                da.da_spmm_bias_relu(m, N, full, b, relu)
                C = torch.full((m * N + 1,), float("nan"), device="cuda")[1:]    # every element is written
                da.da_spmm_layer(m, k, N, rowptr, colind, vals, B, ldb, C, b, relu, algo)
                assert torch.equal(C.view(m, N), full)
                assert torch.equal(torch.signbit(C.view(m, N)), torch.signbit(full)) or b is None and not relu
    finally:
        da.da_spmm_release(rowptr)


# EB finishes layers itself from 2 M elements of C on: either side of the line, empty rows, short ones, rows of several chunks
@pytest.mark.parametrize("N", [8, 16, 30, 37, 64, 67, 128, 130, 257])
@pytest.mark.parametrize("rows", [-1, 0, 301])
@pytest.mark.parametrize("prepared", [False, True])
def test_layers_of_many_rows(N, rows, prepared):
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import kernels_of
    m, k = (2 * 2 ** 20 + N - 1) // N + rows, 3001
    g = torch.Generator().manual_seed(N)
    lens = torch.randint(0, 6, (m,), generator=g)
    lens[::3] = 0
    lens[5::900] = 130
    lens[[0, m // 2, m - 1]] = 2900
    rowptr = torch.zeros(m + 1, dtype=torch.int32)
    rowptr[1:] = lens.cumsum(0)
    nnz = int(rowptr[-1])
    colind = torch.randint(0, k, (nnz,), generator=g).to(torch.int32).cuda()
    vals = torch.randint(-3, 4, (nnz,), generator=g).float().cuda()
    rowptr = rowptr.cuda()
    B = torch.randint(-4, 5, (k, N), generator=g).float().cuda()
    bias = torch.randint(-9, 10, (N + 1,), generator=g).float().cuda()[1:]
    try:
        if prepared:
            da.da_spmm_prepare(m, k, nnz, rowptr, colind)
        for algo in (da.DA_EB_RM_SR, da.DA_EB_RM_PR):
            want = torch.empty((m, N), device="cuda")
            da.da_spmm(m, k, N, rowptr, colind, vals, B, want, algo)
            for b, relu in ((bias, True), (bias, False), (None, True)):
                print(f"layer m={m} N={N} prepared={prepared} algo={algo} bias={b is not None} relu={relu}", flush=True)
                full = want.clone()
                da.da_spmm_bias_relu(m, N, full, b, relu)
                C = torch.full((m * N + 1,), float("nan"), device="cuda")[1:]
                names = kernels_of(lambda: da.da_spmm_layer(m, k, N, rowptr, colind, vals, B, N, C, b, relu, algo))
                assert torch.equal(C.view(m, N), full)
                here = rows >= 0 and not (N == 8 and algo == da.DA_EB_RM_PR)     # two lanes of four columns have no such form
                assert any("eb_finish_kernel" in n for n in names) == here, names
                assert any("bias_relu_kernel" in n for n in names) == (not here), names
    finally:
        da.da_spmm_release(rowptr)


@pytest.mark.parametrize("algo", range(8))
def test_layer_keeps_what_is_not_finite(algo):
    from paper_2202_08556_amd import binding as da
    m, k, rowptr, colind, vals = matrix("mixed")
    N = 36
    vals[::97] = float("nan")
    vals[50::101] = float("inf")
    B = torch.ones((k, N), device="cuda")
    bias = torch.full((N,), -2.0, device="cuda")
    bias[5], bias[6] = float("nan"), float("-inf")
    want, C = torch.empty((m, N), device="cuda"), torch.empty((m, N), device="cuda")
    da.da_spmm(m, k, N, rowptr, colind, vals, B, want, algo)
    da.da_spmm_bias_relu(m, N, want, bias, True)
    da.da_spmm_layer(m, k, N, rowptr, colind, vals, B, N, C, bias, True, algo)
    assert torch.equal(torch.isnan(C), torch.isnan(want))
    assert torch.equal(torch.nan_to_num(C), torch.nan_to_num(want))


def test_layer_refuses_what_the_product_refuses():
    from paper_2202_08556_amd import binding as da
    t = torch.zeros(64, device="cuda")
    i = torch.zeros(64, dtype=torch.int32, device="cuda")
    da.da_spmm_layer(0, 4, 4, i, i, t, t, 4, t, t, True, 0)
    for args in ((4, 4, 4, i, i, t, t, 3, t, t, True, 0), (4, 4, 4, i, i, t, t, 4, None, t, True, 0),
                 (4, 4, 4, i, i, t, t, 4, t, t, True, 8), (-1, 4, 4, i, i, t, t, 4, t, t, True, 0)):
        with pytest.raises(da.DaSpmmError):
            da.da_spmm_layer(*args)
