"""da_spmm_dense_split (fp32 products as products of bf16 pieces) at the edges of its tiles and steps against float64,
its error against the fp32 kernel's, and numbers that the pieces do not carry or carry in part."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def split(X, ldx, W, wk, wn, rows, k, n, ldc):
    from paper_2202_08556_amd import binding as da
    size = da.da_spmm_dense_split_workspace(k, n)
    C = torch.full((rows, ldc), -7.0, device="cuda")
    da.da_spmm_dense_split(rows, k, n, X, ldx, W, wk, wn, C, ldc, torch.full((size,), 255, dtype=torch.uint8, device="cuda"), size)
    assert (C[:, n:] == -7.0).all()
    return C[:, :n]


# rows around a wave's 16 and a block's 128, sums around a step of 32, columns around tiles of 16 and blocks of 32 ... 128
@pytest.mark.parametrize("rows,k,n", [(1, 32, 1), (16, 33, 16), (17, 63, 17), (127, 64, 32), (128, 65, 33), (129, 96, 64), (300, 97, 65),
                                      (257, 602, 96), (1000, 130, 97), (129, 1000, 128), (129, 40, 129), (65, 255, 300)])
@pytest.mark.parametrize("transposed", [False, True])
def test_split_product(rows, k, n, transposed):
    print(f"split rows={rows} k={k} n={n}", flush=True)
    g = torch.Generator().manual_seed(rows + k)
    ldx = k + rows % 3
    X, W = torch.randn((rows, ldx), generator=g), torch.randn((k, n), generator=g)
    X[:, k:] = float("nan")                                       # padding: never part of a result
    want = X[:, :k].double() @ W.double()
    w = (W.t().contiguous() if transposed else W).cuda()
    got = split(X.cuda(), ldx, w, *((1, k) if transposed else (n, 1)), rows, k, n, n + rows % 4).double().cpu()
    # pieces left out: 3 * 2^-24 of |X||W| at most; fp32 sums of k terms of random sign: sqrt(k) * 2^-24 of it
    bound = (3 + k ** 0.5) * 2.0 ** -24 * (X[:, :k].double().abs() @ W.double().abs())
    assert ((got - want).abs() <= bound).all(), ((got - want).abs() / bound).max()


@pytest.mark.parametrize("k,n", [(64, 64), (200, 128), (256, 16)])
def test_split_product_is_as_exact_as_fp32(k, n):
    from paper_2202_08556_amd import binding as da
    for dist in (torch.randn, torch.rand):
        X, W = dist((4000, k), device="cuda"), dist((k, n), device="cuda")
        want = X.double() @ W.double()
        C = torch.empty((4000, n), device="cuda")
        da.da_spmm_dense(4000, k, n, X, k, W, n, 1, C, n)
        assert (split(X, k, W, n, 1, 4000, k, n, n).double() - want).norm() <= (C.double() - want).norm()


# in one wave's rows each; the other waves' results are not touched by it
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.4e38, 1e-31, 1e-36, 1e-42])
@pytest.mark.parametrize("where", ["X", "W"])
def test_numbers_that_pieces_do_not_carry(value, where):
    rows, k, n = 300, 70, 50
    g = torch.Generator().manual_seed(3)
    X, W = torch.randn((rows, k), generator=g), torch.randn((k, n), generator=g)
    (X if where == "X" else W)[20, 40] = value
    if value < 1e-20:                                             # the small number alone makes the result
        if where == "X":
            X[20] = 0.0
            X[20, 40] = value
        else:
            W[:, 40] = 0.0
            W[20, 40] = value
    # an fp32 product rounds where float64 does not, and overflows to infinity
    want = (X.double() @ W.double())
    got = split(X.cuda(), k, W.cuda(), n, 1, rows, k, n, n).cpu()
    finite = want.abs() <= torch.finfo(torch.float32).max
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(got[~finite & ~torch.isnan(want)].double().sign(), want[~finite & ~torch.isnan(want)].sign())
    bound = (3 + k ** 0.5) * 2.0 ** -24 * (X.double().abs() @ W.double().abs()) + k * 2.0 ** -149
    assert ((got.double() - want).abs() <= bound)[finite].all()


# small numbers among ordinary ones: what their pieces lose matters where they meet large ones, and in columns of nothing else
@pytest.mark.parametrize("where", ["X", "W"])
@pytest.mark.parametrize("value,other", [(1e-40, 1.0), (1e-36, 1e30), (3e-34, 1e24), (1e-31, 1e12), (1e-38, 0.0)])
@pytest.mark.parametrize("rows,k,n", [(300, 70, 50), (129, 33, 130), (64, 47, 16)])
def test_small_numbers_among_others(where, value, other, rows, k, n):
    g = torch.Generator().manual_seed(5)
    X, W = torch.randn((rows, k), generator=g), torch.randn((k, n), generator=g)
    X[5], W[:, 3] = 0.0, 0.0                                      # rows and columns of zeros stay zeros
    if where == "X":
        X[20, 10] = X[40, 10] = X[63, k - 1] = value
        W[10, ::2], W[k - 1, 1] = other, other
        X[40] *= 1e-30                                            # a row of nothing but small numbers
    else:
        W[10, 7], W[k - 1, 15] = value, -value
        W[:, n - 1] *= 1e-33
        X[::3, 10], X[7, k - 1] = other, other
    want = X.double() @ W.double()
    got = split(X.cuda(), k, W.cuda(), n, 1, rows, k, n, n).cpu()
    bound = (3 + k ** 0.5) * 2.0 ** -24 * (X.double().abs() @ W.double().abs()) + k * 2.0 ** -149
    assert ((got.double() - want).abs() <= bound).all()
    assert not got[5].any() and not got[:, 3].any()


# infinities and NaN beside small numbers, in the last positions, which the last step reads once more
@pytest.mark.parametrize("k", [32, 33, 47, 48, 49, 70])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_what_is_not_finite_stays_where_it_is(k, value):
    g = torch.Generator().manual_seed(7)
    X, W = torch.randn((200, k), generator=g), torch.randn((k, 40), generator=g).abs() + 1.0
    for j, p in enumerate(range(max(0, k - 34), k)):
        X[3 * j, p] = value
    X[150, 2], W[1, 30] = 1e-42, 1e-42
    want = X.double() @ W.double()
    got = split(X.cuda(), k, W.cuda(), 40, 1, 200, k, 40, 40).cpu()
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(torch.isinf(got), torch.isinf(want)) and torch.equal(got[torch.isinf(got)].double(), want[torch.isinf(want)])
    fine = torch.isfinite(want)
    bound = (3 + k ** 0.5) * 2.0 ** -24 * (X.double().abs() @ W.double().abs())
    assert ((got.double() - want).abs() <= bound)[fine].all()


def test_split_errors():
    from paper_2202_08556_amd import binding as da
    t = torch.zeros(1 << 16, device="cuda")
    size = da.da_spmm_dense_split_workspace(64, 8)
    da.da_spmm_dense_split(0, 64, 8, t, 64, t, 8, 1, t, 8, t, size)
    for args in ((4, 31, 4, t, 31, t, 4, 1, t, 4, t, 1 << 16), (4, 64, 8, t, 63, t, 8, 1, t, 8, t, size),
                 (4, 64, 8, t, 64, t, 8, 1, t, 8, t, size - 1), (4, 64, 8, t, 64, t, 8, 1, t, 8, None, size),
                 (4, 64, 8, t, 64, t, 8, 1, t, 8, t.data_ptr() + 4, size), (-1, 64, 8, t, 64, t, 8, 1, t, 8, t, size)):
        with pytest.raises(da.DaSpmmError):
            da.da_spmm_dense_split(*args)
