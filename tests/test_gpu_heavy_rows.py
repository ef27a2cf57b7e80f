"""Rows that hold a good part of all columns (heavy_rows_kernel, EB+RM+SR on prepared matrices): every lane mapping at its
edges, and plans that no longer describe the matrix, with whole numbers, whose sums have the same bits in any order;
rounding errors beside those of the EB kernels."""
import numpy as np
import pytest
import torch

from oracle import reference as orc

pytestmark = pytest.mark.gpu

K, M, HEAVY = 20011, 2500, 300                    # heavy: from a 32nd of the columns, 625, on; 256 of them for N > 32


def matrix(seed, heavy=HEAVY, lo=640, hi=4000):
    rng = np.random.Generator(np.random.PCG64(seed))
    lens = rng.poisson(3.0, M)
    lens[rng.choice(M, heavy, replace=False)] = rng.integers(lo, hi, heavy)
    lens[:2], lens[-1] = 0, K                     # empty rows, and one with every column
    return _csr(lens, rng)


def _csr(lens, rng):
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    colind = np.concatenate([np.sort(rng.choice(K, n, replace=False)) for n in lens]).astype(np.int32)
    vals = rng.choice(np.array([-3, -2, -1, 1, 2, 3], np.float32), colind.size)
    return rowptr, colind, vals


@pytest.fixture(scope="module")
def prepared():
    from paper_2202_08556_amd import binding as da
    host = matrix(5)
    dev = [torch.from_numpy(x).cuda() for x in host]
    da.da_spmm_prepare(M, K, host[1].size, dev[0], dev[1])
    yield host, dev
    da.da_spmm_release(dev[0])


def product(dev, B, N):
    from paper_2202_08556_amd import binding as da
    C = torch.full((M, N), float("nan"), device="cuda")
    da.da_spmm(M, K, N, *dev, B, C, da.DA_EB_RM_SR)
    return C.cpu().numpy()


def dense(N, seed=1):
    return np.random.Generator(np.random.PCG64(seed)).integers(-4, 5, (K, N)).astype(np.float32)


# between 65 and 128 columns a matrix of less than 10 M entries is the EB kernels'
@pytest.mark.parametrize("N", [1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 130])
def test_every_width(prepared, N):
    from tests.gpu_util import kernels_of
    host, dev = prepared
    print("heavy rows N", N, flush=True)
    B = dense(N)
    want, _ = orc.spmm(*host, B)
    got = []
    names = kernels_of(lambda: got.append(product(dev, torch.from_numpy(B).cuda(), N)))
    assert np.array_equal(got[0], want.astype(np.float32) + 0.0)
    assert any("heavy_rows_kernel" in n for n in names) == (not 65 <= N <= 128), names
    assert any("eb_sr_kernel" in n for n in names) == (65 <= N <= 128), names


# rows around sets of 64, groups of rows of other lengths, with ranges of their own
@pytest.mark.parametrize("heavy", [21, 64, 65, 127, 129, 576, 577, 1030])
@pytest.mark.parametrize("N", [4, 8, 20, 64, 130])
def test_groups_of_rows(heavy, N):
    from paper_2202_08556_amd import binding as da
    host = matrix(heavy, heavy, *((18000, 20012) if heavy < 64 else (640, 12000) if heavy < 500 else (640, 2000)))
    dev = [torch.from_numpy(x).cuda() for x in host]
    da.da_spmm_prepare(M, K, host[1].size, dev[0], dev[1])
    print(f"heavy rows {heavy} N {N}", flush=True)
    B = dense(N)
    want, _ = orc.spmm(*host, B)
    got = product(dev, torch.from_numpy(B).cuda(), N)
    da.da_spmm_release(dev[0])
    assert np.array_equal(got, want.astype(np.float32) + 0.0)


@pytest.mark.parametrize("N", [8, 40])
@pytest.mark.parametrize("order", ["row", "col"])
def test_stored_orders(prepared, N, order):
    from paper_2202_08556_amd import binding as da
    host, dev = prepared
    B = dense(N)
    want, _ = orc.spmm(*host, B)
    if order == "row":
        Bd = torch.full((K, N + 3), float("nan"), device="cuda")
        Bd[:, :N] = torch.from_numpy(B)
        C = torch.full((M, N + 5), -7.0, device="cuda")
        da.da_spmm_ex(M, K, N, *dev, Bd, N + 3, da.DA_ROW_MAJOR, C, N + 5, da.DA_ROW_MAJOR, da.DA_EB_RM_SR)
        assert (C[:, N:] == -7.0).all()
        got = C[:, :N]
    else:
        C = torch.full((N, M), float("nan"), device="cuda")
        da.da_spmm_ex(M, K, N, *dev, torch.from_numpy(np.ascontiguousarray(B.T)).cuda(), K, da.DA_COL_MAJOR, C, M, da.DA_COL_MAJOR,
                      da.DA_EB_RM_SR)
        got = C.t()
    assert np.array_equal(got.cpu().numpy(), want.astype(np.float32) + 0.0)


def test_infinities_stay_in_their_rows(prepared):
    host, dev = prepared
    B = dense(24)
    col = int(host[1][host[0][HEAVY]])
    B[col] = np.inf
    want, _ = orc.spmm(*host, B)
    got = product(dev, torch.from_numpy(B).cuda(), 24)
    assert np.isfinite(want).any() and np.array_equal(got, want.astype(np.float32) + 0.0, equal_nan=True)


# the same arrays with other contents after prepare: another matrix with as many entries, columns out of order,
# and columns that descend
@pytest.mark.parametrize("change", ["other", "shuffled", "descending", "fewer"])
@pytest.mark.parametrize("N", [8, 20, 64])
def test_plans_of_another_matrix(change, N):
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import kernels_of
    rowptr, colind, vals = matrix(7)
    dev = [torch.from_numpy(x).cuda() for x in (rowptr, colind, vals)]
    da.da_spmm_prepare(M, K, colind.size, dev[0], dev[1])
    rng = np.random.Generator(np.random.PCG64(9))
    if change == "other":                          # rows in another order
        lens = np.diff(rowptr)[rng.permutation(M)]
        rowptr, colind, vals = _csr(lens, rng)
    elif change == "fewer":
        rowptr = np.minimum(rowptr, rowptr[-1] - 1)
    else:
        for r in range(M):
            part = colind[rowptr[r]:rowptr[r + 1]]
            part[:] = rng.permutation(part) if change == "shuffled" else part[::-1].copy()
    for d, h in zip(dev, (rowptr, colind, vals)):
        d.copy_(torch.from_numpy(h))
    B = dense(N)
    want, _ = orc.spmm(rowptr, colind[:rowptr[-1]], vals[:rowptr[-1]], B)
    Bd = torch.from_numpy(B).cuda()
    assert np.array_equal(product(dev, Bd, N), want.astype(np.float32) + 0.0)
    # the list is another matrix's, and found to be: the EB kernels from now on, until the matrix is prepared again
    got = []
    names = kernels_of(lambda: got.append(product(dev, Bd, N)))
    assert np.array_equal(got[0], want.astype(np.float32) + 0.0)
    assert any("eb_sr_kernel" in n for n in names) and not any("heavy_rows_kernel" in n for n in names)
    da.da_spmm_prepare(M, K, int(rowptr[-1]), dev[0], dev[1])
    names = kernels_of(lambda: product(dev, Bd, N))
    assert any("heavy_rows_kernel" in n for n in names) == (change in ("other", "fewer"))          # not of columns out of order
    da.da_spmm_release(dev[0])


# what da_spmm_features has seen since
def test_features_of_another_matrix_put_the_list_aside():
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import kernels_of
    rowptr, colind, vals = matrix(17)
    dev = [torch.from_numpy(x).cuda() for x in (rowptr, colind, vals)]
    da.da_spmm_prepare(M, K, colind.size, dev[0], dev[1])
    rowptr = np.minimum(rowptr, rowptr[-1] - 1)
    dev[0].copy_(torch.from_numpy(rowptr))
    da.da_spmm_features(M, 8, dev[0])
    B = dense(8)
    want, _ = orc.spmm(rowptr, colind[:-1], vals[:-1], B)
    got = []
    names = kernels_of(lambda: got.append(product(dev, torch.from_numpy(B).cuda(), 8)))
    da.da_spmm_release(dev[0])
    assert np.array_equal(got[0], want.astype(np.float32) + 0.0)
    assert any("eb_sr_kernel" in n for n in names) and not any("heavy_rows_kernel" in n for n in names)


# the kernel would read every row of B that its plan covers: B ends at the columns that the product declares
@pytest.mark.parametrize("declared", [K + 9000, K + 1, K - 1])
@pytest.mark.parametrize("N", [8, 64])
def test_products_that_declare_other_columns_than_prepare(declared, N):
    from paper_2202_08556_amd import binding as da
    rowptr, colind, vals = matrix(15)
    dev = [torch.from_numpy(x).cuda() for x in (rowptr, np.minimum(colind, declared - 1), vals)]
    print("prepared for", declared, "columns, N", N, flush=True)
    da.da_spmm_prepare(M, declared, colind.size, dev[0], dev[1])
    dev[1].copy_(torch.from_numpy(colind))
    B = dense(N)
    want, _ = orc.spmm(rowptr, colind, vals, B)
    got = product(dev, torch.from_numpy(B).cuda(), N)
    da.da_spmm_release(dev[0])
    assert np.array_equal(got, want.astype(np.float32) + 0.0)


# 8000 rows' list takes 32 MB, the orders some 8: with 20 MB left prepare goes without the list
def test_prepare_without_the_memory_for_the_list():
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import kernels_of
    m, each = 8200, 640
    rng = np.random.Generator(np.random.PCG64(3))
    lens = np.where(np.arange(m) % 41 < 40, each, 2)
    first = rng.integers(0, K - 20 * each, m)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    colind = np.concatenate([first[r] + 20 * np.arange(n) for r, n in enumerate(lens)]).astype(np.int32)
    vals = rng.choice(np.array([-2, -1, 1, 2], np.float32), colind.size)
    B = dense(4)
    want, _ = orc.spmm(rowptr, colind, vals, B)
    dev = [torch.from_numpy(x).cuda() for x in (rowptr, colind, vals, B)]
    C = torch.empty((m, 4), device="cuda")
    call = lambda: da.da_spmm(m, K, 4, *dev, C, da.DA_EB_RM_SR)  # noqa: E731
    da.da_spmm_prepare(m, K, colind.size, dev[0], dev[1])          # with memory: all code is loaded, pools are filled
    assert any("heavy_rows_kernel" in n for n in kernels_of(call))
    da.da_spmm_release(dev[0])
    torch.cuda.empty_cache()
    fill = []
    while (free := torch.cuda.mem_get_info()[0]) > 22 << 20:
        fill.append(torch.empty(max(free - (20 << 20), 1 << 20), dtype=torch.uint8, device="cuda"))
    print("left free", free >> 20, "MB", flush=True)
    try:
        da.da_spmm_prepare(m, K, colind.size, dev[0], dev[1])
    finally:
        del fill
        torch.cuda.empty_cache()
    names = kernels_of(call)
    da.da_spmm_release(dev[0])
    assert any("eb_sr_kernel" in n for n in names) and not any("heavy_rows_kernel" in n for n in names)
    assert np.array_equal(C.cpu().numpy(), want.astype(np.float32) + 0.0)


def test_unsorted_columns_have_no_plan_and_stay_right():
    from paper_2202_08556_amd import binding as da
    rowptr, colind, vals = matrix(11)
    rng = np.random.Generator(np.random.PCG64(2))
    for r in range(M):
        part = colind[rowptr[r]:rowptr[r + 1]]
        part[:] = rng.permutation(part)
    dev = [torch.from_numpy(x).cuda() for x in (rowptr, colind, vals)]
    da.da_spmm_prepare(M, K, colind.size, dev[0], dev[1])
    B = dense(16)
    want, _ = orc.spmm(rowptr, colind, vals, B)
    got = product(dev, torch.from_numpy(B).cuda(), 16)
    da.da_spmm_release(dev[0])
    assert np.array_equal(got, want.astype(np.float32) + 0.0)


def test_recorded_calls_keep_their_plan():
    from paper_2202_08556_amd import binding as da
    host = matrix(13)
    dev = [torch.from_numpy(x).cuda() for x in host]
    da.da_spmm_prepare(M, K, host[1].size, dev[0], dev[1])
    B = dense(12)
    want = orc.spmm(*host, B)[0].astype(np.float32) + 0.0
    Bd, C = torch.from_numpy(B).cuda(), torch.zeros((M, 12), device="cuda")
    da.da_spmm(M, K, 12, *dev, Bd, C, da.DA_EB_RM_SR)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        da.da_spmm(M, K, 12, *dev, Bd, C, da.DA_EB_RM_SR)
    da.da_spmm_prepare(M, K, host[1].size, dev[0], dev[1])         # the recorded plan stays
    for _ in range(3):
        C.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(C.cpu().numpy(), want)
    da.da_spmm_release(dev[0])


# Products of one sign, whose error grows with the number of parts of a row and with the terms that are added one after
# another: short and long heavy rows side by side, other rows up to the length of a chunk and far beyond it.
@pytest.mark.parametrize("N", [1, 4, 8, 16, 24, 32, 64])
@pytest.mark.parametrize("longest_other", [30, 900])
def test_sums_are_as_exact_as_in_chunks(N, longest_other, monkeypatch):
    from paper_2202_08556_amd import binding as da
    m, k = 30000, 60000
    rng = np.random.Generator(np.random.PCG64(21))
    lens = np.full(m, 30)
    lens[10:50] = longest_other
    lens[100:250], lens[300:450] = rng.integers(1900, 2600, 150), rng.integers(15000, 30000, 150)
    lens = lens[rng.permutation(m)]
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    colind = np.concatenate([np.sort(rng.choice(k, n, replace=False)) for n in lens]).astype(np.int32)
    vals, B = rng.random(colind.size, dtype=np.float32), rng.random((k, N), dtype=np.float32)
    want, _ = orc.spmm(rowptr, colind, vals, B, want_abs=False)
    dev = [torch.from_numpy(x).cuda() for x in (rowptr, colind, vals, B)]
    da.da_spmm_prepare(m, k, colind.size, dev[0], dev[1])

    def error(off):
        monkeypatch.setenv("DA_SPMM_NO_HEAVY", off)
        total = np.zeros(m)
        for _ in range(3):
            C = torch.empty((m, N), device="cuda")
            da.da_spmm(m, k, N, *dev, C, da.DA_EB_RM_SR)
            total += ((C.cpu().numpy().astype(np.float64) - want) ** 2).sum(1) / (want ** 2).sum(1)
        return total

    here, chunks = error("0"), error("1")
    da.da_spmm_release(dev[0])
    for name, rows in (("others", lens < 100), ("longest others", lens == longest_other), ("short", (lens >= 1900) & (lens < 2600)),
                       ("long", lens >= 15000)):
        a, b = (np.sqrt(x[rows].mean() / 3) for x in (here, chunks))
        print(f"N={N} {name}: {a:.2e}, in chunks {b:.2e}", flush=True)
        # The order of additions changes the figures by a tenth from run to run; the mean over n sums is off by
        # 1 / sqrt(2 n), 4 % of it for 300.
        assert rows.sum() * N < 300 or a <= 1.15 * b


# B comes in pieces of 16 bytes where its rows are such pieces, and in single numbers where they are not
@pytest.mark.parametrize("N", [4, 8, 20, 64])
@pytest.mark.parametrize("offset, more", [(0, 4), (0, 3), (1, 4), (4, 0), (2, 1)])
def test_rows_of_b_at_any_alignment(prepared, N, offset, more):
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import kernels_of
    host, dev = prepared
    da.da_spmm_prepare(M, K, host[1].size, dev[0], dev[1])         # plans of other tests may have taken its place
    print("heavy rows N", N, "offset", offset, "pitch", N + more, flush=True)
    B = dense(N)
    want, _ = orc.spmm(*host, B)
    room = torch.full((K * (N + more) + offset,), float("nan"), device="cuda")
    inner = room[offset:].view(K, N + more)
    inner[:, :N] = torch.from_numpy(B).cuda()
    C = torch.full((M, N), float("nan"), device="cuda")
    names = kernels_of(lambda: da.da_spmm_ex(M, K, N, *dev, inner, N + more, da.DA_ROW_MAJOR, C, N, da.DA_ROW_MAJOR, da.DA_EB_RM_SR))
    assert np.array_equal(C.cpu().numpy(), want.astype(np.float32) + 0.0)
    assert any("heavy_rows_kernel" in n for n in names), names


# Sets of 4 rows a wave: a block has 15 waves that walk rows, 16 where all bring B, and up to nine sets in each.  A launch has at
# most 17 groups of rows: beyond 17 * 8 * 60 = 8160 rows one of them has nine sets.  8192 are as many as a plan takes.
@pytest.mark.parametrize("heavy, each, N, order", [
    (60, 7000, 8, "row"), (61, 7000, 8, "row"), (64, 7000, 3, "row"), (65, 7000, 3, "row"), (540, 2000, 16, "row"), (541, 2000, 64, "row"),
    (8161, 640, 4, "row"), (8192, 640, 4, "row"), (8161, 3000, 16, "row"), (8161, 3000, 24, "row"), (8192, 3000, 64, "row"),
    (8161, 640, 130, "row"), (8192, 640, 2, "row"), (8192, 640, 12, "col"),
])
def test_rows_that_fill_a_block(heavy, each, N, order):
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import kernels_of
    dev, m = "cuda", heavy + 41
    lens = torch.full((m,), 3, dtype=torch.int64, device=dev)
    lens[torch.arange(heavy, device=dev) * m // heavy] = each
    rowptr = torch.zeros(m + 1, dtype=torch.int32, device=dev)
    torch.cumsum(lens, 0, out=rowptr[1:])
    row = torch.repeat_interleave(torch.arange(m, device=dev), lens)
    at = torch.arange(row.numel(), device=dev) - rowptr[row].long()
    step = (K - 1) // each
    colind = (at * step + row * 7919 % (K - (each - 1) * step)).to(torch.int32)
    vals = ((at + row) % 5 - 2).float()
    B = (torch.arange(K * N, device=dev) * 7919 % 9 - 4).float().view(K, N)
    a = torch.zeros((m, K), device=dev)
    a[row, colind.long()] = vals
    want = a @ B                                              # whole numbers below 2^24: exact in any order
    da.da_spmm_prepare(m, K, colind.numel(), rowptr, colind)
    print("heavy", heavy, "each", each, "N", N, order, flush=True)
    if order == "row":
        C = torch.full((m, N), float("nan"), device=dev)
        names = kernels_of(lambda: da.da_spmm(m, K, N, rowptr, colind, vals, B, C, da.DA_EB_RM_SR))
    else:
        Bt, Ct = B.t().contiguous(), torch.full((N, m), float("nan"), device=dev)
        names = kernels_of(lambda: da.da_spmm_ex(m, K, N, rowptr, colind, vals, Bt, K, da.DA_COL_MAJOR, Ct, m, da.DA_COL_MAJOR, da.DA_EB_RM_SR))
        C = Ct.t()
    da.da_spmm_release(rowptr)
    assert any("heavy_rows_kernel" in n for n in names), names
    assert torch.equal(C, want)


# from 2^29 entries on their bytes are more than an int holds; a plan has less than 2^30 entries
@pytest.mark.parametrize("rows, N", [(513, 8), (513, 64), (1024, 8), (1024, 64)])
def test_plans_of_very_many_entries(rows, N):
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import kernels_of
    dev, k = "cuda", 1 << 20
    nnz = rows * k - 1                                        # every column in every row, but the last one of the last row
    print("rows", rows, "entries", nnz, "N", N, flush=True)
    rowptr = (torch.arange(rows + 1, device=dev) * k).clamp(max=nnz).to(torch.int32)
    colind = torch.arange(k, dtype=torch.int32, device=dev).repeat(rows)
    vals = torch.arange(rows * k, dtype=torch.int32, device=dev).remainder_(5).sub_(2).float()
    vals[nnz] = 0.0
    B = (torch.arange(k * N, device=dev) * 7919 % 9 - 4).float().view(k, N)
    want = vals.view(rows, k) @ B                             # whole numbers below 2^24: exact in any order
    da.da_spmm_prepare(rows, k, nnz, rowptr, colind)
    C = torch.full((rows, N), float("nan"), device=dev)
    names = kernels_of(lambda: da.da_spmm(rows, k, N, rowptr, colind, vals, B, C, da.DA_EB_RM_SR))
    da.da_spmm_release(rowptr)
    assert any("heavy_rows_kernel" in n for n in names), names
    assert torch.equal(C, want)


# a wave of its own brings rows of B of four and more numbers, whatever they are aligned to; all waves bring others
@pytest.mark.parametrize("N", [1, 2, 3, 5, 6, 7, 9, 13, 15, 18, 19, 31, 33, 41, 62, 130])
@pytest.mark.parametrize("order, offset, more", [("row", 0, 0), ("row", 1, 0), ("row", 3, 2), ("col", 0, 0)])
def test_who_brings_rows_of_b(prepared, N, order, offset, more):
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import kernels_of
    host, dev = prepared
    da.da_spmm_prepare(M, K, host[1].size, dev[0], dev[1])         # plans of other tests may have taken its place
    print("heavy rows N", N, order, "offset", offset, "pitch", N + more, flush=True)
    B = dense(N)
    want, _ = orc.spmm(*host, B)
    room = torch.full((offset + (K - 1) * (N + more) + N,), float("nan"), device="cuda")
    if order == "row":
        Bd = room[offset:].as_strided((K, N), (N + more, 1))
        Bd.copy_(torch.from_numpy(B))
        ldb, C = N + more, torch.full((M, N), float("nan"), device="cuda")
        call = lambda: da.da_spmm_ex(M, K, N, *dev, Bd, ldb, da.DA_ROW_MAJOR, C, N, da.DA_ROW_MAJOR, da.DA_EB_RM_SR)  # noqa: E731
    else:
        Bd, C = torch.from_numpy(np.ascontiguousarray(B.T)).cuda(), torch.full((N, M), float("nan"), device="cuda")
        call = lambda: da.da_spmm_ex(M, K, N, *dev, Bd, K, da.DA_COL_MAJOR, C, M, da.DA_COL_MAJOR, da.DA_EB_RM_SR)  # noqa: E731
    names = kernels_of(call)
    got = C if order == "row" else C.t()
    assert np.array_equal(got.cpu().numpy(), want.astype(np.float32) + 0.0)
    by_one = order == "row" and N >= 4
    assert any("heavy_rows_kernel" in n and ("true" if by_one else "false") in n for n in names), names


# matrices on either side of the line between the two: many rows of one length, whose blocks have more than their share of the work
@pytest.mark.parametrize("heavy, each, k, N, taken", [
    (900, 9000, 100_000, 48, True), (900, 9000, 100_000, 41, True), (2000, 6000, 65_536, 24, True), (8000, 1300, 40_000, 24, False),
    (8000, 1300, 40_000, 48, False), (1500, 8000, 130_000, 64, False), (1300, 3000, 50_000, 41, True), (3500, 5000, 100_000, 16, False),
])
def test_which_matrices_take_the_kernel(heavy, each, k, N, taken):
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import kernels_of
    m, step, dev = heavy + 20_000, k // each, "cuda"
    lens = torch.full((m,), 3, dtype=torch.int64, device=dev)
    rows = torch.arange(heavy, device=dev) * (m // heavy)
    lens[rows] = each
    rowptr = torch.zeros(m + 1, dtype=torch.int32, device=dev)
    torch.cumsum(lens, 0, out=rowptr[1:])
    row = torch.repeat_interleave(torch.arange(m, device=dev), lens)
    at = torch.arange(row.numel(), device=dev) - rowptr[row].long()
    colind = (at * step + row % step).to(torch.int32)         # heavy rows with the same remainder are alike but for a factor
    vals = (at % 3 - 1 + (row % 2) * 4).float()
    B = (torch.arange(k * N, device=dev) * 7919 % 9 - 4).float().view(k, N)
    da.da_spmm_prepare(m, k, colind.numel(), rowptr, colind)
    C = torch.full((m, N), float("nan"), device=dev)
    print("heavy", heavy, "each", each, "N", N, flush=True)
    names = kernels_of(lambda: da.da_spmm(m, k, N, rowptr, colind, vals, B, C, da.DA_EB_RM_SR))
    da.da_spmm_release(rowptr)
    assert any("heavy_rows_kernel" in n for n in names) == taken, names
    some = torch.cat([rows[:60], rows[-60:], rows[:60] + 1, torch.tensor([0, m - 1], device=dev)]).clamp(max=m - 1)
    for r in some.tolist():
        part = slice(int(rowptr[r]), int(rowptr[r + 1]))
        assert torch.equal(C[r], (vals[part, None] * B[colind[part].long()]).sum(0))
    assert not torch.isnan(C.sum(1)).any()
