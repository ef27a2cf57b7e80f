"""Launch geometry of the SR ids at the widths where it depends on what is known of the matrix: lanes of one or four
columns, chunk sizes, chunk order.  Whatever is chosen, the product is the oracle's."""
import numpy as np
import pytest
import torch

from oracle import reference as orc
from paper_2202_08556_amd import generators as gen

pytestmark = pytest.mark.gpu

MATRICES = {
    "short": lambda: gen.uniform_csr(m=3001, k=2500, mean_len=12, seed=31),
    "uneven": lambda: gen.lognormal_csr(2500, 30.0, 2.0, seed=32),
    "long_rows": lambda: gen.skewed_csr(m=6000, k=9000, heavy_frac=0.003, heavy_lo=3000, heavy_hi=8000, seed=33),
    "mostly_empty": lambda: gen.hypersparse_csr(60000, 5000, 0.02, 40.0, seed=34),
}


@pytest.mark.parametrize("name", list(MATRICES))
@pytest.mark.parametrize("known", ["nothing", "features", "plan"])
def test_sr_ids_at_every_lane_mapping(name, known):
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import DeviceProblem
    ai = gen.integer_twin(MATRICES[name]())
    da.da_spmm_release()
    for N in (5, 8, 16, 17, 24, 25, 31, 32, 33, 41, 63, 64, 65):
        B = gen.dense_int(ai.k, N, seed=N)
        want, _ = orc.spmm(ai.rowptr, ai.colind, ai.vals, B, want_abs=False)
        prob = DeviceProblem(ai, B)
        if known == "features":
            da.da_spmm_features(ai.m, N, prob.rowptr)
        elif known == "plan":
            da.da_spmm_prepare(ai.m, ai.k, ai.nnz, prob.rowptr, prob.colind)
        for algo in (da.DA_RB_RM_SR, da.DA_EB_RM_SR):
            print(f"geometry {name} {known} N={N} algo={algo}", flush=True)
            assert orc.bit_mismatches(prob.run(algo), want) == 0, (name, known, N, algo)
        if N in (41, 64):                                     # rows that begin anywhere: an offset base, an odd pitch
            wide = torch.zeros((ai.k, N + 1), device="cuda")
            wide[:, 1:] = prob.B
            C = torch.full((ai.m, N + 3), float("nan"), device="cuda")
            for algo in (da.DA_RB_RM_SR, da.DA_EB_RM_SR):
                da.da_spmm_ex(ai.m, ai.k, N, prob.rowptr, prob.colind, prob.vals, wide.data_ptr() + 4, N + 1, da.DA_ROW_MAJOR,
                              C.data_ptr() + 8, N + 3, da.DA_ROW_MAJOR, algo)
                torch.cuda.synchronize()
                flat = C.reshape(-1)[2:2 + (ai.m - 1) * (N + 3) + N].cpu().numpy()
                got = np.lib.stride_tricks.as_strided(flat, (ai.m, N), ((N + 3) * 4, 4))
                assert orc.bit_mismatches(np.ascontiguousarray(got), want) == 0, (name, known, N, algo)
        da.da_spmm_release(prob.rowptr)


@pytest.mark.parametrize("algo", [1, 5])
@pytest.mark.parametrize("N", [41, 65, 127])
def test_pr_sums_are_as_exact_with_wide_lane_groups(algo, N):
    """PR with 4 or 2 slots along a row adds as few terms one after another as with 8.  A sum of L products of random
    sign, one after another, is off by about 2^-24 sqrt(L/6) of its size: 1.7e-7 for the L = 50 of 8 slots on
    rows of 400 entries, 2.4e-7 and 3.5e-7 for 4 and 2; measured were 1.4e-7, 1.9e-7 and 2.3e-7."""
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import DeviceProblem
    a = gen.lognormal_csr(4000, 400.0, 0.2, seed=41)
    B = np.random.default_rng(42).standard_normal((a.k, N)).astype(np.float32)
    prob = DeviceProblem(a, B)
    want, _ = orc.spmm(a.rowptr, a.colind, a.vals, B)
    got = prob.run(algo).astype(np.float64)
    assert np.linalg.norm(got - want) <= 1.55e-7 * np.linalg.norm(want)


@pytest.mark.parametrize("N", [8, 16, 64])
def test_chunks_of_long_rows_are_no_smaller_than_without_a_plan(N):
    """A row of n entries in chunks of c takes n / c additions to C one after another: with chunks of 32 or 64 instead
    of the 56 to 256 without a plan, rows of 20 000 entries were off by 1.3 times as much (4.3e-7 of the result at
    N = 8, 3.0e-7 without a plan).  The order of the additions changes the figures by a tenth from run to run."""
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import DeviceProblem
    a = gen.skewed_csr(m=50000, heavy_frac=0.003, heavy_lo=10000, heavy_hi=24000, seed=51)
    B = np.random.default_rng(52).standard_normal((a.k, N)).astype(np.float32)
    want, _ = orc.spmm(a.rowptr, a.colind, a.vals, B, want_abs=False)
    prob = DeviceProblem(a, B)

    def error():
        runs = [prob.run(da.DA_EB_RM_SR).astype(np.float64) - want for _ in range(4)]
        return np.sqrt(np.mean([np.sum(r * r) for r in runs])) / np.linalg.norm(want)

    da.da_spmm_release()
    da.da_spmm_features(a.m, N, prob.rowptr)
    plain = error()
    da.da_spmm_prepare(a.m, a.k, a.nnz, prob.rowptr, prob.colind)
    planned = error()
    da.da_spmm_release()
    print(f"N={N}: {plain:.2e} without a plan, {planned:.2e} with one", flush=True)
    assert planned <= 1.15 * plain
