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
