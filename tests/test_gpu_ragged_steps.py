"""A row's last gathers may lie behind its end: whatever row 0 of B holds then, rows without entries in column 0 stay as they are."""
import numpy as np
import pytest
import torch

from oracle import reference as orc

pytestmark = pytest.mark.gpu


# one row length each around the blocks of 4 and 8 and the batches of 32 and 64 entries, in one matrix
@pytest.mark.parametrize("N", [1, 5, 8, 16, 20, 32, 41, 64, 128])
@pytest.mark.parametrize("algo", [0, 1, 5])
def test_row_0_of_b_does_not_reach_other_rows(N, algo):
    from paper_2202_08556_amd import binding as da
    lens = np.array(list(range(0, 36)) + [39, 40, 41, 63, 64, 65, 66, 71, 127, 129] * 3)
    k = 300
    rng = np.random.default_rng(N)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    colind = rng.integers(1, k, size=int(rowptr[-1])).astype(np.int32)
    vals = rng.choice(np.array([-2, -1, 1, 2], np.float32), colind.size)
    B = rng.integers(-4, 5, (k, N)).astype(np.float32)
    want, _ = orc.spmm(rowptr, colind, vals, B)
    B[0] = np.where(np.arange(N) % 2 == 0, np.inf, np.nan)
    dev = [torch.from_numpy(x).cuda() for x in (rowptr, colind, vals, B)]
    print(f"row 0 of B not finite, N={N} algo={algo}", flush=True)
    C = torch.full((lens.size, N), float("nan"), device="cuda")
    da.da_spmm(lens.size, k, N, *dev, C, algo)
    assert np.array_equal(C.cpu().numpy(), want.astype(np.float32) + 0.0)
