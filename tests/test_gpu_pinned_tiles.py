"""RB products whose column tiles go to XCDs of their own (2 or 4 about equal tiles, slices of B that an L2 holds a good part
of): every block of rows of every tile is taken, whatever is left over when blocks are dealt to the XCDs."""
import pytest

from oracle import reference as orc
from paper_2202_08556_amd import generators as gen

pytestmark = pytest.mark.gpu


# rows around a block's 4 (PR) and 8 ... 16 (SR) and around 8 blocks, widths around whole tiles and on both sides of the rule
@pytest.mark.parametrize("m", [1, 3, 4, 5, 15, 17, 33, 129, 1001])
@pytest.mark.parametrize("N", [119, 120, 121, 128, 130, 248, 250, 256, 512])
def test_every_row_of_every_tile(m, N):
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import DeviceProblem
    a = gen.uniform_csr(m=m, k=10007, mean_len=6.0, seed=m)
    B = gen.dense(a.k, N, "uniform", seed=N)
    want, s_abs = orc.spmm(a.rowptr, a.colind, a.vals, B)
    p = DeviceProblem(a, B)
    for algo in (da.DA_RB_RM_SR, da.DA_RB_RM_PR):
        print(f"tiles m={m} N={N} algo={algo}", flush=True)
        assert orc.tolerance_ratio(p.run(algo), want, s_abs) <= 1.0


# B and its slice of 64 columns just below and above where the rule lies
@pytest.mark.parametrize("k", [9215, 9216, 9217, 49151, 49152, 49153])
def test_around_the_rule(k):
    from paper_2202_08556_amd import binding as da
    from tests.gpu_util import DeviceProblem
    a = gen.uniform_csr(m=777, k=k, mean_len=20.0, seed=k)
    B = gen.dense(a.k, 128, "uniform", seed=1)
    want, s_abs = orc.spmm(a.rowptr, a.colind, a.vals, B)
    p = DeviceProblem(a, B)
    for algo in (da.DA_RB_RM_SR, da.DA_RB_RM_PR):
        print(f"slice k={k} algo={algo}", flush=True)
        assert orc.tolerance_ratio(p.run(algo), want, s_abs) <= 1.0
