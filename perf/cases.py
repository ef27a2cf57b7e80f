"""Performance cases of the sparse x dense product on one GPU: what a program that uses this library
has it do, through the public entry points.

A case is a dict of plain values: the call (see CALLS), the sparsity law of the matrix with its sizes
(see row_lengths), and the width N of the dense operands.  The laws are those of
paper_2202_08556_amd.generators, drawn on the GPU: row lengths are the quantiles of the law in a
seeded order, so that the number of stored entries follows from the case alone, and the columns of a
row are distinct and sorted.

CALLS
  spmm       C = A.B with da_spmm on a matrix that was analysed once (features, selection,
             preparation), as an iterative method or a trained model does call after call
  ex         the same with da_spmm_ex: operands stored column-major (a block of vectors side by
             side) or as some columns of a wider row-major array
  infer      two GraphConv layers, forward only: scores of all nodes of a graph
  train      one GraphConv layer without activation, forward and backward: gradients of features,
             weight and bias; the backward product runs on the transposed matrix
  batch      a matrix that is new in every pass (a sampled neighbourhood): SparseGraph from its
             CSR arrays, aggregation forward and backward
  transpose  CSR arrays of A^T with da_csr_transpose
"""
import math

import torch

from paper_2202_08556_amd import binding as da
from paper_2202_08556_amd import gcn

CALLS = ("spmm", "ex", "infer", "train", "batch", "transpose")


def listed():
    return [
        # the smallest call: a few thousand short rows and 8 right-hand sides; launches count
        dict(name="uniform_4096_n8", call="spmm", law="poisson", m=4096, k=4096, mean=8.0, N=8),
        # an ordinary call: a matrix of odd size with rows of moderately uneven length
        dict(name="lognormal_61417_n64", call="spmm", law="lognormal", m=61417, k=61417, mean=23.0, cv=1.3, N=64),
        # a graph with a heavy-tailed degree distribution and popular columns, narrow features
        dict(name="powerlaw_262144_n32", call="spmm", law="powerlaw", m=262144, k=262144, scale=6.8, max_len=4096, N=32),
        # the same graph with wide features: the benchmark's default workload
        dict(name="powerlaw_262144_n128", call="spmm", law="powerlaw", m=262144, k=262144, scale=6.8, max_len=4096, N=128),
        # a discretised operator on a 3-D grid times a block of vectors
        dict(name="stencil_64x128x128_n32", call="spmm", law="stencil", nx=64, ny=128, nz=128, N=32),
        # nearly all rows tiny, one in a thousand enormous; few and many right-hand sides
        dict(name="skewed_524288_n8", call="spmm", law="skewed", m=524288, k=524288, heavy=524, lo=20000, hi=100000,
             mean=4.0, N=8),
        dict(name="skewed_524288_n64", call="spmm", law="skewed", m=524288, k=524288, heavy=524, lo=20000, hi=100000,
             mean=4.0, N=64),
        # block of vectors stored one after another, as solvers that come from column-major hold them
        dict(name="stencil_64x64x64_col_n8", call="ex", law="stencil", nx=64, ny=64, nz=64, N=8, layout="col"),
        # node scores of a whole graph: 602 input features, 128 hidden, 41 classes (a ragged width)
        dict(name="gcn_infer_602_128_41", call="infer", law="powerlaw", m=262144, k=262144, scale=6.8, max_len=4096,
             fin=602, hidden=128, N=41),
        # a training step's layer on a graph of middle size
        dict(name="gcn_train_96_64", call="train", law="powerlaw", m=100003, k=100003, scale=6.8, max_len=2048,
             fin=96, N=64),
        # mini-batch training: a sampled block of a graph, used once
        dict(name="batch_8192x65536_n64", call="batch", law="lognormal", m=8192, k=65536, mean=15.0, cv=0.5, N=64),
        # once per graph, for its backward pass
        dict(name="transpose_262144", call="transpose", law="powerlaw", m=262144, k=262144, scale=6.8, max_len=4096, N=1),
    ]


# ------------------------------------------------------------------------------------------------
# drawn cases
# ------------------------------------------------------------------------------------------------
MAX_PRODUCTS = 1.7e9          # stored entries times N of the largest products
MAX_ENTRIES = 2.8e7
MAX_DENSE = 4.0e7             # elements of the dense operands B and C together


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _law(rng, entries, square):
    """A sparsity law with about `entries` stored entries."""
    law = rng.choice(["poisson", "lognormal", "lognormal", "powerlaw", "powerlaw", "stencil", "skewed", "hypersparse"])
    if law == "stencil":
        side = (entries / 27.0) ** (1.0 / 3.0)
        a, b = rng.uniform(0.6, 1.5), rng.uniform(0.7, 1.4)
        return dict(law=law, nx=max(4, round(side * a)), ny=max(4, round(side * b)), nz=max(4, round(side / (a * b))))
    if law == "powerlaw":
        scale = rng.uniform(2.0, 8.0)
        m = max(1000, round(entries / (scale * 7.0)))
        return dict(law=law, m=m, k=m, scale=round(scale, 2), max_len=max(64, min(4096, m // 32)))
    if law == "skewed":
        m = max(2000, round(entries / 60))
        heavy = max(1, round(m * 1e-3))
        mid = min(entries * 0.9 / heavy, m / 6)
        return dict(law=law, m=m, k=m, heavy=heavy, lo=max(1, round(mid * 0.4)), hi=max(2, round(mid * 1.6)),
                    mean=round(rng.uniform(1.0, 6.0), 2))
    if law == "hypersparse":
        mean = _log(rng, 8, 200)
        stored = max(4, round(entries / mean))
        m = min(1500000, round(stored * _log(rng, 10, 200)))
        return dict(law=law, m=m, k=max(2000, m // 8), stored=min(stored, m), mean=round(mean, 1))
    mean = _log(rng, 2, 200)
    m = max(200, round(entries / mean))
    k = m if square or rng.random() < 0.7 else max(1000, round(m * _log(rng, 0.2, 5)))
    out = dict(law=law, m=m, k=max(k, 4 * round(mean)), mean=round(mean, 2))
    if law == "lognormal":
        out["cv"] = round(_log(rng, 0.1, 4.0), 3) if rng.random() < 0.85 else 0.0
    return out


def draw(rng):
    """One more case of the same ranges: 2e4 to 2.8e7 stored entries, N from 1 to 256."""
    while True:
        call = rng.choice(["spmm"] * 9 + ["ex"] * 2 + ["infer"] * 2 + ["train"] * 2 + ["batch"] * 2 + ["transpose"] * 3)
        entries = _log(rng, 2e4, MAX_ENTRIES if call in ("spmm", "transpose") else 1e7)
        c = dict(call=call)
        if call == "batch":
            m = round(_log(rng, 500, 30000))
            c.update(law="lognormal", m=m, k=round(m * _log(rng, 2, 12)), mean=round(rng.uniform(4, 30), 1),
                     cv=round(rng.uniform(0.0, 1.0), 2))
        else:
            c.update(_law(rng, entries, call in ("infer", "train")))
        # widths: powers of two, multiples of 4 and odd ones
        lo, hi = (8, 128) if call in ("infer", "train", "batch") else (1, 32 if call == "ex" else 256)
        n = _log(rng, lo, hi + 0.99)
        c["N"] = rng.choice([2 ** round(math.log2(n)), max(4, 4 * round(n / 4)), int(n), int(n)])
        if call == "ex":
            c["layout"] = rng.choice(["col", "wide"])
        elif call == "infer":
            c.update(fin=rng.randrange(16, 257), hidden=rng.choice([16, 32, 64, 100, 128]))
        elif call == "train":
            c["fin"] = rng.randrange(16, 129)
        elif call == "transpose":
            c["N"] = 1
        m, k = _shape(c)
        nnz = _entries(c)
        widest = max(c["N"], c.get("hidden", 0))
        cap = MAX_PRODUCTS / {"infer": 3, "train": 3, "batch": 2, "ex": 10}.get(call, 1)
        if 1 <= nnz <= MAX_ENTRIES and nnz * widest <= cap and (m + k) * max(widest, c.get("fin", 0)) <= MAX_DENSE:
            return c


# ------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------
def _shape(c):
    if c["law"] == "stencil":
        m = c["nx"] * c["ny"] * c["nz"]
        return m, m
    return c["m"], c["k"]


def row_lengths(c):
    """Lengths of the rows in ascending or descending order of the law's quantiles (float64, CPU)."""
    m, k = _shape(c)
    u = (torch.arange(m, dtype=torch.float64) + 0.5) / m
    if c["law"] == "powerlaw":           # P(length >= d) = scale / d
        lens = torch.floor(c["scale"] / u).clamp(1, min(c["max_len"], k))
    elif c["law"] == "skewed":
        lens = _poisson(u, c["mean"])
        h = c["heavy"]
        lens[:h] = torch.round(c["lo"] + (c["hi"] - c["lo"]) * (torch.arange(h, dtype=torch.float64) + 0.5) / h)
    elif c["law"] == "hypersparse":      # most rows are empty
        lens = torch.zeros(m, dtype=torch.float64)
        s = c["stored"]
        lens[:s] = 1 + _poisson((torch.arange(s, dtype=torch.float64) + 0.5) / s, max(c["mean"] - 1, 0.0))
    elif c["law"] == "poisson":
        lens = _poisson(u, c["mean"])
    elif c["cv"] <= 0:                   # lognormal without spread: rows of one length
        lens = torch.full((m,), float(round(c["mean"])), dtype=torch.float64)
    else:
        s2 = math.log1p(c["cv"] ** 2)
        lens = torch.round(torch.exp(math.log(c["mean"]) - 0.5 * s2 + math.sqrt(s2) * torch.special.ndtri(u)))
    return lens.clamp(0, k // 2)


def _poisson(u, mean):
    """Quantiles of a Poisson law, by its normal approximation."""
    return torch.round(mean + math.sqrt(mean) * torch.special.ndtri(u)).clamp(min=0)


def _entries(c):
    if c["law"] == "stencil":
        return (3 * c["nx"] - 2) * (3 * c["ny"] - 2) * (3 * c["nz"] - 2)
    return int(row_lengths(c).sum())


def _stencil(c, dev):
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    m = nx * ny * nz
    i = torch.arange(m, device=dev)
    x, y, z = i % nx, (i // nx) % ny, i // (nx * ny)
    d = torch.tensor([(a, b, e) for e in (-1, 0, 1) for b in (-1, 0, 1) for a in (-1, 0, 1)], device=dev)
    inside = torch.ones((m, 27), dtype=torch.bool, device=dev)
    for pos, n, col in ((x, nx, 0), (y, ny, 1), (z, nz, 2)):
        q = pos[:, None] + d[None, :, col]
        inside &= (q >= 0) & (q < n)
    cols = i[:, None] + (d[:, 0] + nx * (d[:, 1] + ny * d[:, 2]))[None, :]
    return inside.sum(1), cols[inside].to(torch.int32)


def _columns(rows, k, popular, gen, dev):
    """One column for each entry of `rows` (ascending), distinct inside a row and sorted.  popular:
    rank r is drawn with probability ~ 1/r and the ranks are scattered over the columns."""
    perm = torch.randperm(k, generator=gen, device=dev) if popular else None

    def some(n):
        u = torch.rand(n, generator=gen, device=dev, dtype=torch.float64)
        if not popular:
            return (u * k).long().clamp_(max=k - 1)
        return perm[((k + 1.0) ** u).long().clamp_(1, k) - 1]

    keys = torch.sort(rows * k + some(rows.numel()))[0]
    for _ in range(24):                  # entries that repeat a column of their row draw another one
        again = torch.zeros(keys.numel(), dtype=torch.bool, device=dev)
        again[1:] = keys[1:] == keys[:-1]
        repeated = keys[again]
        if repeated.numel() == 0:
            break
        keys[again] = repeated // k * k + some(repeated.numel())
        keys = torch.sort(keys)[0]
    return (keys % k).to(torch.int32)


def _csr(c, gen, dev):
    m, k = _shape(c)
    if c["law"] == "stencil":
        lens, colind = _stencil(c, dev)
    else:
        lens = row_lengths(c).long().to(dev)[torch.randperm(m, generator=gen, device=dev)]
        rows = torch.repeat_interleave(torch.arange(m, device=dev), lens)
        colind = _columns(rows, k, c["law"] == "powerlaw", gen, dev)
    rowptr = torch.zeros(m + 1, dtype=torch.int32, device=dev)
    rowptr[1:] = torch.cumsum(lens, 0).to(torch.int32)
    if c["law"] == "powerlaw":           # row-normalised adjacency
        vals = torch.repeat_interleave(1.0 / lens.to(torch.float32), lens)
    else:
        vals = torch.rand(colind.numel(), generator=gen, device=dev) * 2 - 1
    return rowptr, colind, vals


class _Analysed:
    """A matrix that a program keeps: its CSR arrays, analysed once."""

    def __init__(self, m, k, N, rowptr, colind, vals):
        self.m, self.k, self.rowptr, self.colind, self.vals = m, k, rowptr, colind, vals
        self.algo = da.da_spmm_select(da.da_spmm_features(m, N, rowptr))
        da.da_spmm_prepare(m, k, colind.numel(), rowptr, colind)

    def __del__(self):
        try:
            da.da_spmm_release(self.rowptr)
        except Exception:                # at the interpreter's end
            pass


def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    m, k = _shape(case)
    N, call = case["N"], case["call"]
    rowptr, colind, vals = _csr(case, gen, dev)
    nnz = colind.numel()
    s = dict(case=dict(case), m=m, k=k, nnz=nnz, N=N)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=dev)

    if call == "spmm":
        s.update(A=_Analysed(m, k, N, rowptr, colind, vals), B=normal(k, N), C=torch.empty((m, N), device=dev))
    elif call == "ex":
        s["A"] = _Analysed(m, k, N, rowptr, colind, vals)
        if case["layout"] == "col":      # N vectors of length k, N vectors of length m
            s.update(B=normal(N, k), ldb=k, C=torch.empty((N, m), device=dev), ldc=m, order=da.DA_COL_MAJOR)
        else:                            # the first N columns of arrays that hold more of them
            pitch = (N + 3) // 4 * 4 + 16
            s.update(B=normal(k, pitch), ldb=pitch, C=torch.empty((m, pitch), device=dev), ldc=pitch, order=da.DA_ROW_MAJOR)
    elif call in ("infer", "train"):
        s["graph"] = gcn.SparseGraph(m, k, rowptr, colind, vals)
        widths = [case["fin"], case["hidden"], N] if call == "infer" else [case["fin"], N]
        layers = []
        for i in range(len(widths) - 1):
            layer = gcn.GraphConv(widths[i], widths[i + 1], relu=i < len(widths) - 2).to(dev)
            with torch.no_grad():
                layer.weight.copy_(normal(widths[i], widths[i + 1]) / math.sqrt(widths[i]))
                layer.bias.copy_(0.1 * normal(widths[i + 1]))
            layers.append(layer)
        s.update(layers=layers, X=normal(k, case["fin"]))
        if call == "train":
            s["X"].requires_grad_(True)
            s["dY"] = normal(m, N)
    elif call == "batch":
        s.update(csr=(rowptr, colind, vals), X=normal(k, N).requires_grad_(True), dY=normal(m, N))
    elif call == "transpose":
        size = da.da_csr_transpose_workspace(m, k, nnz)
        s.update(csr=(rowptr, colind, vals), size=size, work=torch.empty(size, dtype=torch.uint8, device=dev),
                 out=(torch.empty(k + 1, dtype=torch.int32, device=dev), torch.empty_like(colind), torch.empty_like(vals)))
    return s


def run(state):
    s = state
    call = s["case"]["call"]
    if call == "spmm":
        A = s["A"]
        da.da_spmm(s["m"], s["k"], s["N"], A.rowptr, A.colind, A.vals, s["B"], s["C"], A.algo)
        return s["C"]
    if call == "ex":
        A = s["A"]
        da.da_spmm_ex(s["m"], s["k"], s["N"], A.rowptr, A.colind, A.vals, s["B"], s["ldb"], s["order"], s["C"], s["ldc"],
                      s["order"], A.algo)
        return s["C"] if s["order"] == da.DA_COL_MAJOR else s["C"][:, :s["N"]]
    if call == "infer":
        with torch.no_grad():
            first, second = s["layers"]
            return second(s["graph"], first(s["graph"], s["X"]))
    if call == "train":
        layer = s["layers"][0]
        Y = layer(s["graph"], s["X"])
        return Y.detach(), torch.autograd.grad(Y, (s["X"], layer.weight, layer.bias), s["dY"])
    if call == "batch":
        graph = gcn.SparseGraph(s["m"], s["k"], *s["csr"])
        Y = gcn.aggregate(graph, s["X"])
        return Y.detach(), torch.autograd.grad(Y, s["X"], s["dY"])
    rowptr, colind, vals = s["csr"]
    da.da_csr_transpose(s["m"], s["k"], s["nnz"], rowptr, colind, vals, *s["out"], s["work"], s["size"])
    return s["out"]


def work(case):
    m, k = _shape(case)
    N, call, nnz = case["N"], case["call"], _entries(case)
    A, At = 4 * (m + 1) + 8 * nnz, 4 * (k + 1) + 8 * nnz
    if call in ("spmm", "ex"):
        return {"bytes": A + 4 * (k + m) * N, "flops": 2 * nnz * N}
    if call == "infer":
        fin, hid = case["fin"], case["hidden"]
        return {"bytes": A + 4 * (k * fin + fin * hid + hid + hid * N + N + m * N),
                "flops": 2 * k * (fin * hid + hid * N) + 2 * nnz * (hid + N)}
    if call == "train":
        fin = case["fin"]
        return {"bytes": A + At + 4 * (2 * k * fin + 2 * fin * N + 2 * N + 2 * m * N), "flops": 6 * k * fin * N + 4 * nnz * N}
    if call == "batch":
        return {"bytes": A + 4 * (2 * k * N + 2 * m * N), "flops": 4 * nnz * N}
    return {"bytes": A + At, "flops": 0}


def tolerance(case):
    # the transpose moves values and computes none; everything else sums in fp32
    return "exact" if case["call"] == "transpose" else {"rel": 1e-5}
