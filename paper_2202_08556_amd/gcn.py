"""Graph-convolution layer on top of the C ABI: the application of the paper's Sec. 6, where the
data-aware SpMM replaces the framework's aggregation kernel inside GCN layers.

    Z = A . (X . W) + b,   out = relu(Z)

A is the (normalised) adjacency matrix in CSR, X the node features.  The aggregation A.H runs in
da_spmm with the algorithm the selector picks for (A, feature length); its backward pass, the
gradient A^T.dZ, runs in da_spmm on the CSR arrays of A^T, which da_csr_transpose builds once per
graph, with the algorithm the selector picks for (A^T, feature length).  The layer is one operation
forward and one backward, in C++ (csrc/native.cpp): matrix-core kernels for small weights and the
weight gradient, a plain library GEMM for large products, bias and activation in one pass.  This module
only marshals arguments; there is no fallback when the HIP library is missing (importing ``binding``
raises).
"""
from __future__ import annotations

import torch

from . import _native
from . import binding as da


class SparseGraph:
    """CSR matrix A (m x k) resident on the device, with its selector features, the algorithm
    chosen per feature length, and (built on first use) A^T.

    The matrix is prepared (da_spmm_prepare: EB chunk order and row hints) before the second product
    with an EB algorithm: the preparation costs as much as a product or more and RB algorithms do not use
    it, so a graph that is used once, a sampled mini-batch say, goes without.  It is not prepared while a HIP
    graph is captured: call prepare() (also of transposed()) or make two passes before the capture, or the
    captured products run without the chunk order.  The library keeps the plans
    of the 16 most recently prepared matrices; a program that holds more graphs than that (a graph and its
    transpose count as two) loses the oldest plans silently, which costs the EB algorithms their chunk
    order (speed), never the result."""

    def __init__(self, m: int, k: int, rowptr: torch.Tensor, colind: torch.Tensor, vals: torch.Tensor):
        if int(m) != m:                             # before the arrays' lengths are compared with whole numbers
            raise ValueError("CSR array sizes do not match")
        self._g = _native.Graph(int(m), int(k), rowptr, colind, vals)
        self._t = None

    def __getstate__(self):
        """What copies and files hold: the matrix and whatever attributes a program has added."""
        state = {name: value for name, value in self.__dict__.items() if name not in ("_g", "_t", "_algo")}
        state.update((name, getattr(self, name)) for name in ("m", "k", "nnz", "rowptr", "colind", "vals"))
        return state

    def __setstate__(self, state):
        state = dict(state)
        m, k, nnz, *arrays = (state.pop(name) for name in ("m", "k", "nnz", "rowptr", "colind", "vals"))
        for name in ("_features", "_algo", "_prepared", "_t"):       # in files of earlier versions; found again when needed
            state.pop(name, None)
        self.__dict__.update(state)
        self._g = _native.Graph(m, k, *arrays, restored=True)
        self._g.nnz = nnz
        self._t = None

    @classmethod
    def from_numpy(cls, a, device="cuda:0") -> "SparseGraph":
        """From an object with fields m, k, rowptr, colind, vals (e.g. generators.CSR)."""
        dev = torch.device(device)
        return cls(a.m, a.k, torch.from_numpy(a.rowptr).to(dev), torch.from_numpy(a.colind).to(dev),
                   torch.from_numpy(a.vals).to(dev))

    def features(self, N: int) -> dict:
        rows, nnz, mean, std, longest = self._g.features()           # one device reduction per graph
        return dict(rows=rows, nnz=nnz, row_nnz_mean=mean, row_nnz_std=std, row_nnz_max=longest, N=int(N))

    def algo_for(self, N: int) -> int:
        """Algorithm id the selector picks for this matrix and feature length (cached)."""
        if _as_written(self):
            return self._g.algo_for(int(N))
        cached = self.__dict__.setdefault("_algo", {})
        if N not in cached:
            cached[N] = da.da_spmm_select(self.features(N))
        return cached[N]

    def prepare(self) -> None:
        """Build the chunk orders of the EB algorithms now (da_spmm_prepare); released with the graph."""
        self._g.prepare()

    def transposed(self) -> "SparseGraph":
        """A^T as a SparseGraph (k x m); built once by da_csr_transpose."""
        if self._t is None:
            t = SparseGraph.__new__(SparseGraph)
            t._g = self._g.transposed()
            t._t = self
            self._t = t
        return self._t

    def spmm(self, X: torch.Tensor, algo: int | None = None) -> torch.Tensor:
        """A . X for a row-major fp32 k x N tensor on the same device; returns a new m x N tensor."""
        if algo is None and not _as_written(self):
            algo = self.algo_for(int(X.shape[1])) if X.dim() == 2 else 0
        return self._g.spmm(X, None if algo is None else int(algo))


_METHODS = frozenset(("spmm", "transposed", "algo_for", "features"))


def _as_written(graph) -> bool:
    """Whether products of `graph` may be made below its Python methods: it is a SparseGraph and neither its class
    nor the object has replaced one of them."""
    t = type(graph)
    if t is not SparseGraph and not (isinstance(graph, SparseGraph) and
                                     all(getattr(t, name) is getattr(SparseGraph, name) for name in _METHODS)):
        return False
    return _METHODS.isdisjoint(graph.__dict__)


def _field(name):
    def get(self):
        return getattr(self._g, name)

    def put(self, value):
        setattr(self._g, name, value)

    return property(get, put)


for _name in ("m", "k", "nnz", "rowptr", "colind", "vals"):
    setattr(SparseGraph, _name, _field(_name))


class _Aggregate(torch.autograd.Function):
    """The aggregation where torch has more to do than backward differentiation (tracing, function
    transforms, tangents, tensor subclasses, modes) and for graphs with products of their own (any object with
    spmm and transposed): the Function supports or refuses each of them."""

    @staticmethod
    def forward(ctx, X, graph):
        ctx.graph = graph
        return graph.spmm(X)

    @staticmethod
    def backward(ctx, dY):
        return ctx.graph.transposed().spmm(dY), None


def aggregate(graph: SparseGraph, X: torch.Tensor) -> torch.Tensor:
    """A . X with gradient A^T . dY with respect to X (A itself is a constant of the graph)."""
    if _as_written(graph) and _native.aggregate_takes(X):
        return _native.aggregate(graph._g, X)
    return _Aggregate.apply(X, graph)


class GraphConv(torch.nn.Module):
    """relu(A . (X . W) + b): one GCN layer (Sec. 6) whose aggregation is da_spmm."""

    def __init__(self, in_features: int, out_features: int, bias: bool = True, relu: bool = True):
        super().__init__()
        self.weight = torch.nn.Parameter(torch.empty(in_features, out_features))
        self.bias = torch.nn.Parameter(torch.zeros(out_features)) if bias else None
        self.relu = relu
        torch.nn.init.xavier_uniform_(self.weight)

    def forward(self, graph: SparseGraph, X: torch.Tensor) -> torch.Tensor:
        if _as_written(graph) and _native.graph_conv_takes(graph._g, X, self.weight, self.bias):
            return _native.graph_conv(graph._g, X, self.weight, self.bias, self.relu)
        Z = aggregate(graph, X @ self.weight)
        if self.bias is not None:
            Z = Z + self.bias
        return torch.relu(Z) if self.relu else Z
