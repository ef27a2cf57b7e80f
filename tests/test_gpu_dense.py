"""Dense parts of the graph-convolution layer (da_spmm_weight_grad, _column_sums, _bias_relu, _dense) at the edges
of their tiles against float64 on the CPU, and the fused layer against the separate operations."""
import numpy as np
import pytest
import torch

from paper_2202_08556_amd import generators as gen

pytestmark = pytest.mark.gpu

SHAPES = [(1, 4, 4), (15, 5, 7), (17, 64, 64), (63, 65, 63), (64, 16, 128), (129, 130, 41), (1000, 97, 48), (4099, 33, 96),
          (20001, 128, 17), (7, 256, 100)]


def close(got, want, n):
    scale = np.sqrt(n) * max(1e-30, float(np.abs(want).max()))
    assert np.max(np.abs(got.double().cpu().numpy() - want)) <= 2e-6 * scale, np.max(np.abs(got.double().cpu().numpy() - want))


@pytest.mark.parametrize("rows,fin,fout", SHAPES)
def test_weight_grad_column_sums_and_dense(rows, fin, fout):
    from paper_2202_08556_amd import binding as da
    print(f"dense rows={rows} fin={fin} fout={fout}", flush=True)
    g = torch.Generator().manual_seed(rows)
    ldx, ldg = fin + rows % 3, fout + rows % 2
    X, G = torch.randn((rows, ldx), generator=g), torch.randn((rows, ldg), generator=g)
    X[:, fin:], G[:, fout:] = float("nan"), float("nan")          # padding: never part of a result
    W = torch.randn((fin, fout), generator=g)
    x, gg = X[:, :fin].double().numpy(), G[:, :fout].double().numpy()
    Xd, Gd, Wd = X.cuda(), G.cuda(), W.cuda()
    dW = torch.full((fin, fout), float("nan"), device="cuda")
    size = da.da_spmm_weight_grad_workspace(rows, fin, fout)
    da.da_spmm_weight_grad(rows, fin, fout, Xd, ldx, Gd, ldg, dW, torch.full((size,), 255, dtype=torch.uint8, device="cuda"), size)
    close(dW, x.T @ gg, rows)
    sums = torch.full((fout,), float("nan"), device="cuda")
    size = da.da_spmm_column_sums_workspace(rows, fout)
    da.da_spmm_column_sums(rows, fout, Gd, ldg, sums, torch.full((size,), 255, dtype=torch.uint8, device="cuda"), size)
    close(sums, gg.sum(0), rows)
    for transposed in (False, True):
        C = torch.full((rows, fout + 3), -7.0, device="cuda")
        w = Wd.t().contiguous() if transposed else Wd
        da.da_spmm_dense(rows, fin, fout, Xd, ldx, w, *((1, fin) if transposed else (fout, 1)), C, fout + 3)
        close(C[:, :fout], x @ W.double().numpy(), fin)
        assert (C[:, fout:] == -7.0).all()
    for bias in (None, torch.randn(fout, generator=g)):
        for relu in (False, True):
            Z = torch.randn((rows, fout), generator=g)
            want = Z + bias if bias is not None else Z.clone()
            want = torch.relu(want) if relu else want
            Zd = Z.cuda()
            da.da_spmm_bias_relu(rows, fout, Zd, None if bias is None else bias.cuda(), relu)
            assert torch.equal(Zd.cpu(), want)


def test_dense_errors():
    from paper_2202_08556_amd import binding as da
    t = torch.zeros(4096, device="cuda")
    for call in (lambda: da.da_spmm_dense(4, 257, 4, t, 257, t, 4, 1, t, 4), lambda: da.da_spmm_dense(4, 8, 4, t, 7, t, 4, 1, t, 4),
                 lambda: da.da_spmm_weight_grad(4, 3, 8, t, 3, t, 8, t, t, 1 << 30),
                 lambda: da.da_spmm_weight_grad(4, 8, 8, t, 8, t, 8, t, t, 4)):
        with pytest.raises(da.DaSpmmError):
            call()


@pytest.mark.parametrize("fin,fout,relu,bias", [(48, 32, True, True), (3, 5, True, True), (130, 41, False, True), (260, 8, True, False),
                                                (16, 2, False, False)])
def test_fused_layer_matches_separate_operations(fin, fout, relu, bias):
    from paper_2202_08556_amd import gcn
    a = gen.powerlaw_csr(m=1500, seed=77)
    torch.manual_seed(fin)
    graph = gcn.SparseGraph.from_numpy(a)
    layer = gcn.GraphConv(fin, fout, bias=bias, relu=relu).cuda()
    if bias:
        with torch.no_grad():
            layer.bias.uniform_(-0.5, 0.5)
    X = torch.randn((a.m, fin), device="cuda", requires_grad=True)
    dY = torch.randn((a.m, fout), device="cuda")
    params = [X] + list(layer.parameters())
    got = layer(graph, X)
    g_got = torch.autograd.grad(got, params, dY, retain_graph=True)
    g_again = torch.autograd.grad(got, params, dY)
    Z = gcn.aggregate(graph, X @ layer.weight)
    Z = Z + layer.bias if bias else Z
    want = torch.relu(Z) if relu else Z
    g_want = torch.autograd.grad(want, params, torch.where(got > 0, dY, torch.zeros_like(dY)) if relu else dY)
    assert torch.allclose(got, want, rtol=1e-4, atol=1e-5)
    for p, q, r in zip(g_got, g_want, g_again):
        assert p.shape == q.shape and torch.allclose(p, q, rtol=1e-3, atol=1e-4 * float(q.abs().max()))
        assert torch.allclose(p, r, rtol=1e-4, atol=1e-5 * float(q.abs().max()))
    with torch.no_grad():
        assert not layer(graph, X).requires_grad


def test_graph_outside_plain_backward_differentiation():
    """Tangents and function transforms are refused, subclasses and lazy negation honoured, a graph's arrays can be
    replaced and a graph copied."""
    import copy
    import pickle

    import torch.autograd.forward_ad as fwd
    from paper_2202_08556_amd import gcn
    a = gen.powerlaw_csr(m=700, seed=5)
    graph = gcn.SparseGraph.from_numpy(a)
    layer = gcn.GraphConv(12, 8).cuda()
    X = torch.randn((a.m, 12), device="cuda")
    Y = gcn.aggregate(graph, X)
    with fwd.dual_level():
        dual = fwd.make_dual(X, torch.ones_like(X))
        for f in (lambda t: gcn.aggregate(graph, t), lambda t: layer(graph, t)):
            with pytest.raises((RuntimeError, NotImplementedError)):
                f(dual)
    with pytest.raises((RuntimeError, NotImplementedError)):
        torch.func.vmap(lambda t: gcn.aggregate(graph, t))(torch.stack([X, X]))

    class Marked(torch.Tensor):
        seen = 0

        @classmethod
        def __torch_function__(cls, func, types, args=(), kwargs=None):
            cls.seen += func in (torch.Tensor.matmul, torch.Tensor.__matmul__, torch.matmul)
            return super().__torch_function__(func, types, args, kwargs or {})

    with torch.no_grad():
        want = layer(graph, X)
        assert torch.allclose(layer(graph, X.as_subclass(Marked)).as_subclass(torch.Tensor), want, rtol=1e-4, atol=1e-5)
        assert Marked.seen == 1
        assert torch.allclose(gcn.aggregate(graph, torch._neg_view(X)), -Y, rtol=1e-4, atol=1e-6)
    for twin in (copy.deepcopy(graph), pickle.loads(pickle.dumps(graph))):
        assert torch.allclose(gcn.aggregate(twin, X), Y, rtol=1e-4, atol=1e-6)
    graph.vals = graph.vals * 2
    assert torch.allclose(gcn.aggregate(graph, X), 2 * Y, rtol=1e-4, atol=1e-6)


# either side of the lines between the fp32 kernel, the one of bf16 pieces and the GEMM library
@pytest.mark.parametrize("rows,fin,fout,way", [
    (1000, 128, 128, "dense_product"), (70000, 128, 128, "dense_split"), (1000, 256, 16, "dense_product"), (100000, 256, 16, "dense_product"),
    (10000, 200, 41, "dense_product"), (20000, 200, 41, "dense_split"), (100, 256, 64, "dense_split"), (20000, 256, 256, "dense_split"),
    (11000, 300, 128, "library"), (12000, 300, 128, "dense_split"), (9000, 300, 64, "dense_split"), (8000, 300, 64, "library"), (40000, 300, 513, "library"),
    (60000, 200, 193, "dense_split"), (4000, 31, 300, "dense_product")])
def test_ways_of_the_dense_product(rows, fin, fout, way):
    from paper_2202_08556_amd import gcn
    from tests.gpu_util import kernels_of
    print(f"dense {rows} x {fin} x {fout}", flush=True)
    picked = torch.tensor([0, 1, rows // 2, rows - 1], dtype=torch.int32, device="cuda")
    graph = gcn.SparseGraph(4, rows, torch.arange(5, dtype=torch.int32, device="cuda"), picked, torch.ones(4, device="cuda"))
    layer = gcn.GraphConv(fin, fout, bias=False, relu=False).cuda()
    X = torch.randn((rows, fin), device="cuda")
    with torch.no_grad():
        got = layer(graph, X)
        names = kernels_of(lambda: layer(graph, X))
    x = X[picked.long()].double()
    want, size = x @ layer.weight.double(), x.abs() @ layer.weight.double().abs()
    assert ((got - want).abs() <= (3 + fin ** 0.5) * 2.0 ** -24 * size).all()
    ours = [w for w in ("dense_product", "dense_split") if any(w + "_kernel" in n for n in names)]
    assert ours == ([] if way == "library" else [way]), names
