"""Graphs and layers at the edges of what a caller may do with them: one row, sizes beyond the own kernels, operands
changed or dropped between forward and backward, graphs that are not plain, threads, captures, copies, errors."""
import numpy as np
import pytest
import torch

from paper_2202_08556_amd import generators as gen

pytestmark = pytest.mark.gpu


def graph_of(a):
    from paper_2202_08556_amd import gcn
    return gcn.SparseGraph.from_numpy(a)


def dense(a):
    d = torch.zeros((a.m, a.k), dtype=torch.float64)
    for i in range(a.m):
        for p in range(a.rowptr[i], a.rowptr[i + 1]):
            d[i, a.colind[p]] += float(a.vals[p])
    return d


def matrix(m, k, seed=1):
    """A small matrix without empty rows."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, max(2, k // 2), size=m)
    rowptr, colind = gen.csr_from_lens(rng, lens, k)
    return gen.CSR(m, k, rowptr.astype(np.int32), colind.astype(np.int32),
                   rng.uniform(-1, 1, colind.size).astype(np.float32), "small", seed)


def near(got, want):
    """Sums of a few hundred fp32 products against float64: 1e-5 of the largest value is a hundred roundings."""
    want = want.double().cpu()
    return got.shape == want.shape and bool((got.detach().double().cpu() - want).abs().max() <= 1e-5 * max(1.0, float(want.abs().max())))


def layer_of(fin, fout, **kw):
    from paper_2202_08556_amd import gcn
    torch.manual_seed(fin * 1000 + fout)
    layer = gcn.GraphConv(fin, fout, **kw).cuda()
    if layer.bias is not None:
        with torch.no_grad():
            layer.bias.uniform_(-0.5, 0.5)
    return layer


# ---- one row --------------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("m,k", [(7, 1), (1, 9), (1, 1)])
@pytest.mark.parametrize("n", [1, 5, 40])
def test_operands_of_one_row(m, k, n):
    """torch gives a contiguous tensor of one row any row stride: a transposed column, the gradient of a sum."""
    from paper_2202_08556_amd import gcn
    a = matrix(m, k)
    A, graph = dense(a), graph_of(a)
    col = torch.randn((n, k), device="cuda")
    X = col.t().requires_grad_(True)                          # k x n, strides (1, k)
    for dY in (None, torch.randn((n, m), device="cuda").t()):
        Y = gcn.aggregate(graph, X)
        gx, = torch.autograd.grad(Y.sum() if dY is None else Y, X, dY)
        assert near(Y, A @ X.detach().double().cpu())
        assert near(gx, A.t() @ (torch.ones((m, n)) if dY is None else dY).double().cpu())
    layer = layer_of(6, n, relu=False)
    x = torch.randn((6, k), device="cuda").t().requires_grad_(True)
    W, b = layer.weight.detach().double().cpu(), layer.bias.detach().double().cpu()
    for dY in (None, torch.randn((n, m), device="cuda").t()):
        Y = layer(graph, x)
        assert near(Y, A @ (x.detach().double().cpu() @ W) + b)
        gx, gw, gb = torch.autograd.grad(Y.sum() if dY is None else Y, (x, layer.weight, layer.bias), dY)
        d = (torch.ones((m, n)) if dY is None else dY).double().cpu()
        assert near(gx, (A.t() @ d) @ W.t()) and near(gw, x.detach().double().cpu().t() @ (A.t() @ d)) and near(gb, d.sum(0))


# ---- what a layer keeps for its backward pass ------------------------------------------------------------------------
def test_layer_keeps_only_what_its_gradients_need():
    a = gen.powerlaw_csr(m=1500, seed=3)
    graph, layer = graph_of(a), layer_of(24, 16)
    X = torch.randn((a.m, 24), device="cuda")
    dY = torch.randn((a.m, 16), device="cuda")
    params = (layer.weight, layer.bias)
    want = torch.autograd.grad(layer(graph, X), params, dY)
    Y = layer(graph, X)                                       # W changes, and its gradient does not need it
    with torch.no_grad():
        layer.weight.mul_(1.25)
    for g, w in zip(torch.autograd.grad(Y, params, dY), want):
        assert torch.allclose(g, w, rtol=1e-5, atol=1e-5)
    layer.weight.requires_grad_(False)
    leaf = X.clone().requires_grad_(True)
    want, = torch.autograd.grad(layer(graph, leaf), leaf, dY)
    middle = leaf * 1.0
    Y = layer(graph, middle)                                  # X changes, and its gradient does not need it
    with torch.no_grad():
        middle.zero_()
    got, = torch.autograd.grad(Y, leaf, dY)
    assert torch.allclose(got, want, rtol=1e-5, atol=1e-5)
    with torch.inference_mode():
        frozen = X * 1.0
    Y = layer(graph, frozen)                                  # only the bias is trained
    torch.autograd.grad(Y, layer.bias, dY)
    torch.cuda.synchronize()
    big = torch.randn((a.m, 24), device="cuda")
    Y = layer(graph, big)
    before = torch.cuda.memory_allocated()
    del big
    assert before - torch.cuda.memory_allocated() >= a.m * 24 * 4
    torch.autograd.grad(Y, layer.bias, dY)


def test_changes_that_a_gradient_depends_on_are_refused():
    a = gen.powerlaw_csr(m=600, seed=4)
    graph, layer = graph_of(a), layer_of(8, 8)
    X = torch.randn((a.m, 8), device="cuda", requires_grad=True)
    dY = torch.randn((a.m, 8), device="cuda")
    Y = layer(graph, X)
    with torch.no_grad():
        layer.weight.mul_(1.25)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        torch.autograd.grad(Y, X, dY)
    Y = layer(graph, X)
    torch.autograd.grad(Y, X, dY)
    with pytest.raises(RuntimeError, match="second time"):
        torch.autograd.grad(Y, X, dY)


# ---- threads ---------------------------------------------------------------------------------------------------------
def test_arrays_replaced_while_another_thread_multiplies():
    """A product sees the arrays of one moment and keeps them alive: each result is that of the old or the new values."""
    import threading

    from paper_2202_08556_amd import gcn
    a = gen.powerlaw_csr(m=900, seed=6)
    graph = graph_of(a)
    vals = graph.vals.clone()
    X = torch.randn((a.m, 32), device="cuda")
    want = gcn.aggregate(graph, X)
    done, results, errors = threading.Event(), [], []

    def multiply():
        try:
            for _ in range(200):
                results.append(gcn.aggregate(graph, X))
        except BaseException as exc:
            errors.append(exc)
        finally:
            done.set()

    worker = threading.Thread(target=multiply)
    worker.start()
    i = 0
    while not done.is_set():
        graph.vals = vals * (1 + i % 2)                       # the array set before is dropped here
        assert graph.vals.shape == vals.shape and graph.nnz == a.nnz
        i += 1
    worker.join()
    assert not errors and len(results) == 200
    for Y in results:
        assert torch.allclose(Y, want, rtol=1e-4, atol=1e-5) or torch.allclose(Y, 2 * want, rtol=1e-4, atol=1e-5)


# ---- captures --------------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("given", [None, 4])
def test_capture_after_one_pass(given):
    """The second EB product of a graph prepares it, which a capture must not: it goes without."""
    from paper_2202_08556_amd import gcn
    a = gen.skewed_csr(m=16384, heavy_lo=3000, heavy_hi=9000, seed=4001)
    graph, layer = graph_of(a), layer_of(12, 24)
    X = torch.randn((a.m, 24), device="cuda")
    x = torch.randn((a.m, 12), device="cuda", requires_grad=True)
    dY = torch.randn((a.m, 24), device="cuda")
    assert graph.algo_for(24) >= 4

    def passes():
        if given is not None:
            return [graph.spmm(X, given)]
        Y = layer(graph, x)
        return [Y.detach(), *torch.autograd.grad(Y, (x, layer.weight, layer.bias), dY)]

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        if given is None:
            passes()
    side.synchronize()
    held = torch.cuda.CUDAGraph()
    with torch.cuda.graph(held, stream=side):
        outs = passes()
    assert not graph._g.prepared
    for _ in range(3):
        for o in outs:
            o.fill_(float("nan"))
        want = passes()                                       # eager work between the replays, which prepares
        torch.cuda.synchronize()
        held.replay()
        torch.cuda.synchronize()
        for o, w in zip(outs, want):
            assert torch.allclose(o, w, rtol=1e-3, atol=1e-5 * float(w.abs().max()))
    assert graph._g.prepared


def test_features_are_refused_in_a_capture_and_wait_for_no_other_stream():
    """Nothing is recorded for them, and new scratch is cleared on the stream of its call."""
    from concurrent.futures import ThreadPoolExecutor

    from oracle import reference as orc
    from paper_2202_08556_amd import binding as da
    a = gen.powerlaw_csr(m=5000, seed=8)
    rp = torch.from_numpy(a.rowptr).cuda()
    want = orc.features(a.rowptr, 4)
    side = torch.cuda.Stream()
    out = torch.zeros(4, device="cuda")
    held = torch.cuda.CUDAGraph()
    with torch.cuda.graph(held, stream=side):
        out.add_(1)
        with pytest.raises(da.DaSpmmError):
            da.da_spmm_features(a.m, 4, rp)
        out.add_(1)
    for _ in range(3):
        held.replay()
    torch.cuda.synchronize()
    assert out.tolist() == [6.0] * 4

    def some(i):                                              # more calls at once than idle slots are kept
        with torch.cuda.stream(torch.cuda.Stream()):
            return [da.da_spmm_features(a.m, 4, rp) for _ in range(20)]

    with ThreadPoolExecutor(12) as pool:
        for got in (f for fs in pool.map(some, range(12)) for f in fs):
            assert got["nnz"] == want["nnz"] and got["row_nnz_max"] == want["row_nnz_max"]
            assert got["row_nnz_std"] == pytest.approx(want["row_nnz_std"], rel=1e-9)


# ---- graphs with methods of their own --------------------------------------------------------------------------------
@pytest.mark.parametrize("kind", ["spmm", "transposed", "algo_for", "features", "object", "instance"])
def test_graphs_with_methods_of_their_own(kind):
    """aggregate and GraphConv go through spmm and transposed of the graph they are given, spmm through algo_for and
    algo_for through features, where a subclass or an object brings its own."""
    from paper_2202_08556_amd import gcn
    a = gen.powerlaw_csr(m=800, seed=9)
    plain = graph_of(a)
    seen = []

    class Own(gcn.SparseGraph):
        pass

    class Other:
        def spmm(self, X, algo=None):
            seen.append("object")
            return plain.spmm(X, algo)

        def transposed(self):
            return plain.transposed()

    def noting(name):
        def method(self, *args):
            seen.append(name)
            return getattr(gcn.SparseGraph, name)(self, *args)
        return method

    if kind == "object":
        graph = Other()
    else:
        graph = Own(a.m, a.k, plain.rowptr, plain.colind, plain.vals) if kind != "instance" else graph_of(a)
        if kind == "instance":
            graph.spmm = lambda X, algo=None: (seen.append(kind), gcn.SparseGraph.spmm(graph, X, algo))[1]
        else:
            setattr(Own, kind, noting(kind))
    layer = layer_of(16, 8)
    X = torch.randn((a.m, 16), device="cuda", requires_grad=True)
    dY = torch.randn((a.m, 16), device="cuda")
    for f, d in ((lambda g: gcn.aggregate(g, X), dY), (lambda g: layer(g, X), dY[:, :8])):
        del seen[:]
        got, want = f(graph), f(plain)
        g_got, g_want = torch.autograd.grad(got, X, d), torch.autograd.grad(want, X, d)
        assert kind in seen
        assert torch.allclose(got, want, rtol=1e-4, atol=1e-5) and torch.allclose(g_got[0], g_want[0], rtol=1e-4, atol=1e-5)


# ---- sizes beyond the own dense kernels ------------------------------------------------------------------------------
@pytest.mark.parametrize("fin,fout", [(4, 2 ** 22 + 3), (65600, 4160), (448, 512), (449, 512)],
                         ids=["columns", "tiles", "56_tiles", "64_tiles"])
def test_layers_beyond_the_own_dense_kernels(fin, fout):
    """More columns than the kernels take, more tiles of a weight gradient than a grid holds, and both sides of the
    number of tiles from which the library is faster."""
    a = matrix(5, 6)
    A, graph, layer = dense(a).float().cuda(), graph_of(a), layer_of(fin, fout, relu=False)
    X = torch.randn((a.k, fin), device="cuda", requires_grad=True)
    Y = layer(graph, X)
    dY = torch.randn((a.m, fout), device="cuda")
    gx, gw, gb = torch.autograd.grad(Y, (X, layer.weight, layer.bias), dY)
    with torch.no_grad():
        dH = A.t() @ dY
        for got, want in ((Y, A @ (X @ layer.weight) + layer.bias), (gx, dH @ layer.weight.t()), (gw, X.t() @ dH), (gb, dY.sum(0))):
            # fp32 on both sides: sums of up to 2^22 products of either sign, a hundred roundings of the largest
            assert got.shape == want.shape and float((got - want).abs().max()) <= 1e-5 * float(want.abs().max())


# ---- copies ----------------------------------------------------------------------------------------------------------
def test_operands_are_laid_out_once():
    """A non-contiguous X or gradient costs one contiguous copy, also where several products read it."""
    from paper_2202_08556_amd import gcn
    a = gen.powerlaw_csr(m=1024, seed=11)
    graph, layer = graph_of(a), layer_of(32, 32, relu=False)
    wide = torch.randn((32, a.m), device="cuda").t()
    dense_x = wide.contiguous()
    ones = torch.ones((1, 1), device="cuda").expand(a.m, 32)
    dense_g = ones.contiguous()
    size = a.m * 32 * 4

    def allocated(f):
        f()                                                   # plans and scratch of the first calls
        f()
        before = torch.cuda.memory_stats()["allocated_bytes.all.allocated"]
        f()
        return torch.cuda.memory_stats()["allocated_bytes.all.allocated"] - before

    def aggregated(x, g):
        x = x.detach().requires_grad_(True)
        return torch.autograd.grad(gcn.aggregate(graph, x), x, g)

    def layered(x, g):
        return torch.autograd.grad(layer(graph, dense_x.requires_grad_(True)), (dense_x, layer.weight, layer.bias), g)

    both = allocated(lambda: aggregated(dense_x, dense_g))
    assert allocated(lambda: aggregated(wide, dense_g)) == both + size
    assert allocated(lambda: aggregated(dense_x, ones)) == both + size
    assert allocated(lambda: layered(dense_x, ones)) == allocated(lambda: layered(dense_x, dense_g)) + size


# ---- errors ----------------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("algo", [-1, -7, 8])
def test_algorithm_ids_outside_the_table_are_refused(algo):
    from paper_2202_08556_amd import binding as da
    a = gen.powerlaw_csr(m=300, seed=12)
    graph = graph_of(a)
    with pytest.raises(da.DaSpmmError) as err:
        graph.spmm(torch.ones((a.m, 4), device="cuda"), algo)
    assert err.value.status == da.DA_ERR_BAD_ALGO


@pytest.mark.parametrize("call", ["aggregate", "layer"])
def test_errors_of_a_backward_pass_are_the_library_s(call):
    """The transpose of a graph whose row count was spoilt after the forward pass is refused on the host."""
    from paper_2202_08556_amd import binding as da
    from paper_2202_08556_amd import gcn
    a = gen.powerlaw_csr(m=300, seed=13)
    graph, layer = graph_of(a), layer_of(4, 4)
    X = torch.randn((a.m, 4), device="cuda", requires_grad=True)
    Y = gcn.aggregate(graph, X) if call == "aggregate" else layer(graph, X)
    graph.m = -1
    with pytest.raises(da.DaSpmmError) as err:
        torch.autograd.grad(Y, X, torch.ones_like(Y))
    assert err.value.status == da.DA_ERR_INVALID_ARG


def test_operands_on_the_host_are_refused():
    from paper_2202_08556_amd import gcn
    a = gen.powerlaw_csr(m=300, seed=14)
    graph, X = graph_of(a), torch.ones((a.m, 4))
    for call in (graph.spmm, lambda x: gcn.aggregate(graph, x), lambda x: gcn._Aggregate.apply(x, graph)):
        with pytest.raises(ValueError, match="device"):
            call(X)
    with pytest.raises((ValueError, RuntimeError)):
        gcn.GraphConv(4, 4)(graph, X)                         # weights on the host too


# ---- copies of graphs and sizes ----------------------------------------------------------------------------------------
def test_copies_keep_added_attributes_and_files_of_earlier_versions_load():
    import copy
    import io
    import pickle

    from paper_2202_08556_amd import gcn
    a = gen.powerlaw_csr(m=400, seed=15)
    graph = graph_of(a)
    X = torch.randn((a.m, 8), device="cuda", requires_grad=True)
    want = gcn.aggregate(graph, X)
    graph.label = "train"
    graph.transposed()
    twins = [copy.copy(graph), copy.deepcopy(graph), pickle.loads(pickle.dumps(graph))]
    old = gcn.SparseGraph.__new__(gcn.SparseGraph)            # the attributes that an instance used to consist of
    old.__setstate__(dict(m=a.m, k=a.k, nnz=a.nnz, rowptr=graph.rowptr, colind=graph.colind, vals=graph.vals, label="train",
                          _features=dict(rows=a.m), _algo={8: 3}, _t=None, _prepared=True))
    file = io.BytesIO()
    torch.save(graph, file)
    file.seek(0)
    host = torch.load(file, map_location="cpu", weights_only=False)
    assert not host.vals.is_cuda
    for name in ("rowptr", "colind", "vals"):
        setattr(host, name, getattr(host, name).cuda())
    for twin in twins + [old, host]:
        Y = gcn.aggregate(twin, X)
        assert twin.label == "train" and torch.allclose(Y, want, rtol=1e-4, atol=1e-6)
        g, w = torch.autograd.grad(Y.sum(), X)[0], torch.autograd.grad(want.sum(), X, retain_graph=True)[0]
        assert torch.allclose(g, w, rtol=1e-4, atol=1e-5)
    assert twins[0].vals is graph.vals or twins[0].vals.data_ptr() == graph.vals.data_ptr()
    assert twins[1].vals.data_ptr() != graph.vals.data_ptr()


def test_sizes_given_as_floats():
    from paper_2202_08556_amd import gcn
    a = gen.powerlaw_csr(m=300, seed=16)
    arrays = graph_of(a)
    graph = gcn.SparseGraph(float(a.m), np.float64(a.k), arrays.rowptr, arrays.colind, arrays.vals)
    assert (graph.m, graph.k) == (a.m, a.k) and isinstance(graph.m, int)
    with pytest.raises(ValueError):
        gcn.SparseGraph(a.m + 0.5, a.k, arrays.rowptr, arrays.colind, arrays.vals)


# ---- gradients of gradients ------------------------------------------------------------------------------------------
@pytest.mark.parametrize("relu", [False, True])
def test_gradients_of_gradients_are_those_of_separate_operations(relu):
    """The dense parts stay differentiable under create_graph; the aggregation's gradient is a constant either way."""
    from paper_2202_08556_amd import gcn
    a = gen.powerlaw_csr(m=500, seed=17)
    graph, layer = graph_of(a), layer_of(6, 5, relu=relu)
    X = torch.randn((a.m, 6), device="cuda", requires_grad=True)
    dY = torch.randn((a.m, 5), device="cuda")

    def separate():
        Z = gcn.aggregate(graph, X @ layer.weight) + layer.bias
        return torch.relu(Z) if relu else Z

    results = []
    for Y in (layer(graph, X), separate()):
        gx, gw = torch.autograd.grad(Y, (X, layer.weight), dY, create_graph=True)
        assert gx.requires_grad and gw.requires_grad
        results.append((gx, gw, *torch.autograd.grad((gw ** 2).sum() + (gx ** 2).sum(), (X, layer.weight))))
    for got, want in zip(*results):
        assert torch.allclose(got, want, rtol=1e-3, atol=1e-4 * float(want.abs().max()))
