"""The native calls on torch tensors: arguments they must turn down, and gradients through other types and shapes."""
import numpy as np
import pytest

import oracle
from paper_2106_16064_amd import binding as dg
from paper_2106_16064_amd import workloads as wl


@pytest.mark.parametrize("wrong", ["host", "dtype", "length", "none"])
def test_arguments_that_are_not_the_arrays_of_a_product_raise(wrong):
    """Checked before anything is launched, so no GPU is needed to be turned down."""
    import torch
    rowptr, colidx = torch.tensor([0, 1], dtype=torch.int32), torch.zeros(1, dtype=torch.int32)
    vals, X, Y = torch.ones(1), torch.ones(1, 1), torch.ones(1, 1)
    if wrong == "dtype":
        vals = vals.double()
    elif wrong == "length":
        rowptr = rowptr[:1]
    elif wrong == "none":
        colidx = None
    f = dg.Features(M=1, K=1, nnz=1, avg_row=1.0, max_row=1, min_row=1)
    for call in (lambda: dg.dgsp_spmm_csr(1, 1, 1, rowptr, colidx, vals, X, Y, dg.AUTO),
                 lambda: dg.dgsp_spmm_csr_nnz(1, 1, 1, 1, rowptr, colidx, vals, X, Y, dg.AUTO),
                 lambda: dg.dgsp_spmm_csr_auto(1, 1, 1, f, rowptr, colidx, vals, X, Y),
                 lambda: dg.dgsp_spmm_csr_ld(1, 1, 1, 1, rowptr, colidx, vals, X, Y),
                 lambda: dg.dgsp_spmm_csr_axpby(1, 1, 1, 1, rowptr, colidx, vals, X, Y)):
        with pytest.raises(dg.DgspError):
            call()


def _one_entry(device):
    import torch
    return (torch.tensor([0, 1], dtype=torch.int32, device=device), torch.zeros(1, dtype=torch.int32, device=device),
            torch.full((1,), 3.0, device=device), torch.full((1, 1), 2.0, device=device), torch.zeros(1, 1, device=device))


def test_numbers_are_taken_as_int_and_float_take_them():
    """On host tensors, which are turned down for what they are: a TypeError would mean the number was."""
    arrays = _one_entry("cpu")
    for nnz, algo, alpha in ((1.0, 2.0, 1), (np.float32(1.0), np.int64(2), np.float64(0.5)), ("1", "2", "0.5")):
        for call in (lambda: dg.dgsp_spmm_csr_nnz(1, 1, 1, nnz, *arrays, algo), lambda: dg.dgsp_spmm_csr(1, 1, 1, *arrays, algo),
                     lambda: dg.dgsp_spmm_csr_ld(1, 1, 1, nnz, *arrays, algo),
                     lambda: dg.dgsp_spmm_csr_axpby(1, 1, 1, nnz, *arrays, alpha, alpha, algo)):
            with pytest.raises(dg.DgspError):
                call()
    for call in (lambda: dg.dgsp_spmm_csr_nnz(1, 1, 1, None, *arrays, dg.AUTO),
                 lambda: dg.dgsp_spmm_csr_axpby(1, 1, 1, 1, *arrays, None, 0.0),
                 lambda: dg.dgsp_spmm_csr_axpby(1, 1, 1, 1, *arrays, 1.0, None)):
        with pytest.raises(TypeError):
            call()


@pytest.mark.gpu
def test_numbers_of_other_types_give_the_product():
    arrays = _one_entry("cuda")
    Y = arrays[-1]
    for call, want in ((lambda: dg.dgsp_spmm_csr_nnz(1, 1, 1, 1.0, *arrays, 2.0), 6.0),
                       (lambda: dg.dgsp_spmm_csr(1, 1, 1, *arrays, np.float64(3.0)), 6.0),
                       (lambda: dg.dgsp_spmm_csr_ld(1, 1, 1, 1.0, *arrays, 0.0), 6.0),
                       (lambda: dg.dgsp_spmm_csr_axpby(1, 1, 1, np.float32(1.0), *arrays, np.float64(2.0), 1, 1.0), 13.0)):
        Y.fill_(1.0)
        call()
        assert Y.item() == want

@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("N", [0, 1, 5, 33])
def test_gradient_of_other_types_and_layouts(dtype, N):
    """N = 0 stands for a vector.  A transposed (not contiguous) operand, used twice, with a float64 one cast and cast back."""
    import torch
    from paper_2106_16064_amd.autograd import SparseOperator, transpose_csr
    A = wl.sweep_csr(700, 9, "lognormal", seed=4)
    op = SparseOperator(A)
    cols = max(N, 1)
    X = wl.dense_matrix(A.K, cols, "normal", seed=1)
    Gy = wl.dense_matrix(A.M, cols, "uniform", seed=2)
    leaf = torch.from_numpy(X).cuda().to(getattr(torch, dtype))
    leaf = (leaf[:, 0] if N == 0 else leaf.t()).contiguous().requires_grad_(True)
    x = leaf if N == 0 else leaf.t()
    G = torch.from_numpy(Gy).cuda()
    print(f"[case] gradient {dtype} N={N}", flush=True)
    y = op(x)
    assert y.shape == ((A.M,) if N == 0 else (A.M, N)) and y.dtype == torch.float32
    (y + op(x)).backward(G[:, 0] if N == 0 else G)
    with torch.no_grad():
        assert op(x).grad_fn is None
    T = transpose_csr(A)
    ref, bnd = oracle.spmm_ref(T.M, T.K, cols, T.rowptr, T.colidx, T.vals, Gy)
    got = leaf.grad if N == 0 else leaf.grad.t()
    assert got.dtype == leaf.dtype
    ok, worst = oracle.within_bound(got.float().cpu().numpy().reshape(T.M, cols), 2 * ref, 2 * bnd, 1e-5)
    assert ok, worst


class _DenseMatrix:
    """Stands in for a ``DeviceCsr`` on the CPU, where the native product cannot run."""

    def __init__(self, D):
        self.D, self.tuned = D, {}
        self.M, self.K = D.shape
        self.features = self.rowptr = self.colidx = self.vals = None

    def spmm(self, X, algo=dg.AUTO):
        return self.D @ (X if X.dim() == 2 else X[:, None])


def _operator(device):
    """(operator, its dense matrix): a stand-in on the CPU, the real one on the GPU."""
    import torch
    from paper_2106_16064_amd.autograd import SparseOperator
    A = wl.sweep_csr(60, 5, "poisson", seed=2)
    D = torch.zeros(A.M, A.K)
    D.index_put_((torch.from_numpy(np.repeat(np.arange(A.M), A.row_lengths())), torch.from_numpy(A.colidx).long()),
                 torch.from_numpy(A.vals), accumulate=True)
    if device == "cuda":
        return SparseOperator(A), D.cuda()
    op = SparseOperator.__new__(SparseOperator)
    op.fwd, op.bwd = _DenseMatrix(D), _DenseMatrix(D.t().contiguous())
    return op, D


DEVICES = ["cpu", pytest.param("cuda", marks=pytest.mark.gpu)]


@pytest.mark.parametrize("device", DEVICES)
@pytest.mark.parametrize("requires_grad", [False, True])
def test_a_tangent_on_the_operand_is_refused(device, requires_grad):
    """Forward mode is not implemented: a product without its tangent would read as a derivative of zero."""
    import torch
    from torch.autograd import forward_ad
    op, D = _operator(device)
    X = torch.randn(D.shape[1], 3, device=device, requires_grad=requires_grad)
    with forward_ad.dual_level():
        with pytest.raises(NotImplementedError):
            op(forward_ad.make_dual(X, torch.ones_like(X)))


@pytest.mark.parametrize("device", DEVICES)
@pytest.mark.parametrize("transform", ["vmap", "grad", "jvp"])
def test_function_transforms_are_refused(device, transform):
    import torch
    op, D = _operator(device)
    X = torch.randn(D.shape[1], 3, device=device)
    call = {"vmap": lambda: torch.func.vmap(op)(torch.stack([X, X])),
            "grad": lambda: torch.func.grad(lambda x: op(x).sum())(X),
            "jvp": lambda: torch.func.jvp(op, (X,), (X,))}[transform]
    with pytest.raises(RuntimeError, match="setup_context"):
        call()


@pytest.mark.parametrize("device", DEVICES)
def test_a_traced_product_follows_its_input(device):
    """A recorded product is computed again on every input, inside other operations, with its gradient."""
    import torch
    op, D = _operator(device)
    X = torch.randn(D.shape[1], 3, device=device)
    traced = torch.jit.trace(lambda x: op(x * 2.0).relu(), X, check_trace=False)
    for scale in (1.0, -3.0):
        x = (X * scale + 1.0).requires_grad_(True)
        y = traced(x)
        want = (D @ (2.0 * x)).relu()
        assert torch.allclose(y, want, rtol=1e-5, atol=1e-5)
        dx, = torch.autograd.grad(y.sum(), x)
        want_dx, = torch.autograd.grad(want.sum(), x)
        assert torch.allclose(dx, want_dx, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("device", DEVICES)
def test_a_mode_that_intercepts_operations_sees_the_product(device):
    import torch
    from torch.utils._python_dispatch import TorchDispatchMode

    class Names(TorchDispatchMode):
        seen = []

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.seen.append(str(func))
            return func(*args, **(kwargs or {}))

    op, D = _operator(device)
    X = torch.randn(D.shape[1], 3, dtype=torch.float64, device=device, requires_grad=True)
    with Names() as mode:
        y = op(X)
    assert any("_to_copy" in name for name in mode.seen)
    y.sum().backward()
    assert torch.allclose(y, (D.double() @ X).float(), rtol=1e-5, atol=1e-5)
    assert torch.allclose(X.grad, D.double().sum(0)[:, None].expand_as(X), rtol=1e-5, atol=1e-5)


STATS = {
    "chunk_edges": [2047, 1, 2048, 2049, 0, 1, 2046, 2, 0, 0],
    "one_row": [5000],
    "one_entry": [1],
    "empty_rows_around": [0] * 3000 + [7] + [0] * 3000,
    "no_entries": [0] * 300,
    "many_blocks": [3, 1, 0, 8] * 160000,
    "one_block_each": [2048] * 7,
    "long_and_empty": [1500000] + [0] * 900000 + [1] * 700000,
}


def _columns_by_position(lens):
    """Rows of any length whose columns ascend in steps of two."""
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    colidx = (np.arange(rowptr[-1]) - np.repeat(rowptr[:-1], lens)).astype(np.int32) * 2
    return wl.CsrMatrix(len(lens), 2 * max(lens), rowptr, colidx, np.ones(rowptr[-1], dtype=np.float32), "by_position", {})


@pytest.mark.gpu
@pytest.mark.parametrize("order", ["ascending", "one_descent", "shuffled"])
@pytest.mark.parametrize("name", sorted(STATS))
def test_statistics_and_index_types(name, order):
    """Statistics of device arrays and the 32-bit copies of int64 ones, at the edges of the pieces the entries are counted in."""
    import torch
    lens = STATS[name]
    if max(lens) > 6000:
        A = _columns_by_position(lens)
    else:
        A = wl.csr_from_lens(lens, K=6000, seed=3, name=name)
    colidx = A.colidx.copy()
    rng = np.random.default_rng(1)
    longest = int(np.argmax(A.row_lengths()))
    s, e = A.rowptr[longest], A.rowptr[longest + 1]
    if order == "one_descent" and e - s > 1:
        colidx[[e - 2, e - 1]] = colidx[[e - 1, e - 2]]
    elif order == "shuffled":
        colidx[s:e] = rng.permutation(colidx[s:e])
    want = dg.dgsp_features_from_csr_host(A.M, A.K, A.rowptr, colidx)
    vals = torch.from_numpy(A.vals).cuda()
    for dtype in (np.int32, np.int64):
        print(f"[case] statistics {name} {order} {dtype.__name__}", flush=True)
        D = dg.DeviceCsr.from_device(A.M, A.K, torch.from_numpy(A.rowptr.astype(dtype)).cuda(),
                                     torch.from_numpy(colidx.astype(dtype)).cuda(), vals)
        assert D.features.as_dict() == want.as_dict()
        assert D.rowptr.dtype == torch.int32 and np.array_equal(D.rowptr.cpu().numpy(), A.rowptr)
        assert D.colidx.dtype == torch.int32 and np.array_equal(D.colidx.cpu().numpy(), colidx)


@pytest.mark.gpu
def test_statistics_from_several_threads():
    """More calls under way than there are places for, each on a stream of its own."""
    import threading
    import torch
    mats = [wl.sweep_csr(3000 + 700 * i, 12, "lognormal", seed=i) for i in range(12)]
    arrays = [(torch.from_numpy(A.rowptr.astype(np.int64)).cuda(), torch.from_numpy(A.colidx.astype(np.int64)).cuda(),
               torch.from_numpy(A.vals).cuda()) for A in mats]
    torch.cuda.synchronize()
    got, errors = [None] * len(mats), []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(20):
                    got[i] = dg.DeviceCsr.from_device(mats[i].M, mats[i].K, *arrays[i]).features.as_dict()
        except Exception as e:          # surfaced in the main thread below
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(mats))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for A, f in zip(mats, got):
        assert f == dg.dgsp_features_from_csr_host(A.M, A.K, A.rowptr, A.colidx).as_dict()


@pytest.mark.gpu
@pytest.mark.parametrize("rows, mean", [(5, 3), (3001, 9), (200_003, 11), (700_001, 16)])
def test_a_matrix_from_int64_arrays_is_ready_for_every_stream(rows, mean):
    """The call returns on a word that its kernel writes before it ends; the 32-bit arrays are complete by then, so that
    nothing orders a reader on another stream behind that kernel."""
    import torch
    rng = np.random.default_rng(rows)
    lens = rng.integers(0, 2 * mean, size=rows)
    rowptr = np.concatenate([[0], np.cumsum(lens)])
    colidx = (np.arange(rowptr[-1]) - np.repeat(rowptr[:-1], lens)) * 3 + np.repeat(np.arange(rows) % 7, lens)
    rp, ci = torch.from_numpy(rowptr).cuda(), torch.from_numpy(colidx).cuda()
    vals = torch.ones(colidx.size, device="cuda")
    first, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    print(f"[case] int64 arrays on two streams rows={rows}", flush=True)
    kept = []
    for _ in range(10):
        with torch.cuda.stream(first):
            D = dg.DeviceCsr.from_device(rows, 6 * mean + 7, rp, ci, vals)
        with torch.cuda.stream(other):
            kept.append((D, D.rowptr.clone(), D.colidx.clone()))
    torch.cuda.synchronize()
    for _, rp32, ci32 in kept:
        assert torch.equal(rp32.long(), rp) and torch.equal(ci32.long(), ci)


@pytest.mark.gpu
def test_statistics_are_refused_while_a_graph_is_recorded():
    """Nothing of the call gets into the graph, which goes on, and the next call outside it is like any other."""
    import torch
    A = wl.sweep_csr(3000, 12, "lognormal", seed=1)
    arrays = [torch.from_numpy(a).cuda() for a in (A.rowptr.astype(np.int64), A.colidx.astype(np.int64), A.vals)]
    x = torch.zeros(5, device="cuda")
    torch.cuda.synchronize()
    print("[case] statistics while a graph is recorded", flush=True)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        x.add_(1.0)
        with pytest.raises(dg.DgspError):
            dg.DeviceCsr.from_device(A.M, A.K, *arrays)
        x.mul_(2.0)
    want = dg.dgsp_features_from_csr_host(A.M, A.K, A.rowptr, A.colidx).as_dict()
    value = 0.0
    for _ in range(3):
        graph.replay()
        value = 2.0 * (value + 1.0)
        assert dg.DeviceCsr.from_device(A.M, A.K, *arrays).features.as_dict() == want
        assert torch.equal(x, torch.full_like(x, value))


@pytest.mark.gpu
@pytest.mark.parametrize("K", [1, 1000, 1 << 18, 1 << 20, (1 << 31) - 4097])
@pytest.mark.parametrize("entries", [4096, 4097, 70_001, 1_000_003])
def test_counts_of_sampled_columns(K, entries):
    import ctypes
    import torch
    from test_host_api import reuse_counts
    rng = np.random.default_rng(K + entries)
    col = (K * rng.random(entries) ** 3).astype(np.int32)
    col[-1] = K - 1
    dev = torch.from_numpy(col).cuda()
    counts = (ctypes.c_uint64 * 6)()
    f = dg.lib().dgsp_internal_column_reuse
    f.restype, f.argtypes = ctypes.c_int, [ctypes.c_int64, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p]
    print(f"[case] sampled columns K={K} entries={entries}", flush=True)
    assert f(entries, dev.data_ptr(), counts, torch.cuda.current_stream().cuda_stream) == dg.OK
    assert list(counts) == reuse_counts(col)
    assert f(4095, dev.data_ptr(), counts, None) == dg.ERR_INVALID_ARG


def _from_device(A, dtype, vals):
    import torch
    return dg.DeviceCsr.from_device(A.M, A.K, torch.from_numpy(A.rowptr.astype(dtype)).cuda(),
                                    torch.from_numpy(A.colidx.astype(dtype)).cuda(), vals)


@pytest.mark.gpu
def test_narrow_column_blocks_where_they_save_enough():
    """A graph of more than four million entries, taken from the host, from int32 and from int64 arrays: its columns are
    measured when it is taken, and the products on narrow blocks plain and scaled."""
    import torch
    from test_host_api import column_block
    A = wl.rmat_csr(19, 12, seed=3)
    dA = dg.DeviceCsr(A)
    for N in (64, 128):
        X = wl.dense_matrix(A.K, N, "normal", seed=N)
        Y0 = wl.dense_matrix(A.M, N, "uniform", seed=1)
        ref, bnd = oracle.spmm_ref(A.M, A.K, N, A.rowptr, A.colidx, A.vals, X)
        dX, Y = torch.from_numpy(X).cuda(), torch.from_numpy(Y0).cuda()
        print(f"[case] narrow column blocks N={N}", flush=True)
        ok, worst = oracle.within_bound(dA.spmm(dX).cpu().numpy(), ref, bnd, 1e-5)
        assert ok, worst
        dg.dgsp_spmm_csr_axpby(A.M, A.K, N, A.nnz, dA.rowptr, dA.colidx, dA.vals, dX, Y, -0.5, 1.5, features=dA.features)
        ok, worst = oracle.within_bound(Y.cpu().numpy(), -0.5 * ref + 1.5 * Y0, 0.5 * bnd + 1.5 * np.abs(Y0), 1e-5)
        assert ok, worst
    share = dA.features.saved_share
    assert A.nnz > 4_000_000 and 0.1 < share < 0.2 and column_block(dA.features, 128) == 32
    for dtype in (np.int32, np.int64):
        assert _from_device(A, dtype, dA.vals).features.saved_share == share


@pytest.mark.gpu
def test_columns_that_are_not_measured_or_save_too_little():
    """Rows as uneven with uniform columns keep the blocks of 64 and small matrices are not sampled.  A product neither
    measures nor waits: one that is the matrix's first is recorded, and its graph gives the eager result."""
    import torch
    from test_host_api import column_block
    A = wl.rmat_csr(19, 12, seed=3)
    U = dg.DeviceCsr(wl.CsrMatrix(A.M, A.K, A.rowptr, np.random.default_rng(0).integers(0, A.K, A.nnz).astype(np.int32), A.vals, "uniform", {}))
    assert 0.0 <= U.features.saved_share < 0.1 and column_block(U.features, 128) == 64
    assert dg.DeviceCsr(wl.rmat_csr(14, 24, seed=3)).features.saved_share == 0.0
    D = dg.DeviceCsr(A)
    X = torch.randn(A.K, 64, device="cuda")
    Y = torch.empty(A.M, 64, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    print("[case] narrow column blocks while a graph is recorded", flush=True)
    with torch.cuda.graph(graph, stream=side):
        D.spmm(X, Y=Y)
    assert D.features.saved_share > 0.1
    want = D.spmm(X)
    scale = want.abs().max()
    for _ in range(3):
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert (Y - want).abs().max() <= 1e-4 * scale


@pytest.mark.gpu
def test_gradient_on_narrow_column_blocks():
    import torch
    from paper_2106_16064_amd.autograd import SparseOperator, transpose_csr
    A = wl.rmat_csr(19, 12, seed=3)
    op = SparseOperator(A)
    X = torch.zeros(A.K, 64, device="cuda", requires_grad=True)
    G = wl.dense_matrix(A.M, 64, "uniform", seed=2)
    op(X).backward(torch.from_numpy(G).cuda())
    assert op.fwd.features.saved_share > 0.1 and op.bwd.features.saved_share > 0.1
    T = transpose_csr(A)
    ref, bnd = oracle.spmm_ref(T.M, T.K, 64, T.rowptr, T.colidx, T.vals, G)
    ok, worst = oracle.within_bound(X.grad.cpu().numpy(), ref, bnd, 1e-5)
    assert ok, worst
