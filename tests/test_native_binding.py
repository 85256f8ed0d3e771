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
