"""Rows without entries in nb_sr's run kernel: stretches of them around the 64 rows of a window, the eight windows that a block remembers
and the further ones whose bounds are asked for before the rows so far are written."""
import numpy as np
import pytest

import oracle
from paper_2106_16064_amd import binding as dg
from paper_2106_16064_amd import workloads as wl

STRETCHES = [1, 63, 64, 65, 447, 448, 449, 511, 512, 513, 959, 960, 961, 2000]


def matrix(between, seed):
    """`between(rng)`: lengths of the rows between one stretch and the next."""
    rng = np.random.default_rng(seed)
    lens = np.concatenate([part for s in STRETCHES for part in (np.zeros(s, int), between(rng))] + [np.zeros(300, int)])
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return wl.CsrMatrix(len(lens), 2003, rowptr, rng.integers(0, 2003, rowptr[-1]).astype(np.int32),
                        rng.uniform(-1, 1, rowptr[-1]).astype(np.float32), "stretches", {})


def long_rows():
    """Rows over several chunks; more entries than rows by far, so chunks stay in order."""
    return matrix(lambda rng: rng.integers(1, 2000, 12), 1)


def short_rows():
    """Rows that a wave keeps whole, few entries a row: chunks dealt out to the XCDs."""
    return matrix(lambda rng: rng.integers(0, 12, 700), 2)


def single_entries():
    return matrix(lambda rng: np.ones(3, int), 3)


@pytest.mark.gpu
@pytest.mark.parametrize("make, dealt", [(long_rows, False), (short_rows, True), (single_entries, True)])
@pytest.mark.parametrize("N", [4, 7, 8, 15, 16, 33, 64, 93, 128, 257])
def test_rows_without_entries(make, dealt, N):
    """`dealt`: with fewer than six entries a row (eight from 32 lanes a row of X on) chunks are dealt out to the XCDs and such rows are
    written in front of the walk, others behind it."""
    import torch
    A = make()
    assert A.nnz // A.M < 6 if dealt else A.nnz // A.M >= 8
    D = dg.DeviceCsr(A)
    X = wl.dense_matrix(A.K, N, "normal", seed=N)
    ref, bnd = oracle.spmm_ref(A.M, A.K, N, A.rowptr, A.colidx, A.vals, X)
    dX = torch.from_numpy(X).cuda()
    wide = torch.full((A.M, N + 5), float("nan"), device="cuda")
    packed = torch.full((A.M, N), float("nan"), device="cuda")
    print(f"[case] {make.__name__} N={N}", flush=True)
    dg.dgsp_spmm_csr_ld(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, dX, wide[:, 3:3 + N], dg.NB_SR, D.features)
    dg.dgsp_spmm_csr_nnz(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, dX, packed, dg.NB_SR)
    for got in (wide[:, 3:3 + N].cpu().numpy(), packed.cpu().numpy()):
        ok, worst = oracle.within_bound(got, ref, bnd, 1e-5)          # exact zeros where nothing is added
        assert ok, worst
    assert bool(torch.isnan(wide[:, :3]).all()) and bool(torch.isnan(wide[:, 3 + N:]).all())
