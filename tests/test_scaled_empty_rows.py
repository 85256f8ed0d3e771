"""Rows without entries in the scaled form of nb_sr: the launch before the product scales them, together with the rows that several
chunks share (nb_prepare_kernel), as many lanes to a row as it has columns."""
import numpy as np
import pytest

import oracle
from paper_2106_16064_amd import binding as dg
from paper_2106_16064_amd import workloads as wl


def holes():
    """Workgroups of the launch with no, one, some and only empty rows, the last one short; one row over many chunks."""
    rng = np.random.default_rng(6)
    lens = np.concatenate([np.zeros(256, int), [70_000], np.zeros(600, int), rng.integers(0, 3, 3000), rng.integers(1, 30, 1024), [0],
                           rng.integers(1, 30, 300), np.zeros(37, int)])
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return wl.CsrMatrix(len(lens), 4001, rowptr, rng.integers(0, 4001, rowptr[-1]).astype(np.int32),
                        rng.uniform(-1, 1, rowptr[-1]).astype(np.float32), "holes", {})


@pytest.mark.gpu
@pytest.mark.parametrize("beta", [0.0, 0.5])
@pytest.mark.parametrize("N", [4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 130])
def test_rows_without_entries_are_scaled_once(N, beta):
    import torch
    A = holes()
    D = dg.DeviceCsr(A)
    X = wl.dense_matrix(A.K, N, "normal", seed=N)
    wide = np.random.default_rng(N).uniform(-1, 1, (A.M, N + 3)).astype(np.float32)
    ref, bnd = oracle.spmm_ref(A.M, A.K, N, A.rowptr, A.colidx, A.vals, X)
    Y = torch.from_numpy(wide).cuda()
    if beta == 0.0:
        Y[:, 2:2 + N] = float("nan")                     # not read
    print(f"[case] holes N={N} beta={beta}", flush=True)
    dg.dgsp_spmm_csr_axpby(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, torch.from_numpy(X).cuda(), Y[:, 2:2 + N], -2.0, beta,
                           dg.NB_SR, D.features)
    got, Y0 = Y.cpu().numpy(), wide[:, 2:2 + N].astype(np.float64)
    ok, worst = oracle.within_bound(got[:, 2:2 + N], -2.0 * ref + beta * Y0, 2.0 * bnd + beta * np.abs(Y0), 1e-5)
    assert ok, worst
    empty = np.diff(A.rowptr) == 0
    assert (got[empty, 2:2 + N] == np.float32(beta) * wide[empty, 2:2 + N]).all()
    assert (got[:, :2] == wide[:, :2]).all() and (got[:, 2 + N:] == wide[:, 2 + N:]).all()
