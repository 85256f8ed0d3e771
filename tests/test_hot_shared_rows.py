"""Products with hot runs whose waves see to the rows that they share themselves (nb_pr_kernel, HOT and SHARES), against the oracle."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2106_16064_amd import binding as dg
from paper_2106_16064_amd import workloads as wl
from test_chunk_queues import requested
from test_hot_columns import hot_shift, launches


def matrix(hubs, columns):
    """7.2 million entries, three quarters of them on 200 runs of 32 columns or more; row lengths far apart.  `hubs`: rows of 300 000 entries, next to
    each other, a wave's share between two of their ends and in the end of the matrix."""
    rng = np.random.default_rng(columns)
    M, per_hub = 250_003, 300_000
    lens = (rng.pareto(0.9, M) * (rng.random(M) < 0.7)).clip(0, 3000).astype(np.int64)
    lens[::41] += (7_200_000 - hubs * per_hub - int(lens.sum())) // len(lens[::41])
    at = [0, 1, 2, 100_000, 100_001, M - 1][:hubs - 1] + [M - 1] if hubs else []
    lens[at] = per_hub
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    n = int(rowptr[-1])
    shift = hot_shift(columns)
    runs = rng.choice((columns - 1) >> shift, 200, replace=False)
    inside = (rng.choice(runs, n) << shift) + rng.integers(0, 1 << shift, n)
    cols = np.where(rng.random(n) < 0.75, inside, rng.integers(0, columns, n)).astype(np.int32)
    return wl.CsrMatrix(M, columns, rowptr, cols, rng.uniform(-1, 1, n).astype(np.float32), "hubs", {})


@pytest.mark.gpu
@pytest.mark.parametrize("hubs, columns", [(1, 300_007), (6, 1 << 20), (3, 1_300_003)])
def test_shared_rows_with_hot_runs(hubs, columns):
    import torch
    A = matrix(hubs, columns)
    D = dg.DeviceCsr(A)
    f = D.features
    words = 8 * 8 * torch.cuda.get_device_properties(0).multi_processor_count       # a word for each of the eight waves a CU
    for N in (1, 2, 3, 4):
        assert dg.lib().dgsp_internal_wants_hot_columns(ctypes.byref(f), ctypes.c_int64(N)) and f.hot_columns is not None
        X = wl.dense_matrix(A.K, N, "normal", seed=N)
        Y0 = wl.dense_matrix(A.M, N, "uniform", seed=1)
        ref, bnd = oracle.spmm_ref(A.M, A.K, N, A.rowptr, A.colidx, A.vals, X)
        for offset, alpha, beta in ((0, 1.0, 0.0), (1, 1.0, 0.0), (3, -0.5, 1.5), (0, 2.0, 0.0)):
            buffer = torch.empty(A.K * N + 4, device="cuda")
            dX = buffer[offset:offset + A.K * N].view(A.K, N)
            dX.copy_(torch.from_numpy(X))

            def call(Y):
                if alpha == 1.0:
                    D.spmm(dX, Y=Y)
                else:
                    dg.dgsp_spmm_csr_axpby(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, dX, Y, alpha, beta, features=f)

            print(f"[case] hubs={hubs} N={N} offset={offset} alpha={alpha} beta={beta}", flush=True)
            for _ in range(3):                            # words that earlier calls have left behind
                Y = torch.from_numpy(Y0).cuda() if beta else torch.full((A.M, N), float("nan"), device="cuda")
                assert requested(lambda: call(Y)) == words
                ok, worst = oracle.within_bound(Y.cpu().numpy(), alpha * ref + beta * Y0, abs(alpha) * bnd + abs(beta) * np.abs(Y0), 1e-5)
                assert ok, worst
            kernels = launches(lambda: call(Y))
            assert any("nb_pr_kernel" in k for k in kernels) and not any("nb_prepare_kernel" in k for k in kernels)
