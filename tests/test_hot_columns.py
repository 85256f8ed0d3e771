"""Products with one to four columns that read the hottest runs of X from LDS (nb_pr_kernel, HOT), against the oracle."""
import copy
import pickle

import numpy as np
import pytest

import oracle
from paper_2106_16064_amd import binding as dg
from paper_2106_16064_amd import workloads as wl

WORDS, PIECES, TABLE = 1024, 512, 3 * 1024
FLOATS = {1: 31 * 1024, 2: 28 * 1024, 3: 24 * 1024, 4: 20 * 1024}


def uneven_matrix(M, K, power, seed, nnz=4_200_000):
    """Row lengths far apart (CV above 4, empty rows among them); columns K * u^power, duplicates kept."""
    rng = np.random.default_rng(seed)
    weight = rng.pareto(0.9, M) * (rng.random(M) < 0.8)
    lens = np.minimum((weight * (1.3 * nnz / weight.sum())).astype(np.int64), 60_000)
    lens[rng.integers(0, M, 64)] += max(nnz - int(lens.sum()), 0) // 64 + 1
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cols = np.minimum((K * rng.random(rowptr[-1]) ** power).astype(np.int64), K - 1)
    return wl.CsrMatrix(M, K, rowptr, cols.astype(np.int32), rng.uniform(-1, 1, rowptr[-1]).astype(np.float32), "uneven", {})


def hot_shift(K):
    shift = 5
    while (K - 1) >> shift >= 32 * WORDS:
        shift += 1
    return shift


def expected_table(colidx, K, V):
    """Bitmap words, the words' running counts and the runs, as the selection's sample gives them; the share of the sample."""
    shift = hot_shift(K)
    room = FLOATS[V] // (V << shift)
    at = (len(colidx) - 64) // (PIECES - 1) * np.arange(PIECES)[:, None] + np.arange(64)
    counts = np.bincount(colidx[at.ravel()] >> shift, minlength=32 * WORDS)
    level = 1
    while (counts >= level).sum() > room:
        level += 1
    hot = counts >= level
    if level > 1:
        below = np.flatnonzero(counts == level - 1)
        hot[below[:room - hot.sum()]] = True
    runs = np.flatnonzero(hot)
    words = (hot.reshape(WORDS, 32) * (1 << np.arange(32, dtype=np.int64))).sum(1)
    before = np.concatenate([[0], np.cumsum(hot.reshape(WORDS, 32).sum(1))[:-1]])
    table = np.full(TABLE, -1, dtype=np.int64)
    table[0:2 * WORDS:2], table[1:2 * WORDS:2] = words, before
    table[2 * WORDS:2 * WORDS + len(runs)] = runs
    return table.astype(np.uint32).view(np.int32), counts[hot].sum() / (64 * PIECES)


CASES = [("graph", 0, 0, 0), ("odd", 300_007, 700_001, 4.0), ("wide runs", 200_000, 3_000_001, 6.0),
         ("every column hot", 150_001, 20_011, 1.0), ("few columns", 120_000, 37, 1.0), ("short last run", 262_144, 1_048_573, 4.0)]


def matrix(name, M, K, power):
    return wl.rmat_csr(19, 12, seed=3) if name == "graph" else uneven_matrix(M, K, power, seed=M)


@pytest.mark.gpu
@pytest.mark.parametrize("name, M, K, power", CASES, ids=[c[0] for c in CASES])
def test_products_with_hot_runs(name, M, K, power):
    import torch
    A = matrix(name, M, K, power)
    D = dg.DeviceCsr(A)
    f = D.features
    assert f.cv_row >= 4 and f.nnz >= 4_000_000
    tables = f.hot_columns.cpu().numpy().reshape(4, TABLE)
    for N in (1, 2, 3, 4):
        table, share = expected_table(A.colidx, A.K, N)
        assert f.hot_share[N - 1] == pytest.approx(share)
        assert np.array_equal(tables[N - 1], table)
        assert N > 1 or f.nnz * share >= 1.5e6
        X = wl.dense_matrix(A.K, N, "normal", seed=2)
        Y0 = wl.dense_matrix(A.M, N, "uniform", seed=1)
        ref, bnd = oracle.spmm_ref(A.M, A.K, N, A.rowptr, A.colidx, A.vals, X)
        dX = torch.from_numpy(X).cuda()
        print(f"[case] hot runs {name} N={N}", flush=True)
        # X at every alignment of a float
        for offset in (0, 1, 3):
            buffer = torch.empty(A.K * N + 4, device="cuda")
            x = buffer[offset:offset + A.K * N].view(A.K, N)
            x.copy_(dX)
            ok, worst = oracle.within_bound(D.spmm(x).cpu().numpy(), ref, bnd, 1e-5)
            assert ok, worst
        for alpha, beta in ((-0.5, 1.5), (2.0, 0.0)):
            Y = torch.from_numpy(Y0).cuda() if beta else torch.full((A.M, N), float("nan"), device="cuda")
            dg.dgsp_spmm_csr_axpby(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, dX, Y, alpha, beta, features=f)
            ok, worst = oracle.within_bound(Y.cpu().numpy(), alpha * ref + beta * Y0, abs(alpha) * bnd + abs(beta) * np.abs(Y0), 1e-5)
            assert ok, worst


@pytest.mark.gpu
def test_infinities_and_nan_in_hot_and_other_runs():
    import torch
    A = matrix(*CASES[0])
    D = dg.DeviceCsr(A)
    hot = D.features.hot_columns.cpu().numpy()[2 * WORDS:TABLE]
    inside, outside = 32 * int(hot[5]) + 7, next(c for c in np.unique(A.colidx)[::-1] if c // 32 not in hot)
    X = np.ones((A.K, 1), dtype=np.float32)
    X[inside], X[outside] = np.inf, np.nan
    rows = np.repeat(np.arange(A.M), np.diff(A.rowptr))
    want_nan = np.zeros(A.M, dtype=bool)
    want_nan[rows[A.colidx == outside]] = True
    has_inf = np.zeros(A.M, dtype=bool)
    has_inf[rows[(A.colidx == inside) & (A.vals != 0)]] = True
    print("[case] hot runs with infinities", flush=True)
    y = D.spmm(torch.from_numpy(X).cuda()).cpu().numpy()[:, 0]
    assert np.array_equal(np.isnan(y), want_nan)
    assert np.array_equal(np.isinf(y), has_inf & ~want_nan)


@pytest.mark.gpu
def test_the_table_stays_with_its_matrix():
    """Other K, other widths, strided vectors and structures without the table take the general way; copies keep it alive."""
    import torch
    A = matrix(*CASES[0])
    D = dg.DeviceCsr(A)
    f = D.features
    X = torch.randn(A.K, 1, device="cuda")
    want = D.spmm(X, algo=dg.NB_SR)
    scale = want.abs().max()
    print("[case] hot runs: features passed on", flush=True)

    def check(x, features, K=A.K):
        Y = torch.full((A.M, 1), float("nan"), device="cuda")
        dg.dgsp_spmm_csr_ld(A.M, K, 1, A.nnz, D.rowptr, D.colidx, D.vals, x, Y, features=features)
        assert (Y - want).abs().max() <= 1e-5 * scale

    bare = dg.MatrixFeatures.from_buffer_copy(bytes(f))
    assert list(bare.hot_share) == list(f.hot_share) and bare.hot_columns is None
    restored = pickle.loads(pickle.dumps(f))
    assert restored.hot_columns is None or torch.equal(restored.hot_columns, f.hot_columns)
    wrong = copy.copy(bare)
    wrong.hot_columns = f.hot_columns[:-1].contiguous()
    for features in (f, bare, wrong, restored, copy.copy(f), dg.Features(**f.as_dict())):
        check(X, features)
    check(torch.cat([X, X + 1], 1)[:, :1], f)                       # rows two floats apart
    check(torch.cat([X, X[:5000]]), f, A.K + 5000)                  # not the K the runs were counted for
    assert dg.DeviceCsr(wl.rmat_csr(14, 24, seed=3)).features.hot_columns is None


@pytest.mark.gpu
def test_hot_runs_in_a_graph_and_on_a_stream():
    import torch
    A = matrix(*CASES[0])
    D = dg.DeviceCsr.from_device(A.M, A.K, torch.from_numpy(A.rowptr.astype(np.int64)).cuda(),
                                 torch.from_numpy(A.colidx.astype(np.int64)).cuda(), torch.from_numpy(A.vals).cuda())
    assert D.features.hot_columns is not None
    X = torch.randn(A.K, 1, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    Y = torch.empty(A.M, 1, device="cuda")
    print("[case] hot runs while a graph is recorded", flush=True)
    with torch.cuda.graph(graph, stream=side):
        D.spmm(X, Y=Y)
    want = D.spmm(X, algo=dg.NB_SR)
    scale = want.abs().max()
    for k in range(3):
        X.mul_(2.0)
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert (Y - want * 2.0 ** (k + 1)).abs().max() <= 1e-5 * scale * 2.0 ** (k + 1)
