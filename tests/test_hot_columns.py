"""Products with one to four columns that read the hottest runs of X from LDS (nb_pr_kernel, HOT), against the oracle."""
import copy
import ctypes
import pickle

import numpy as np
import pytest

import oracle
from paper_2106_16064_amd import binding as dg
from paper_2106_16064_amd import workloads as wl
from test_chunk_queues import requested

WORDS, PIECES, TABLE = 1024, 512, 3 * 1024
FLOATS = {1: 31 * 1024, 2: 28 * 1024, 3: 24 * 1024, 4: 20 * 1024}


def column_law(K, law, count, rng):
    """K * u^law, or the pair (H, share): that share of the entries uniform over H scattered runs, the others over all columns."""
    if not isinstance(law, tuple):
        return np.minimum((K * rng.random(count) ** law).astype(np.int64), K - 1)
    shift = hot_shift(K)
    runs = rng.choice((K - 1) >> shift, law[0], replace=False)
    inside = (rng.choice(runs, count) << shift) + rng.integers(0, 1 << shift, count)
    return np.where(rng.random(count) < law[1], inside, rng.integers(0, K, count))


def uneven_matrix(M, K, law, seed, nnz=4_200_000, longest=60_000):
    """Row lengths far apart (CV above 4, empty rows among them); duplicate columns kept.  longest = 3100: one row in twenty has
    140 entries, a hundred have as many as that, more than a wave's share, and short enough that the waves take whole rows."""
    rng = np.random.default_rng(seed)
    if longest == 3100:
        lens = np.where(rng.random(M) < 0.05, 140, 0)
        lens[rng.choice(M, 100, replace=False)] = longest
    else:
        weight = rng.pareto(0.9, M) * (rng.random(M) < 0.8)
        lens = np.minimum((weight * (1.3 * nnz / weight.sum())).astype(np.int64), longest)
        lens[rng.integers(0, M, 64)] += max(nnz - int(lens.sum()), 0) // 64 + 1
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cols = column_law(K, law, rowptr[-1], rng)
    return wl.CsrMatrix(M, K, rowptr, cols.astype(np.int32), rng.uniform(-1, 1, rowptr[-1]).astype(np.float32), "uneven", {})


def hot_shift(K):
    shift = 5
    while (K - 1) >> shift >= 32 * WORDS:
        shift += 1
    return shift


def run_counts(colidx, K):
    """How often the selection's sample meets each run."""
    at = (len(colidx) - 64) // (PIECES - 1) * np.arange(PIECES)[:, None] + np.arange(64)
    return np.bincount(colidx[at.ravel()] >> hot_shift(K), minlength=32 * WORDS)


def fullest(counts, places):
    """The runs that `places` places go to (the first of those that tie), and how many sampled entries would find their run among
    them by the other entries' counts alone."""
    level = 1
    while (counts >= level).sum() > places:
        level += 1
    taken = counts >= level
    if level == 1:
        return taken, counts[counts > 1].sum()
    left, tied = places - taken.sum(), np.flatnonzero(counts == level - 1)
    sure, shared = counts[counts > level].sum(), counts[counts == level].sum()
    taken[tied[:left]] = True
    return taken, sure + shared * (left + 1) / (len(tied) + 1)


def places(K, V):
    """Runs that the table has room for, runs that an L1 holds anyway."""
    per_run = V << hot_shift(K)
    return FLOATS[V] // per_run, 4096 // per_run


def expected_table(colidx, K, V):
    """Bitmap words, the words' running counts and the runs, as the selection's sample gives them; the share that they save."""
    counts = run_counts(colidx, K)
    room, cached = places(K, V)
    hot, met = fullest(counts, room)
    share = max(met - fullest(counts, cached)[1], 0) / (64 * PIECES)
    runs = np.flatnonzero(hot)
    words = (hot.reshape(WORDS, 32) * (1 << np.arange(32, dtype=np.int64))).sum(1)
    before = np.concatenate([[0], np.cumsum(hot.reshape(WORDS, 32).sum(1))[:-1]])
    table = np.full(TABLE, -1, dtype=np.int64)
    table[0:2 * WORDS:2], table[1:2 * WORDS:2] = words, before
    table[2 * WORDS:2 * WORDS + len(runs)] = runs
    return table.astype(np.uint32).view(np.int32), share


CASES = [("graph", 0, 0, 0), ("odd", 300_007, 700_001, (400, 0.6)), ("runs of 64", 200_000, 1_500_007, (200, 0.6)),
         ("runs of 128", 200_000, 3_000_001, (100, 0.6)), ("every column hot", 150_001, 4_999, 1.0),
         ("short last run", 262_144, 262_141, 4.0), ("whole rows", 600_000, 3_000_001, (100, 0.6))]


def matrix(name, M, K, law):
    if name == "graph":
        return wl.rmat_csr(19, 12, seed=3)
    return uneven_matrix(M, K, law, seed=M, longest=3100 if name == "whole rows" else 60_000)


def launches(call):
    """Names of the kernels that a call launches."""
    import torch
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return [e.key for e in prof.key_averages()]


def test_statistics_are_saved_without_the_table():
    """They are read where the GPU that holds the table is not; copies in the same program share it."""
    import torch
    f = dg.MatrixFeatures(M=3, K=5, saved_share=0.25)
    f.hot_share[1] = 0.5
    f.hot_columns, f.hot_stream, f.note = torch.arange(4), 16, "kept"
    saved = pickle.dumps(f)
    assert b"tensor" not in saved and b"storage" not in saved
    restored = pickle.loads(saved)
    assert bytes(restored) == bytes(f) and restored.note == "kept"
    assert restored.hot_columns is None and restored.hot_stream == 0
    for copied in (copy.copy(f), copy.deepcopy(f)):
        assert bytes(copied) == bytes(f) and copied.hot_columns is f.hot_columns and copied.hot_stream == 16 and copied.note == "kept"
        copied.M = 4
        assert f.M == 3


@pytest.mark.gpu
@pytest.mark.parametrize("K, law", [(262_144, 1.0), (500_000, 1.0), (1 << 20, 3.0), (3_000_001, (60, 0.3)), (3_000_001, (20, 1.0))])
def test_the_share_is_the_matrix_s_and_not_the_sample_s(K, law):
    """The runs are those that the sample met most often, by luck among other things: what they save is counted over all entries here.
    The sample's share is off by the square root of p (1 - p) / n; five times that."""
    A = uneven_matrix(M := 200_000, K, law, seed=M)
    print(f"[case] share of hot runs K={K}", flush=True)
    f = dg.DeviceCsr(A).features
    counts, runs = run_counts(A.colidx, K), A.colidx >> hot_shift(K)
    for V in (1, 2, 3, 4):
        hot, cached = (fullest(counts, n)[0] for n in places(K, V))
        assert abs(f.hot_share[V - 1] - (np.mean(hot[runs]) - np.mean(cached[runs]))) <= 5 * 0.5 / (64 * PIECES) ** 0.5
    # an L1 that holds all columns is saved nothing
    assert dg.DeviceCsr(uneven_matrix(120_000, 37, 1.0, seed=1)).features.hot_columns is None


@pytest.mark.gpu
@pytest.mark.parametrize("name, M, K, law", CASES, ids=[c[0] for c in CASES])
def test_products_with_hot_runs(name, M, K, law):
    import torch
    A = matrix(name, M, K, law)
    D = dg.DeviceCsr(A)
    f = D.features
    assert f.cv_row >= 4 and f.nnz >= 4_000_000
    tables = f.hot_columns.cpu().numpy().reshape(4, TABLE)
    for N in (1, 2, 3, 4):
        table, share = expected_table(A.colidx, A.K, N)
        assert f.hot_share[N - 1] == pytest.approx(share, abs=1.0 / (64 * PIECES))       # whole entries
        assert np.array_equal(tables[N - 1], table)
        assert dg.lib().dgsp_internal_wants_hot_columns(ctypes.byref(f), ctypes.c_int64(N))
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
        # One launch: waves see to the rows that they share, with a word a wave.  Waves that take whole rows share none; some of them
        # have no row at all here.
        shares = name != "whole rows"
        Y = torch.full((A.M, N), float("nan"), device="cuda")
        kernels = launches(lambda: D.spmm(dX, Y=Y))
        assert any("nb_pr_kernel" in k for k in kernels) and not any("nb_prepare_kernel" in k for k in kernels)
        assert requested(lambda: D.spmm(dX, Y=Y)) == (8 * 8 * torch.cuda.get_device_properties(0).multi_processor_count if shares else 0)
        # a call in two phases has no memory for them: there the launch in front clears the rows
        Y = torch.full((A.M, N), float("nan"), device="cuda")
        phase = lambda which: dg.dgsp_spmm_csr_phase(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, dX, Y, dg.NB_PR, which, f)  # noqa: E731
        assert any("nb_prepare_kernel" in k for k in launches(lambda: phase(dg.PHASE_PREPARE))) == shares
        assert any("nb_pr_kernel" in k for k in launches(lambda: phase(dg.PHASE_MAIN)))
        ok, worst = oracle.within_bound(Y.cpu().numpy(), ref, bnd, 1e-5)
        assert ok, worst
        # the product looks at the table
        lies = dg.MatrixFeatures.from_buffer_copy(bytes(f))
        lies.hot_columns = zeros_table()
        Y = torch.full((A.M, N), float("nan"), device="cuda")
        dg.dgsp_spmm_csr_auto(A.M, A.K, N, lies, D.rowptr, D.colidx, D.vals, dX, Y)
        assert not Y.any()
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
    assert bytes(restored) == bytes(f) and restored.hot_columns is None
    again = pickle.loads(pickle.dumps(D))                           # a whole matrix comes back with a table
    assert torch.equal(again.features.hot_columns, f.hot_columns) and bytes(again.features) == bytes(f)
    for copied in (copy.copy(D), copy.deepcopy(D)):                 # and copies in the same program share it
        assert copied.features.hot_columns is f.hot_columns
    small = dg.DeviceCsr(wl.rmat_csr(14, 24, seed=3))
    small.features.hot_share[0] = 0.01                              # measured, and not worth a table: nothing is measured again
    assert copy.copy(small).features.hot_share[0] == pickle.loads(pickle.dumps(small)).features.hot_share[0] == 0.01
    wrong = copy.copy(bare)
    wrong.hot_columns = f.hot_columns[:-1].contiguous()
    for features in (f, bare, wrong, restored, copy.copy(f), dg.Features(**f.as_dict())):
        check(X, features)
    check(torch.cat([X, X + 1], 1)[:, :1], f)                       # rows two floats apart
    check(torch.cat([X, X[:5000]]), f, A.K + 5000)                  # not the K the runs were counted for
    assert dg.DeviceCsr(wl.rmat_csr(14, 24, seed=3)).features.hot_columns is None


@pytest.mark.gpu
def test_a_graph_does_not_depend_on_the_table():
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
    D.features.hot_columns.copy_(zeros_table())            # what becomes of the table is nothing to the graph
    for k in range(3):
        X.mul_(2.0)
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert (Y - want * 2.0 ** (k + 1)).abs().max() <= 1e-5 * scale * 2.0 ** (k + 1)


def zeros_table():
    """Calls every run hot and stages nothing: a product that looks at it is zero."""
    import torch
    return torch.tensor([-1, 0] * WORDS + [-1] * WORDS, dtype=torch.int32, device="cuda").repeat(4)


def device_matrix(A):
    """With int32 arrays, which the caller keeps."""
    import torch
    arrays = [torch.from_numpy(a).cuda() for a in (A.rowptr, A.colidx, A.vals)]
    return dg.DeviceCsr.from_device(A.M, A.K, *arrays), arrays


@pytest.mark.gpu
@pytest.mark.parametrize("by_argument", [True, False])
def test_the_table_s_memory_is_not_reused_under_a_product_on_another_stream(by_argument):
    """The matrix may go while its products on other streams are still to run: the arrays are the caller's, the table is not."""
    import torch
    A = matrix(*CASES[0])
    D, arrays = device_matrix(A)
    X = torch.randn(A.K, 1, device="cuda")
    want = D.spmm(X, algo=dg.NB_SR)
    side, busy = torch.cuda.Stream(), torch.randn(8192, 8192, device="cuda")
    Y = torch.empty(A.M, 1, device="cuda")
    torch.cuda.synchronize()
    print("[case] hot runs: the matrix goes before its product runs", flush=True)
    with torch.cuda.stream(side):
        for _ in range(20):
            busy @ busy
        if not by_argument:
            D.spmm(X, Y=Y)
    if by_argument:
        D.spmm(X, Y=Y, stream=side)
    table = D.features.hot_columns.data_ptr()
    del D
    blocks = [torch.full((4 * TABLE,), -1, dtype=torch.int32, device="cuda") for _ in range(64)]
    assert not side.query()                               # the product is still to come
    assert table not in [b.data_ptr() for b in blocks]
    torch.cuda.synchronize()
    assert (Y - want).abs().max() <= 1e-5 * want.abs().max()


@pytest.mark.gpu
def test_a_matrix_without_memory_for_a_table():
    """Arrays in the library's types are taken over without an allocation: where there is no memory for a table there is none."""
    import torch
    A = matrix(*CASES[0])
    D, arrays = device_matrix(A)
    X, Y = torch.randn(A.K, 1, device="cuda"), torch.empty(A.M, 1, device="cuda")
    want = D.spmm(X)
    assert D.features.hot_columns is not None
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    print("[case] hot runs: no memory for the table", flush=True)
    torch.cuda.set_per_process_memory_fraction(0.0)
    try:
        rest = []
        with pytest.raises(torch.OutOfMemoryError):
            while len(rest) < 100_000:
                rest.append(torch.empty(4 * TABLE, dtype=torch.int32, device="cuda"))
        bare = dg.DeviceCsr.from_device(A.M, A.K, *arrays)
        assert bare.features.hot_columns is None and bare.features.saved_share == D.features.saved_share
        bare.spmm(X, Y=Y)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert (Y - want).abs().max() <= 1e-5 * want.abs().max()


@pytest.mark.gpu
def test_streams_that_torch_does_not_know():
    """The allocator cannot be told of them for good: products go without the table, unless its memory is that stream's own."""
    import torch
    A = matrix(*CASES[0])
    X = torch.randn(A.K, 1, device="cuda")
    foreign = torch.cuda.ExternalStream(torch.cuda.Stream().cuda_stream)
    torch.cuda.synchronize()
    print("[case] hot runs on a foreign stream", flush=True)

    def looks_at_the_table(D, **stream):
        return not D.spmm(X, Y=torch.full((A.M, 1), float("nan"), device="cuda"), **stream).any()

    D, _ = device_matrix(A)
    D.features.hot_columns.copy_(zeros_table())
    assert looks_at_the_table(D)
    with torch.cuda.stream(torch.cuda.Stream()):
        assert looks_at_the_table(D)
    torch.cuda.synchronize()
    with torch.cuda.stream(foreign):
        assert not looks_at_the_table(D)
        own, _ = device_matrix(A)
        own.features.hot_columns.copy_(zeros_table())
        assert looks_at_the_table(own)
    torch.cuda.synchronize()
    assert not looks_at_the_table(D, stream=foreign)
