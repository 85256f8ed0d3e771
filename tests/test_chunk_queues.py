"""Products whose waves take chunks from queues (nb_sr_run_kernel, QUEUED), against the oracle.  The queues live in memory that the
call asks torch's allocator for, so its statistics tell that a product ran this way: by how much it asked for, as rows that waves
share without queues take memory, too."""
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_2106_16064_amd import binding as dg
from paper_2106_16064_amd import workloads as wl


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("check", ["pieces", "fits", "even_split"])
def test_how_items_are_shared_out(check, tmp_path):
    """The arithmetic that the prepare launch and the product have to agree on, against counting."""
    exe = tmp_path / "chunk_queues_check"
    subprocess.run(["g++", "-std=c++17", "-O1", "-o", str(exe), os.path.join(ROOT, "tests", "chunk_queues_check.cpp")], check=True)
    assert subprocess.run([str(exe), check], timeout=100).returncode == 0


def rows_of(lens, K, seed):
    rng = np.random.default_rng(seed)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return wl.CsrMatrix(len(lens), K, rowptr, rng.integers(0, K, rowptr[-1]).astype(np.int32),
                        rng.uniform(-1, 1, rowptr[-1]).astype(np.float32), "rows", {})


def graph(scale=19, degree=17):
    return wl.rmat_csr(scale, degree, seed=3)


def hub():
    """One row over a thousand chunks between rows of all lengths; empty rows at both ends."""
    rng = np.random.default_rng(1)
    lens = np.concatenate([np.zeros(700, int), rng.integers(0, 40, 200_000), [900_000], np.zeros(70_000, int), rng.integers(0, 40, 200_000),
                           np.zeros(1000, int)])
    return rows_of(lens, 50_001, 2)


def few_rows():
    """Every row over hundreds of chunks, fewer rows than threads of a workgroup, the last one long."""
    return rows_of(np.full(41, 220_000), 30_000, 3)


def ends_in_a_quantum():
    """Items a multiple of the quantum and of the chunks, so that the last chunk ends with the list."""
    lens = np.full(1 << 18, 35)
    lens[5], lens[6] = 35 + 3000, 35
    lens[9:9 + 100] -= 30
    return rows_of(lens, 1 << 18, 4)


def fewer_rows_than_queues():
    return rows_of(np.full(5, 1_900_000), 30_000, 3)


def odd_rows():
    """The prepare launch takes two rows a thread (2^19 of them and more): here its last thread has one, which is long."""
    lens = np.random.default_rng(5).integers(0, 38, (1 << 19) + 1)
    lens[-1] = 70_000
    return rows_of(lens, 40_000, 6)


CASES = [("fewer rows than queues", fewer_rows_than_queues, 64), ("graph", graph, 41), ("hub", hub, 45), ("few rows", few_rows, 64),
         ("aligned", ends_in_a_quantum, 44), ("three column blocks", few_rows, 300), ("pinned blocks", graph, 128),
         ("one line", lambda: graph(20, 17), 32), ("odd rows", odd_rows, 64)]


def allocations(call):
    import torch
    before = torch.cuda.memory_stats()["allocation.all.allocated"]
    call()
    return torch.cuda.memory_stats()["allocation.all.allocated"] - before


def requested(call):
    """Bytes of the one block that a call asks for, 0 for none."""
    import torch
    stats = torch.cuda.memory_stats()
    before = stats["allocation.all.allocated"], stats["requested_bytes.all.allocated"]
    call()
    stats = torch.cuda.memory_stats()
    assert stats["allocation.all.allocated"] - before[0] <= 1
    return stats["requested_bytes.all.allocated"] - before[1]


def queue_bytes(entries, M, lists=1):
    """What queues over so many entries take: a counter for each XCD in a line of its own, the first rows of chunks of 512 or 1024 items."""
    return {8 * lists * 128 + 4 * (-(-(entries + M) // size) + 1) for size in (512, 1024)}


@pytest.mark.gpu
@pytest.mark.parametrize("name, make, N", CASES, ids=[c[0] for c in CASES])
def test_products_from_queues(name, make, N):
    import torch
    A = make()
    D = dg.DeviceCsr(A)
    X = wl.dense_matrix(A.K, N, "normal", seed=2)
    Y0 = wl.dense_matrix(A.M, N, "uniform", seed=1)
    ref, bnd = oracle.spmm_ref(A.M, A.K, N, A.rowptr, A.colidx, A.vals, X)
    dX, Y = torch.from_numpy(X).cuda(), torch.full((A.M, N), float("nan"), device="cuda")
    print(f"[case] queues {name} N={N}", flush=True)
    queues = queue_bytes(A.nnz, A.M, 3 if N == 300 else 1)
    assert requested(lambda: dg.dgsp_spmm_csr_phase(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, dX, Y, dg.NB_SR, dg.PHASE_ALL, D.features)) in queues
    ok, worst = oracle.within_bound(Y.cpu().numpy(), ref, bnd, 1e-5)
    assert ok, worst
    Y = torch.from_numpy(Y0).cuda()
    assert requested(lambda: dg.dgsp_spmm_csr_axpby(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, dX, Y, -0.5, 1.5, dg.NB_SR, D.features)) in queues
    ok, worst = oracle.within_bound(Y.cpu().numpy(), -0.5 * ref + 1.5 * Y0, 0.5 * bnd + 1.5 * np.abs(Y0), 1e-5)
    assert ok, worst


@pytest.mark.gpu
@pytest.mark.parametrize("make, N, longer", [(graph, 41, 1.0001), (graph, 128, 1.5), (hub, 45, 1.1), (few_rows, 64, 2.0)])
def test_arrays_longer_than_the_matrix(make, N, longer):
    """Calls with a named kernel take the length of colidx for the entry count: chunks are then more or longer than one quantum."""
    import torch
    A = make()
    D = dg.DeviceCsr(A)
    room = int(A.nnz * longer) + 1
    colidx, vals = torch.zeros(room, dtype=torch.int32, device="cuda"), torch.full((room,), float("nan"), device="cuda")
    colidx[:A.nnz], vals[:A.nnz] = D.colidx, D.vals
    X = wl.dense_matrix(A.K, N, "normal", seed=2)
    Y0 = wl.dense_matrix(A.M, N, "uniform", seed=1)
    ref, bnd = oracle.spmm_ref(A.M, A.K, N, A.rowptr, A.colidx, A.vals, X)
    dX, Y = torch.from_numpy(X).cuda(), torch.full((A.M, N), float("nan"), device="cuda")
    print(f"[case] queues, arrays {longer} times as long N={N}", flush=True)
    queues = queue_bytes(room, A.M)
    assert requested(lambda: dg.dgsp_spmm_csr_phase(A.M, A.K, N, room, D.rowptr, colidx, vals, dX, Y, dg.NB_SR, dg.PHASE_ALL, D.features)) in queues
    ok, worst = oracle.within_bound(Y.cpu().numpy(), ref, bnd, 1e-5)
    assert ok, worst
    Y = torch.from_numpy(Y0).cuda()
    assert requested(lambda: dg.dgsp_spmm_csr_axpby(A.M, A.K, N, room, D.rowptr, colidx, vals, dX, Y, -0.5, 1.5, dg.NB_SR, D.features)) in queues
    ok, worst = oracle.within_bound(Y.cpu().numpy(), -0.5 * ref + 1.5 * Y0, 0.5 * bnd + 1.5 * np.abs(Y0), 1e-5)
    assert ok, worst


def short_rows():
    return rows_of(np.random.default_rng(7).integers(0, 9, 2_200_000), 40_000, 8)


@pytest.mark.gpu
@pytest.mark.parametrize("make, N, longer", [(graph, 41, 1.0), (odd_rows, 64, 1.3), (hub, 128, 30.0), (lambda: graph(17, 20), 41, 8.0),
                                             (lambda: graph(16, 20), 128, 16.0), (lambda: rows_of(np.full(41, 100_000), 30_000, 3), 300, 4.0),
                                             (short_rows, 41, 3.0), (lambda: rows_of(np.ones(3, int), 500, 1), 64, 4_000_000.0)])
def test_calls_that_know_no_entry_count(make, N, longer):
    """The length of colidx stands for it: queues are fitted to the matrix, from the fourth on down to equal shares - pinned column blocks,
    three lists, rows too short for queues, a single chunk."""
    import torch
    A = make()
    D = dg.DeviceCsr(A)
    room = int(A.nnz * longer)
    colidx, vals = torch.zeros(room, dtype=torch.int32, device="cuda"), torch.full((room,), float("nan"), device="cuda")
    colidx[:A.nnz], vals[:A.nnz] = D.colidx[:A.nnz], D.vals[:A.nnz]
    X = wl.dense_matrix(A.K, N, "normal", seed=2)
    ref, bnd = oracle.spmm_ref(A.M, A.K, N, A.rowptr, A.colidx, A.vals, X)
    dX = torch.from_numpy(X).cuda()
    for algo in (dg.AUTO, dg.NB_SR):
        Y = torch.full((A.M, N), float("nan"), device="cuda")
        print(f"[case] queues without an entry count, arrays {longer} times as long N={N}", flush=True)
        assert requested(lambda: dg.dgsp_spmm_csr(A.M, A.K, N, D.rowptr, colidx, vals, dX, Y, algo)) in queue_bytes(room, A.M, 3 if N == 300 else 1)
        ok, worst = oracle.within_bound(Y.cpu().numpy(), ref, bnd, 1e-5)
        assert ok, worst


@pytest.mark.gpu
def test_queues_of_calls_on_several_streams_and_none_in_a_graph():
    """Calls in flight together have queues of their own; a product that is recorded goes without."""
    import torch
    A = graph()
    D = dg.DeviceCsr(A)
    N = 41
    X = torch.randn(A.K, N, device="cuda")
    Y = torch.empty(A.M, N, device="cuda")
    want = D.spmm(X, algo=dg.RS_SR)
    scale = want.abs().max()
    streams = [torch.cuda.Stream() for _ in range(4)]
    torch.cuda.synchronize()
    print("[case] queues on four streams", flush=True)
    results = []
    for _ in range(3):
        for s in streams:
            with torch.cuda.stream(s):
                results.append(D.spmm(X))
    results.append(D.spmm(X, Y=torch.empty_like(Y), stream=streams[1]))
    torch.cuda.synchronize()
    for r in results:
        assert (r - want).abs().max() <= 1e-5 * scale
    del results
    side = streams[0]
    graph_ = torch.cuda.CUDAGraph()
    print("[case] queues while a graph is recorded", flush=True)
    with torch.cuda.graph(graph_, stream=side):
        assert allocations(lambda: D.spmm(X, Y=Y)) == 0
    assert allocations(lambda: D.spmm(X, Y=Y)) == 1
    for _ in range(3):
        Y.fill_(float("nan"))
        graph_.replay()
        torch.cuda.synchronize()
        assert (Y - want).abs().max() <= 1e-5 * scale
