"""Rows whose entries several waves of a balanced kernel hold, in products without a launch that clears them first: calls that have
memory for it (RowSharing), against the oracle and against the calls of the C interface, which have none."""
import math
import os
import subprocess

import numpy as np
import pytest

import oracle
from paper_2106_16064_amd import binding as dg
from paper_2106_16064_amd import workloads as wl
from test_chunk_queues import queue_bytes, requested

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("check", ["every_part_once", "the_start_comes_late", "in_turn", "every_claim_ends", "ragged_blocks", "call_numbers",
                                   "workgroups_that_meet"])
def test_waves_agree_on_a_row(check, tmp_path):
    exe = tmp_path / "shared_rows_check"
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-o", str(exe), os.path.join(ROOT, "tests", "shared_rows_check.cpp")],
                   check=True)
    assert subprocess.run([str(exe), check], timeout=100).returncode == 0


def test_the_library_takes_random_numbers_without_exceptions():
    """Its entry points are C functions, and most of their callers never share rows: std::random_device throws where there is no source."""
    names = subprocess.run(["nm", "-D", "--undefined-only", os.path.join(ROOT, "paper_2106_16064_amd", "libdgsp.so")],
                           check=True, capture_output=True, text=True).stdout
    assert "getrandom" in names and "random_device" not in names


def rows_of(lens, K, seed):
    rng = np.random.default_rng(seed)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return wl.CsrMatrix(len(lens), K, rowptr, rng.integers(0, K, rowptr[-1]).astype(np.int32),
                        rng.uniform(-1, 1, rowptr[-1]).astype(np.float32), "rows", {})


def one_row():
    return rows_of([300_001], 5000, 1)


def ends_at_every_item():
    """Rows of 63, 64 and 65 items and their neighbours: a row's last entry, its end marker and the next row's first entry meet the
    chunks' ends (multiples of 64 items) in every order; long rows between them, empty ones at the ends."""
    lens = np.concatenate([[0, 0]] + [np.full(120, k) for k in range(60, 68)] + [[5000, 0, 0, 63, 20_000, 0]] +
                          [np.full(40, k) for k in range(125, 130)] + [[3001], np.zeros(70, int)])
    return rows_of(lens, 3001, 2)


def ends_at_32_items():
    """The same around 32 items, the quantum of nb_sr's run kernel."""
    lens = np.concatenate([[0]] + [np.full(150, k) for k in range(29, 35)] + [[900, 0, 31, 4000, 0, 0]] + [np.full(60, k) for k in (15, 16, 61, 62, 63)] +
                          [np.ones(90, int), [1500], np.zeros(33, int)])
    return rows_of(lens, 2003, 6)


def few_items():
    return rows_of([0, 3, 0, 29, 1, 33, 0, 64, 1], 70, 7)


def hubs():
    """A power-law graph's rows: hubs over many chunks, half of the rows empty; six million entries and more (entry blocks)."""
    return wl.rmat_csr(17, 56, seed=4)


CASES = [("one row", one_row), ("ends", ends_at_every_item), ("ends at 32", ends_at_32_items), ("few items", few_items), ("hubs", hubs)]


@pytest.mark.gpu
@pytest.mark.parametrize("name, make", CASES, ids=[c[0] for c in CASES])
def test_shared_rows(name, make):
    import torch
    A = make()
    D = dg.DeviceCsr(A)
    arrays = (D.rowptr, D.colidx, D.vals)
    for N in (1, 2, 3, 4, 5, 6, 7, 8, 16, 24, 41, 130):
        X = wl.dense_matrix(A.K, N, "normal", seed=N)
        Y0 = wl.dense_matrix(A.M, N, "uniform", seed=1)
        ref, bnd = oracle.spmm_ref(A.M, A.K, N, A.rowptr, A.colidx, A.vals, X)
        dX = torch.from_numpy(X).cuda()
        for algo in (dg.NB_PR, dg.NB_SR):
            print(f"[case] shared rows {name} N={N} algo={algo}", flush=True)
            Y = torch.full((A.M, N), float("nan"), device="cuda")
            # the run kernel takes NB_SR from four columns on, and NB_PR at five to eight unless the call is short
            run = N >= 4 if algo == dg.NB_SR else 5 <= N <= 8 and A.nnz >= 1_000_000
            for call in (lambda: dg.dgsp_spmm_csr(A.M, A.K, N, *arrays, dX, Y, algo),
                         lambda: dg.dgsp_spmm_csr_nnz(A.M, A.K, N, A.nnz, *arrays, dX, Y, algo),
                         lambda: dg.dgsp_spmm_csr_ld(A.M, A.K, N, A.nnz, *arrays, dX, Y, algo)):
                Y.fill_(float("nan"))
                memory = requested(call)
                # words for the rows, none for the queues that the largest calls have
                if run or (algo == dg.NB_PR and N <= 24):
                    assert memory > 0 and ((memory % 8 == 0 and memory not in queue_bytes(A.nnz, A.M)) or (run and N >= 41 and name == "hubs"))
                elif algo == dg.NB_SR:
                    assert memory == 0                         # a lane's items are cut further there, by the prepare launch
                ok, worst = oracle.within_bound(Y.cpu().numpy(), ref, bnd, 1e-5)
                assert ok, worst
            # against rows that the prepare launch has cleared: the same parts, added up in another order
            before = torch.full((A.M, N), float("nan"), device="cuda")
            for phase in (dg.PHASE_PREPARE, dg.PHASE_MAIN):
                dg.dgsp_spmm_csr_phase(A.M, A.K, N, A.nnz, *arrays, dX, before, algo, phase)
            ok, worst = oracle.within_bound(Y.cpu().numpy(), before.cpu().numpy().astype(np.float64), bnd, 1e-5)
            assert ok, worst
            for beta in (0.0, 0.5):                        # 0: the old values are not read
                Y.copy_(torch.from_numpy(Y0)) if beta else Y.fill_(float("nan"))
                memory = requested(lambda: dg.dgsp_spmm_csr_axpby(A.M, A.K, N, A.nnz, *arrays, dX, Y, -2.0, beta, algo))
                if algo == dg.NB_PR and not run:
                    assert memory > 0 or N > 24                # (many column groups: test_words_are_bounded)
                elif memory:                                   # the scaled run kernel has queues or its prepare launch
                    assert memory in queue_bytes(A.nnz, A.M)
                ok, worst = oracle.within_bound(Y.cpu().numpy(), -2.0 * ref + beta * Y0, 2.0 * bnd + beta * np.abs(Y0), 1e-5)
                assert ok, worst


LAYOUTS = {16: (2, 1), 32: (3, 1), 64: (4, 1), 128: (4, 2), 300: (5, 3)}       # log2 of the lanes a row of X, column blocks
ITEMS_A_CU = 700                                                                # kSharedRunItems


def workgroups(items, N, cus):
    """All column blocks' where nb_sr's run kernel shares rows: one a CU and as many more as the square root of the CU's items over 700,
    and no more than leave a wave 64 items, 128 below eight lanes.  None: as many as fit, four a CU."""
    lanes, blocks = LAYOUTS[N]
    per_cu = 1 + math.floor(math.sqrt(items * blocks / (cus * ITEMS_A_CU)))
    if per_cu >= 4:
        return None
    least = 64 if lanes >= 3 else 128
    most = min(cus * per_cu, math.ceil(items * blocks / (4 * least)))
    groups = max(1, int(most / blocks))
    return -(-groups * blocks // 8) * 8 if blocks == 2 else groups * blocks         # two blocks: every XCD works on one of them


@pytest.mark.gpu
@pytest.mark.parametrize("N", sorted(LAYOUTS))
def test_workgroups_follow_the_items(N):
    """Around the steps of the rule, from a single entry on: as many words as waves, and the right product."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    blocks = LAYOUTS[N][1]
    steps = [k * k * ITEMS_A_CU * cus // blocks for k in (1, 2, 3) if N <= 64 or k == 1]
    for items in [2, 33, 64, 65, 128, 129, 513, 1025, 64 * 4 * cus // blocks + 1] + [s + d for s in steps for d in (-1, 0, 1)]:
        M = 1 if items < 64 else max(1, min(items // 9, 3001))
        lens = np.random.default_rng(items).multinomial(items - M, np.full(M, 1.0 / M))
        A = rows_of(lens, 1501, items)
        assert A.nnz + A.M == items
        D = dg.DeviceCsr(A)
        X = wl.dense_matrix(A.K, N, "normal", seed=N)
        ref, bnd = oracle.spmm_ref(A.M, A.K, N, A.rowptr, A.colidx, A.vals, X)
        dX, Y = torch.from_numpy(X).cuda(), torch.full((A.M, N), float("nan"), device="cuda")
        print(f"[case] workgroups items={items} N={N}", flush=True)
        memory = requested(lambda: dg.dgsp_spmm_csr_nnz(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, dX, Y, dg.NB_SR))
        assert memory == 8 * 4 * (workgroups(items, N, cus) or 4 * cus)
        ok, worst = oracle.within_bound(Y.cpu().numpy(), ref, bnd, 1e-5)
        assert ok, worst


@pytest.mark.gpu
@pytest.mark.parametrize("N", [1, 16, 48, 127, 1009])
def test_words_are_bounded(N):
    """One word a chunk and column group, and a prime number of columns has as many groups: where that is more than two rounds of
    resident waves below eight columns a lane, or more than a megabyte, the prepare launch clears the rows."""
    import torch
    A = one_row()
    D = dg.DeviceCsr(A)
    X = wl.dense_matrix(A.K, N, "normal", seed=N)
    ref, bnd = oracle.spmm_ref(A.M, A.K, N, A.rowptr, A.colidx, A.vals, X)
    dX, Y = torch.from_numpy(X).cuda(), torch.full((A.M, N), float("nan"), device="cuda")
    print(f"[case] many column groups N={N}", flush=True)
    memory = requested(lambda: dg.dgsp_spmm_csr_nnz(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, dX, Y, dg.NB_PR))
    assert (memory > 0) == (N <= 48) and memory <= 1 << 20
    ok, worst = oracle.within_bound(Y.cpu().numpy(), ref, bnd, 1e-5)
    assert ok, worst


def long_rows():
    """Few rows, all over many chunks."""
    return rows_of(np.concatenate([[0, 0], np.full(30, 700), [3000, 0, 65, 2500], np.full(20, 333)]), 500, 5)


@pytest.mark.gpu
@pytest.mark.parametrize("N", [257, 300, 16129, 16130, 16131, 16132])
def test_shared_rows_in_several_column_blocks(N):
    """From 16129 on there are column blocks of 256 and the last one may have a single column: what is cleared and written under the
    sums of a row stays off the columns of the block before."""
    import torch
    A = long_rows()
    D = dg.DeviceCsr(A)
    X = wl.dense_matrix(A.K, N, "normal", seed=N)
    ref, bnd = oracle.spmm_ref(A.M, A.K, N, A.rowptr, A.colidx, A.vals, X)
    dX = torch.from_numpy(X).cuda()
    Y = torch.empty((A.M, N), device="cuda")
    print(f"[case] shared rows in several column blocks N={N}", flush=True)
    for call in (lambda: dg.dgsp_spmm_csr(A.M, A.K, N, D.rowptr, D.colidx, D.vals, dX, Y, dg.NB_SR),
                 lambda: dg.dgsp_spmm_csr_nnz(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, dX, Y, dg.NB_SR)):
        for _ in range(3):
            Y.fill_(float("nan"))
            assert requested(call) % (8 * -(-N // 256)) == 0 and requested(call) > 0      # words for every column block
            ok, worst = oracle.within_bound(Y.cpu().numpy(), ref, bnd, 1e-5)
            assert ok, worst


@pytest.mark.gpu
def test_calls_in_flight_together_and_in_a_graph():
    """Every call has words of its own; a product that is recorded takes the prepare launch, and its replays are right."""
    import torch
    A = ends_at_every_item()
    D = dg.DeviceCsr(A)
    N = 41
    X = wl.dense_matrix(A.K, N, "normal", seed=2)
    ref, bnd = oracle.spmm_ref(A.M, A.K, N, A.rowptr, A.colidx, A.vals, X)
    dX = torch.from_numpy(X).cuda()
    streams = [torch.cuda.Stream() for _ in range(4)]
    results = []
    torch.cuda.synchronize()
    print("[case] shared rows on four streams", flush=True)
    for i in range(40):
        with torch.cuda.stream(streams[i % 4]):
            Y = torch.full((A.M, N), float("nan"), device="cuda")
            dg.dgsp_spmm_csr_nnz(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, dX, Y, dg.NB_SR)
            results.append(Y)
    torch.cuda.synchronize()
    for Y in results:
        ok, worst = oracle.within_bound(Y.cpu().numpy(), ref, bnd, 1e-5)
        assert ok, worst
    print("[case] shared rows while a graph is recorded", flush=True)
    Y = torch.empty((A.M, N), device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        dg.dgsp_spmm_csr_nnz(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, dX, Y, dg.NB_SR)
    for _ in range(3):
        Y.fill_(float("nan"))
        graph.replay()
        dg.dgsp_spmm_csr_nnz(A.M, A.K, N, A.nnz, D.rowptr, D.colidx, D.vals, dX, results[0], dg.NB_SR)
        torch.cuda.synchronize()
        for y in (Y, results[0]):
            ok, worst = oracle.within_bound(y.cpu().numpy(), ref, bnd, 1e-5)
            assert ok, worst
