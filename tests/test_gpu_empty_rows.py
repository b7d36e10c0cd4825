"""Rows without entries by the million: y exact, and in a time that the rows
alone explain.  Integer-valued inputs; y starts as NaN."""
import time

import numpy as np
import pytest

import oracle
from helpers import note, assert_exact, csr_from_lengths, to_dev_precision

pytestmark = pytest.mark.gpu


def best_ms(f, runs=4):
    import torch
    out = []
    for _ in range(runs):
        torch.cuda.synchronize()
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        out.append((time.perf_counter() - t) * 1e3)
    return min(out)


def check(lens, n, kind="f64", seed=5, **plan):
    """y of both plan forms against the oracle; the time of the slower one."""
    import torch
    from paper_1504_06474_amd import sss
    A, x = csr_from_lengths(lens, n, seed=seed)
    rp, col, v, xx, ve, xe = to_dev_precision(A, x, kind)
    want = oracle.spmv(A.row_ptr, A.col, ve, xe)
    y = torch.empty(A.m, dtype=xx.dtype, device="cuda")
    ms = 0.0
    for bind in (True, False):
        p = sss.Plan(A.m, A.n, A.nnz, dtype=v.dtype, row_ptr=rp, bind_rows=bind, **plan)
        y.fill_(float("nan"))
        p.execute(rp, col, v, xx, y)
        assert_exact(y.double().cpu().numpy(), want)
        ms = max(ms, best_ms(lambda: p.execute(rp, col, v, xx, y)))
    return ms


@pytest.mark.parametrize("B", [1, 2, 3, 4])
@pytest.mark.parametrize("kind", ["f64", "bf16"])
def test_leading_rows_shared_out(kind, B):
    """The leading rows' shares: fewer rows than wavefronts, one more and one
    less than a share, wavefronts without a bunch."""
    note(f"[gpu-test] leading rows {kind} B={B}")
    for lead in (1, 63, 64, 65, 4095, 4096, 8191 * B, 8192 * B + 1, 100_003):
        for W, S in ((4, 1), (8, 5)):
            check([0] * lead + [7] * 300 + [0, 0, 5], 900, kind, W=W, S=S, B=B)
    # slots in column order, some of them empty
    check([0] * 50_000 + [300_000, 260_000, 7], 330_001, kind, W=4, S=1, B=B)


def test_leading_rows_take_their_stores_time():
    """4M leading rows, 32 MB of y: one wavefront's stores alone take 2 ms, a
    load waited for per 64 rows takes 60,000 times its latency, 10 ms and more."""
    note("[gpu-test] leading rows, time")
    for rows in (1, 1000):
        assert check([0] * 4_000_000 + [5] * rows, 1000) < 3.0


def test_rows_between_and_behind_take_one_pass():
    """A million empty rows inside a tile and behind the last entry: one
    wavefront reads their row_ptr twice (to count, to store), 64 a round, each
    round about a load's latency: 11 ms, where marking the tile 64 times a
    round and waiting for the stores as well made it 44."""
    note("[gpu-test] empty rows inside a tile, time")
    few = [3] * 20 + [0, 0, 0, 1]
    assert check(few * 20 + [0] * 1_000_000 + few * 20, 1000) < 25.0
    assert check(few * 20 + [0] * 1_000_000, 1000) < 25.0


@pytest.mark.parametrize("kind", ["f64", "f32", "bf16"])
def test_runs_of_empty_rows(kind):
    """Runs of every length around a chunk of 64 rows, one after another and at
    the ends of tiles, over more than the 64 chunks a bunch keeps."""
    note(f"[gpu-test] runs of empty rows {kind}")
    lens = []
    for run in list(range(0, 5)) + list(range(60, 70)) + list(range(125, 131)) + [700, 64 * 70, 3, 64 * 3]:
        lens += [0] * run + [1, 2] + [0] * run + [61]
    for W, S in ((4, 1), (8, 2), (16, 3)):
        check(lens, 500, kind, W=W, S=S)
