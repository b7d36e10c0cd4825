"""A bound plan that saw no row cross into a bunch by more than 64 entries
leaves the carry launch out.  row_ptr rewritten in place with such rows: the
last of a row's bunches to finish adds up its parts.  Exact (integer-valued
inputs), the same bits every time, and at about the time of a plan that knew."""
import time

import numpy as np
import pytest

import oracle
from helpers import note, assert_exact, csr_from_lengths, to_dev_precision

pytestmark = pytest.mark.gpu


def structures(m, nnz, SWT):
    """Row lengths (of m rows, nnz entries) whose long rows begin with a bunch,
    inside one, 64 and 65 entries before one, and end on and off a boundary."""
    out = []
    for head in ([], [SWT // 2], [SWT - 64], [SWT - 65], [3] * 40 + [0] * 5):
        for rows in ([SWT + 1], [2 * SWT], [SWT * 3 + 17, 0, SWT * 2, SWT * 2], [SWT + 64, SWT + 65], [nnz - sum(head)],
                     [20 * SWT + 5, 1, 1, 18 * SWT]):
            if sum(head) + sum(rows) <= nnz:
                lens = head + rows
                left = nnz - sum(lens)
                rest = m - len(lens)
                lens = lens + [left // rest + (1 if i < left % rest else 0) for i in range(rest)]
                assert len(lens) == m and sum(lens) == nnz
                out.append(np.array(lens, dtype=np.int64))
    return out


def to_row_ptr(lens):
    rp = np.zeros(len(lens) + 1, dtype=np.int32)
    np.cumsum(lens, out=rp[1:])
    return rp


@pytest.mark.parametrize("kind", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("W,S", [(4, 1), (8, 2), (16, 1)])
def test_long_rows_a_plan_did_not_know(kind, W, S):
    import torch
    from paper_1504_06474_amd import sss
    note(f"[gpu-test] rewritten {kind} W={W} S={S}")
    SWT = 64 * W * S
    m, nnz = 60 * SWT // 8, 60 * SWT
    A, x = csr_from_lengths([8] * m, 5000, seed=W)
    rp, col, v, xx, ve, xe = to_dev_precision(A, x, kind)
    plan = sss.Plan(m, A.n, nnz, dtype=v.dtype, W=W, S=S, row_ptr=rp, bind_rows=True)
    y = torch.empty(m, dtype=xx.dtype, device="cuda")
    yb = torch.empty(m, dtype=xx.dtype, device="cuda")
    batches = [sss.BatchPlan([(rp, col, v, xx, yb, A.n)], dtype=v.dtype, W=W, S=S, persistent=p) for p in (False, True)]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.execute(rp, col, v, xx, y)
    for lens in structures(m, nnz, SWT):
        rp2 = to_row_ptr(lens)
        rp.copy_(torch.from_numpy(rp2).to("cuda"))
        want = oracle.spmv(rp2, A.col, ve, xe)
        for call in (lambda: plan.execute(rp, col, v, xx, y), g.replay, lambda: plan.execute(rp, col, v, xx, y)):
            y.fill_(float("nan"))
            call()
            assert_exact(y.double().cpu().numpy(), want)
        for batch in batches:
            yb.fill_(float("nan"))
            batch.execute()
            assert_exact(yb.double().cpu().numpy(), want)


def test_unknown_long_row_same_bits_and_time():
    """One row of 1M entries: shared out over its 390 bunches like any other
    row (a wavefront alone took 8 ms)."""
    import torch
    from paper_1504_06474_amd import sss
    note("[gpu-test] rewritten, time")
    N = 1_000_000
    A, x = csr_from_lengths([8] * (2 * N // 8), 100_000, seed=3, int_valued=False)
    rp, col, v, xx = to_dev_precision(A, x, "f64")[:4]
    plan = sss.Plan(A.m, A.n, A.nnz, row_ptr=rp, bind_rows=True)
    rest = A.m - 2
    lens = np.array([5, N - 5] + [N // rest + (1 if i < N % rest else 0) for i in range(rest)], dtype=np.int64)
    rp2 = to_row_ptr(lens)
    rp.copy_(torch.from_numpy(rp2).to("cuda"))
    want, scale = oracle.spmv(rp2, A.col, A.val, x), oracle.abs_spmv(rp2, A.col, A.val, x)
    y = plan.execute(rp, col, v, xx).clone()
    assert np.all(np.abs(y.cpu().numpy() - want) <= 1e-12 * scale)
    ms = []
    for _ in range(20):
        torch.cuda.synchronize()
        t = time.perf_counter()
        again = plan.execute(rp, col, v, xx)
        torch.cuda.synchronize()
        ms.append((time.perf_counter() - t) * 1e3)
        assert torch.equal(again, y)
    assert min(ms) < 0.5


@pytest.mark.parametrize("W,S", [(4, 1), (8, 2)])
def test_cg_over_long_rows_the_plan_did_not_know(W, S):
    """The product with p.q beside it, on a row_ptr rewritten in place: one
    step's scalars against numpy's, the same bits every time."""
    import torch
    from paper_1504_06474_amd import sss
    note(f"[gpu-test] rewritten cg W={W} S={S}")
    SWT = 64 * W * S
    m, nnz = 60 * SWT // 8, 60 * SWT
    A, _ = csr_from_lengths([8] * m, m, seed=W, int_valued=False)
    b = np.random.default_rng(2).uniform(-1, 1, m)
    rp, col, v, db = to_dev_precision(A, b, "f64")[:4]
    plan = sss.Plan(m, m, nnz, W=W, S=S, row_ptr=rp, bind_rows=True)
    for lens in structures(m, nnz, SWT):
        rp2 = to_row_ptr(lens)
        rp.copy_(torch.from_numpy(rp2).to("cuda"))
        q = oracle.spmv(rp2, A.col, A.val, b)
        alpha = b @ b / (b @ q)
        seen = None
        for _ in range(3):
            x, r, d, qd = (torch.zeros(m, dtype=torch.float64, device="cuda") for _ in range(4))
            work = torch.zeros(sss.cg_workspace_size() // 8, dtype=torch.float64, device="cuda")
            sss.cg_start(plan, rp, col, v, db, x, r, d, qd, work)
            sss.cg_iterate(plan, rp, col, v, x, r, d, qd, work, 1)
            # p.q is a sum of m products: each side within (m + 100) 2^-53 of sum |p q|,
            # on top of 1e-12 (|A||p|) in q
            size = np.abs(b) @ oracle.abs_spmv(rp2, A.col, A.val, b)
            tol = 2 * (1e-12 + (m + 100) * 2.0 ** -53) * size / abs(b @ q) + 1e-12
            assert np.linalg.norm(x.cpu().numpy() - alpha * b) <= tol * np.linalg.norm(alpha * b)
            if seen is not None:
                assert torch.equal(x, seen)
            seen = x
