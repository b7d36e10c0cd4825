"""Bound plans whose stage 1 runs the bunches of long rows in column order
(x of 2.5 MB or more, 2,048 or more bunches): every bunch must run exactly
once, whatever the share of long rows and the workgroup size.  Integer-valued
inputs, so y is exact; y starts as NaN."""
import numpy as np
import pytest

import oracle
from helpers import note, to_dev, assert_exact, csr_from_lengths

pytestmark = pytest.mark.gpu

N = 330_001  # 2.64 MB of x in FP64

LENGTHS = {
    # long bunches only, and a number of them that 8 XCDs cannot share equally
    "all_long": [300_000, 260_000, 7],
    # long rows among short and empty ones
    "mixed": ([5] * 900 + [3000] + [0] * 3 + [1] * 40) * 70 + [200_000],
    # 9 long bunches in all (W = 4, S = 1): too few, the order is not taken
    "few_long": [4] * 140_000 + [2_500],
    # about one bunch in sixteen is long: where the order begins
    "at_the_limit": [4] * 140_000 + [40_000],
}


@pytest.mark.parametrize("name", sorted(LENGTHS))
@pytest.mark.parametrize("B", [1, 2, 3, 4])
def test_column_order_exact(name, B):
    import torch
    from paper_1504_06474_amd import sss
    note(f"[gpu-test] column order {name} B={B}")
    A, x = csr_from_lengths(LENGTHS[name], N, seed=B)
    rp, col, v, xx = to_dev(A, x)
    want = oracle.spmv(A.row_ptr, A.col, A.val, x)
    for W, S in ((4, 1), (8, 1)) if name == "mixed" else ((4, 1),):
        plan = sss.Plan(A.m, A.n, A.nnz, W=W, S=S, B=B, row_ptr=rp, bind_rows=True)
        for _ in range(2):
            y = torch.full((A.m,), float("nan"), dtype=torch.float64, device="cuda")
            plan.execute(rp, col, v, xx, y)
            assert_exact(y.cpu().numpy(), want)


def _strided_csr(lengths, n, seed):
    """Entry j of a row of length L in column j n / L: sorted and distinct."""
    import csrgen
    rng = csrgen.rng_for(seed)
    rp = np.zeros(len(lengths) + 1, dtype=np.int64)
    np.cumsum(lengths, out=rp[1:])
    each = np.repeat(lengths, lengths)
    j = np.arange(rp[-1]) - np.repeat(rp[:-1], lengths)
    val = rng.integers(-3, 4, rp[-1]).astype(np.float64)
    return csrgen.CSR(len(lengths), n, rp.astype(np.int32), (j * n // each).astype(np.int32), val), \
        rng.integers(-3, 4, n).astype(np.float64)


def test_column_order_per_call_exact():
    """Plans without bind_rows from 32M nonzeros on: every call orders the
    bunches of the row_ptr it is given (two structures on one plan, calls
    replayed from a graph, the one-call forms)."""
    import torch
    from paper_1504_06474_amd import sss
    note("[gpu-test] column order per call")
    rng = np.random.default_rng(5)
    lens = np.concatenate([[N, N - 1, 150_000], np.full(900, 9000), np.zeros(5000, int), rng.integers(1, 60, 760_000)])
    lens = np.append(lens.astype(np.int64), 0)
    lens[-1] = 32_000_001 - lens.sum() if lens.sum() < 32_000_001 else 1
    assert lens.max() <= N and lens.sum() >= 32_000_000
    A, x = _strided_csr(rng.permutation(lens), N, 1)
    A2, _ = _strided_csr(np.sort(lens), N, 2)
    d, d2 = to_dev(A, x), to_dev(A2, x)
    want, want2 = oracle.spmv(A.row_ptr, A.col, A.val, x), oracle.spmv(A2.row_ptr, A2.col, A2.val, x)
    y = torch.full((A.m,), float("nan"), dtype=torch.float64, device="cuda")
    for W, S, B in ((8, 5, 2), (4, 2, 3), (16, 1, 1)):
        plan = sss.Plan(A.m, A.n, A.nnz, W=W, S=S, B=B)
        for args, expect in ((d, want), (d2, want2), (d, want)):
            y.fill_(float("nan"))
            plan.execute(*args, y)
            assert_exact(y.cpu().numpy(), expect)
    plan = sss.Plan(A.m, A.n, A.nnz)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.execute(*d, y)
    for _ in range(3):
        y.fill_(float("nan"))
        g.replay()
        assert_exact(y.cpu().numpy(), want)
    for call in (sss.csr_spmv, sss.csr_spmv_noalloc):
        for args, expect in ((d2, want2), (d, want)):
            y.fill_(float("nan"))
            call(*args, y)
            assert_exact(y.cpu().numpy(), expect)
    sss.csr_spmv_cache_clear()


def test_cg_repeats_over_plans_in_column_order():
    """Within a bin the column order is that of atomics.  CG's dot products
    must not follow it: plans of the same matrix give the same bits.  Rows of
    one whole bunch each, which cross no boundary, among empty ones."""
    import torch
    from paper_1504_06474_amd import sss
    note("[gpu-test] column order, CG repeats")
    rng = np.random.default_rng(9)
    lens = np.zeros(N, dtype=np.int64)
    lens[rng.choice(N, 2900, replace=False)] = 256
    A, b = csr_from_lengths(lens, N, seed=1, int_valued=False)
    rp, col, v, db = to_dev(A, b)
    seen = None
    for _ in range(6):
        plan = sss.Plan(N, N, A.nnz, W=4, S=1, B=1, row_ptr=rp, bind_rows=True)
        x, r, p, q = (torch.zeros(N, dtype=torch.float64, device="cuda") for _ in range(4))
        work = torch.zeros(sss.cg_workspace_size() // 8, dtype=torch.float64, device="cuda")
        sss.cg_start(plan, rp, col, v, db, x, r, p, q, work)
        sss.cg_iterate(plan, rp, col, v, x, r, p, q, work, 2)
        if seen is not None:
            assert torch.equal(x, seen)
        seen = x


@pytest.mark.parametrize("sort", [True, False], ids=["sorted", "unsorted"])
@pytest.mark.parametrize("kind", ["f64", "f32", "bf16"])
def test_column_order_changes_no_bit(kind, sort):
    """The order decides when a bunch runs, not what it adds: the bits of the
    two-stage form, for columns sorted within their rows or not."""
    import torch
    from helpers import to_dev_precision
    from paper_1504_06474_amd import sss
    note(f"[gpu-test] column order, bits {kind} {sort}")
    n = N if kind == "f64" else 2 * N
    A, x = csr_from_lengths(LENGTHS["mixed"], n, seed=4, int_valued=False)
    if not sort:
        rng = np.random.default_rng(8)
        for r in np.flatnonzero(np.diff(A.row_ptr) > 1):
            a, b = A.row_ptr[r], A.row_ptr[r + 1]
            A.col[a:b] = rng.permutation(A.col[a:b])
    rp, col, v, xx = to_dev_precision(A, x, kind)[:4]
    for W, S in ((4, 1), (8, 1)):
        args = dict(dtype=v.dtype, W=W, S=S, row_ptr=rp)
        want = sss.Plan(A.m, A.n, A.nnz, debug=True, **args).execute(rp, col, v, xx).clone()
        assert torch.equal(sss.Plan(A.m, A.n, A.nnz, bind_rows=True, **args).execute(rp, col, v, xx), want)


@pytest.mark.parametrize("B", [1, 3])
def test_column_order_row_ptr_rewritten(B):
    """Slots in column order carry the rows and spans of the row_ptr they were
    made from.  Rewritten in place (same rows, same entries): short rows
    only, the long rows elsewhere, empty rows in front, behind and between."""
    import torch
    from paper_1504_06474_amd import sss
    note(f"[gpu-test] column order, rewritten B={B}")
    lens = np.array(LENGTHS["mixed"], dtype=np.int64)
    A, x = csr_from_lengths(lens, N, seed=2)
    rp, col, v, xx = to_dev(A, x)
    plan = sss.Plan(A.m, A.n, A.nnz, W=4, S=1, B=B, row_ptr=rp, bind_rows=True)
    rng = np.random.default_rng(B)
    even = np.full(A.m, A.nnz // A.m, dtype=np.int64)
    even[: A.nnz % A.m] += 1
    few = np.zeros(A.m, dtype=np.int64)
    few[rng.choice(A.m, 5000, replace=False)] = 1
    few *= A.nnz // 5000
    few[np.flatnonzero(few)[-1]] += A.nnz - few.sum()
    front = np.concatenate([np.zeros(A.m - 2000, np.int64), np.full(2000, A.nnz // 2000, np.int64)])
    front[-1] += A.nnz - front.sum()
    y = torch.empty(A.m, dtype=torch.float64, device="cuda")
    for new in (lens[::-1].copy(), rng.permutation(lens), even, few, front, front[::-1].copy(), lens):
        rp2 = np.zeros(A.m + 1, dtype=np.int32)
        np.cumsum(new, out=rp2[1:])
        assert rp2[-1] == A.nnz
        rp.copy_(torch.from_numpy(rp2).to("cuda"))
        want = oracle.spmv(rp2, A.col, A.val, x)
        for _ in range(2):
            y.fill_(float("nan"))
            plan.execute(rp, col, v, xx, y)
            assert_exact(y.cpu().numpy(), want)
