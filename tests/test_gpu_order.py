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
