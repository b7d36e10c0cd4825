"""CG steps over every branch of the product that forms p.q itself, three of
them against numpy's on the oracle's products, normwise 1e-11 (two FP64 runs
that differ in the order of their sums only stay within 1e-14)."""
import numpy as np
import pytest

import csrgen
import oracle
from helpers import note, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,W,S,B", [(600, 4, 2, 2), (1150, 8, 5, 2), (640, 4, 2, 1), (790, 4, 2, 2), (795, 4, 2, 2)])
def test_steps_of_the_dot_branches(grid, W, S, B):
    """The branches of the product that forms p.q: 1,025 sums and more (600^2:
    1,756), non-temporal loads (1150^2: 106 MB with 10.6 MB of x, 1,291 sums), and
    both sides of the most sums it forms (3,072; 640^2 at B = 1: 3,995, 790^2:
    3,045, 795^2: 3,083)."""
    import torch
    from paper_1504_06474_amd import sss
    note(f"[gpu-test] cg steps {grid} W={W} S={S} B={B}")
    A = csrgen.laplacian2d_csr(grid)
    b = csrgen.rng_for(grid).uniform(-1, 1, A.m)
    rp, col, v, db = to_dev(A, b)
    plan = sss.Plan(A.m, A.m, A.nnz, W=W, S=S, B=B, row_ptr=rp, bind_rows=True)
    vec = [torch.zeros(A.m, dtype=torch.float64, device="cuda") for _ in range(4)]
    work = torch.zeros(sss.cg_workspace_size() // 8, dtype=torch.float64, device="cuda")
    sss.cg_start(plan, rp, col, v, db, *vec, work)
    sss.cg_iterate(plan, rp, col, v, *vec, work, 3)
    x, r, p = np.zeros(A.m), b.copy(), b.copy()
    for _ in range(3):
        q = oracle.spmv(A.row_ptr, A.col, A.val, p)
        alpha = r @ r / (p @ q)
        x, r_new = x + alpha * p, r - alpha * q
        p = r_new + (r_new @ r_new) / (r @ r) * p
        r = r_new
    for got, want in zip(vec, (x, r, p)):
        assert np.linalg.norm(got.cpu().numpy() - want) <= 1e-11 * max(np.linalg.norm(want), np.linalg.norm(b))
