"""The one-launch execute (fused kernel) where it can go wrong: rows that
cross a bunch boundary by 0 to 64 entries and by more, row spans around the
64 and 128 row_ptr entries that a bunch loads ahead, more than 4,096 rows in
a bunch, ragged ends, rows the plan did not know of, streamed and wide forms.

Integer-valued inputs are exact against the oracle.  On other values the
fused kernel must give the two stages' y (a debug plan runs them) bit for
bit: it adds the same partial sums in the same order."""
import numpy as np
import pytest

import csrgen
import oracle
from helpers import note, assert_exact, csr_from_lengths, to_dev_precision

pytestmark = pytest.mark.gpu

DTYPES = ("f64", "f32", "bf16")


def torch_types(kind):
    import torch
    return {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}[kind], \
        torch.float64 if kind == "f64" else torch.float32


def patterns():
    rng = csrgen.rng_for(7)
    out = {f"rows_of_{L}": [L] * (6000 // L + 3) for L in (1, 2, 4, 63, 64, 65, 66, 130, 300)}
    out["rows_of_5000"] = [5000, 3, 5000, 5000, 1]
    out["around_64_rows"] = list(rng.integers(3, 6, 3000))
    out["around_128_rows"] = list(rng.integers(1, 4, 4000))
    out["empty_between"] = [x for v in rng.integers(0, 70, 300) for x in (int(v), 0)]
    out["empty_runs"] = [9] * 40 + [0] * 70 + [3] * 100 + [0] * 5000 + [80] * 9 + [0] * 300
    out["leading_empty"] = [0] * 3000 + [33] * 200
    out["one_entry"] = [0, 0, 1, 0]
    return {k: [int(v) for v in lens] for k, lens in out.items()}


PATTERNS = patterns()


def run(plan, rp, col, v, xx, m, ydt):
    import torch
    y = torch.full((m,), float("nan"), dtype=ydt, device="cuda")
    return plan.execute(rp, col, v, xx, y).cpu()


@pytest.mark.parametrize("kind", DTYPES)
@pytest.mark.parametrize("name", sorted(PATTERNS))
def test_fused_exact_and_same_bits(name, kind):
    import torch
    from paper_1504_06474_amd import sss
    vt, yt = torch_types(kind)
    note(f"[gpu-test] fused {name} {kind}")
    A, x = csr_from_lengths(PATTERNS[name], 6000, seed=3)
    U, ux = csr_from_lengths(PATTERNS[name], 6000, seed=3, int_valued=False)
    want = oracle.spmv(A.row_ptr, A.col, A.val, x)
    di, du = to_dev_precision(A, x, kind)[:4], to_dev_precision(U, ux, kind)[:4]
    for W, S in ((4, 1), (4, 3), (8, 2), (16, 1)):
        split = sss.Plan(A.m, A.n, A.nnz, dtype=vt, W=W, S=S, debug=True)
        bits = run(split, *du, A.m, yt)
        for bind in (True, False):
            for d, check in ((di, False), (du, True)):
                plan = sss.Plan(A.m, A.n, A.nnz, dtype=vt, W=W, S=S, row_ptr=d[0], bind_rows=bind)
                y = run(plan, *d, A.m, yt)
                if check:
                    assert torch.equal(y, bits), (W, S, bind)
                else:
                    assert_exact(y.double().numpy(), want)
    # the same matrix twice in a batch, beside one with no nonzero
    ys = [torch.full((A.m,), float("nan"), dtype=yt, device="cuda") for _ in range(2)]
    y0 = torch.full((70,), float("nan"), dtype=yt, device="cuda")
    e = torch.empty(0, dtype=torch.int32, device="cuda")
    mats = [(*di, ys[0], A.n), (torch.zeros(71, dtype=torch.int32, device="cuda"), e, e.to(vt), di[3], y0, A.n),
            (*di, ys[1], A.n)]
    for persistent in (False, True):
        batch = sss.BatchPlan(mats, dtype=vt, persistent=persistent)
        for y in ys + [y0]:
            y.fill_(float("nan"))
        batch.execute()
        for y in ys:
            assert_exact(y.double().cpu().numpy(), want)
        assert y0.tolist() == [0.0] * 70


@pytest.mark.parametrize("kind", DTYPES)
def test_bound_plan_meets_long_rows_it_did_not_know(kind):
    """Planned with rows of 8 (no carry launch), then row_ptr rewritten in
    place with a row over many bunches, and with empty rows before it."""
    import torch
    from paper_1504_06474_amd import sss
    vt, yt = torch_types(kind)
    note(f"[gpu-test] fused rewritten {kind}")
    A, x = csr_from_lengths([8] * 2000, 16000, seed=1)
    rp, col, v, xx = to_dev_precision(A, x, kind)[:4]
    plan = sss.Plan(A.m, A.n, A.nnz, dtype=vt, W=4, S=2, row_ptr=rp, bind_rows=True)
    assert_exact(run(plan, rp, col, v, xx, A.m, yt).double().numpy(), oracle.spmv(A.row_ptr, A.col, A.val, x))
    for lens in ([0] * 100 + [9000] + [0] * 100 + [100] * 60 + [1] * 739 + [261], [1] * 1000 + [0] * 900 + [150] * 100):
        lens = np.array(lens + [0] * (A.m - len(lens)), dtype=np.int64)
        assert lens.sum() == A.nnz and len(lens) == A.m
        rp2 = np.zeros(A.m + 1, dtype=np.int32)
        np.cumsum(lens, out=rp2[1:])
        rp.copy_(torch.from_numpy(rp2).to("cuda"))
        assert_exact(run(plan, rp, col, v, xx, A.m, yt).double().numpy(), oracle.spmv(rp2, A.col, A.val, x))


def test_entries_past_the_end_add_nothing():
    """The last tile's idle lanes read column 0: an infinite x[0] that no row
    uses must not reach y."""
    from paper_1504_06474_amd import sss
    A, x = csr_from_lengths([3] * 101, 500, seed=2)
    A.col[A.col == 0] = 1
    x[0] = 0.0
    want = oracle.spmv(A.row_ptr, A.col, A.val, x)
    x[0] = np.inf
    rp, col, v, xx = to_dev_precision(A, x, "f64")[:4]
    import torch
    for bind in (True, False):
        plan = sss.Plan(A.m, A.n, A.nnz, row_ptr=rp, bind_rows=bind)
        assert_exact(run(plan, rp, col, v, xx, A.m, torch.float64).numpy(), want)


@pytest.mark.parametrize("kind", DTYPES)
def test_streamed_form(kind):
    """A matrix past the last-level cache: non-temporal loads.  Six copies of a
    smaller one below each other."""
    import torch
    from paper_1504_06474_amd import sss
    vt, yt = torch_types(kind)
    rows = {"f64": 200_003, "f32": 300_007, "bf16": 400_003}[kind]
    note(f"[gpu-test] fused streamed {kind}")
    A, x = csr_from_lengths([27] * rows, 20_000, seed=4)
    rp, col, v, xx = to_dev_precision(A, x, kind)[:4]
    m, nnz = 6 * A.m, 6 * A.nnz
    rp = torch.cat([rp[:-1] + k * A.nnz for k in range(6)] + [torch.tensor([nnz], dtype=torch.int32, device="cuda")])
    plan = sss.Plan(m, A.n, nnz, dtype=vt, W=8, S=2, row_ptr=rp, bind_rows=True)
    y = run(plan, rp, col.repeat(6), v.repeat(6), xx, m, yt).double().numpy()
    assert_exact(y, np.tile(oracle.spmv(A.row_ptr, A.col, A.val, x), 6))


@pytest.mark.parametrize("kind", ["f64", "f32"])
def test_wide_x(kind):
    """x of more than 4 GB: gathers past a 32-bit byte offset, single and batch."""
    import torch
    from paper_1504_06474_amd import sss
    vt, yt = torch_types(kind)
    n = {"f64": 540_000_011, "f32": 1_080_000_007}[kind]
    note(f"[gpu-test] fused wide x {kind}")
    A, x = csr_from_lengths([7] * 400 + [200] * 5, 5000, seed=6)
    spread = (np.arange(5000, dtype=np.int64) * ((n - 1) // 4999)).astype(np.int32)
    rp, col, v, xx = to_dev_precision(A, x, kind)[:4]
    big = torch.zeros(n, dtype=yt, device="cuda")
    big[torch.from_numpy(spread).to("cuda").long()] = xx
    col = torch.from_numpy(spread).to("cuda")[col.long()].contiguous()
    want = oracle.spmv(A.row_ptr, A.col, A.val, x)
    plan = sss.Plan(A.m, n, A.nnz, dtype=vt, W=4, S=2, row_ptr=rp, bind_rows=True)
    assert_exact(run(plan, rp, col, v, big, A.m, yt).double().numpy(), want)
    y = torch.full((A.m,), float("nan"), dtype=yt, device="cuda")
    sss.BatchPlan([(rp, col, v, big, y, n)], dtype=vt).execute()
    assert_exact(y.double().cpu().numpy(), want)


@pytest.mark.parametrize("W,S,B", [(4, 1, 2), (8, 2, 3), (16, 1, 1), (4, 3, 4)])
@pytest.mark.parametrize("grid", [5, 60])
def test_product_with_dot(grid, W, S, B):
    """CG steps whose product forms p.q itself (bound plans without long
    crossing rows), on a Laplacian with some unknowns taken out: their rows
    are empty, so tiles are dirty.  Three steps against numpy's, normwise
    1e-11 as the CG tests have it."""
    import torch
    from paper_1504_06474_amd import sss
    note(f"[gpu-test] product with dot {grid} W={W} S={S} B={B}")
    L = csrgen.laplacian2d_csr(grid)
    out = np.zeros(L.m, dtype=bool)
    out[csrgen.rng_for(3).choice(L.m, L.m // 6, replace=False)] = True
    out[:2] = True
    rows = np.repeat(np.arange(L.m), np.diff(L.row_ptr))
    keep = ~(out[rows] | out[L.col])
    rp = np.zeros(L.m + 1, dtype=np.int32)
    np.cumsum(np.bincount(rows[keep], minlength=L.m), out=rp[1:])
    A = csrgen.CSR(L.m, L.m, rp, L.col[keep], L.val[keep])
    b = np.where(out, 0.0, csrgen.rng_for(4).uniform(-1, 1, L.m))
    drp, col, v, db = to_dev_precision(A, b, "f64")[:4]
    plan = sss.Plan(A.m, A.m, A.nnz, W=W, S=S, B=B, row_ptr=drp, bind_rows=True)
    vec = [torch.zeros(A.m, dtype=torch.float64, device="cuda") for _ in range(4)]
    work = torch.zeros(sss.cg_workspace_size() // 8, dtype=torch.float64, device="cuda")
    sss.cg_start(plan, drp, col, v, db, vec[0], vec[1], vec[2], vec[3], work)
    sss.cg_iterate(plan, drp, col, v, *vec, work, 3)
    x, r, p = np.zeros(A.m), b.copy(), b.copy()
    for _ in range(3):
        q = oracle.spmv(A.row_ptr, A.col, A.val, p)
        alpha = r @ r / (p @ q)
        x, r_new = x + alpha * p, r - alpha * q
        p = r_new + (r_new @ r_new) / (r @ r) * p
        r = r_new
    for got, want in zip(vec, (x, r, p)):
        assert np.linalg.norm(got.cpu().numpy() - want) <= 1e-11 * max(np.linalg.norm(want), np.linalg.norm(b))


@pytest.mark.parametrize("W", [4, 8, 16])
def test_bf16_odd_last_value(W):
    """An odd number of BF16 values ends inside a 32-bit word: every place of
    the last value in a tile's lanes, one tile and more; val ends where its
    array does."""
    import torch
    from paper_1504_06474_amd import sss
    note(f"[gpu-test] bf16 odd W={W}")
    tile = 64 * W
    for nnz in [1, 3, 5, 7, 9, 63, 65, tile - 1, tile + 1, 2 * tile - 1, 2 * tile + 3, 3 * tile + tile // 2 + 5]:
        A, x = csr_from_lengths([2] * (nnz // 2) + [nnz % 2], 4000, seed=nnz)
        A.val[-1], x[A.col[-1]] = 3.0, 2.0
        rp, col, v, xx, ve, xe = to_dev_precision(A, x, "bf16")
        want = oracle.spmv(A.row_ptr, A.col, ve, xe)
        for S in (1, 3):
            for bind in (True, False):
                plan = sss.Plan(A.m, A.n, A.nnz, dtype=torch.bfloat16, W=W, S=S, row_ptr=rp, bind_rows=bind)
                assert_exact(run(plan, rp, col, v, xx, A.m, torch.float32).double().numpy(), want)


@pytest.mark.parametrize("nnz,W,S", [(649_999, 4, 1), (650_000, 8, 1), (2_299_999, 8, 1), (2_300_000, 8, 2),
                                     (7_999_999, 8, 2), (8_000_000, 8, 5)])
def test_one_call_schedule(nnz, W, S):
    """The one-call forms run the schedule that their lines give: the bits of a
    plan of that W and S, on both sides of each line."""
    import torch
    from paper_1504_06474_amd import sss
    note(f"[gpu-test] one-call schedule {nnz}")
    g = torch.Generator(device="cuda")
    g.manual_seed(nnz)
    m = 3001
    lens = torch.full((m,), nnz // m, dtype=torch.int64, device="cuda")
    lens[: nnz % m] += 1
    rp = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(lens, 0, out=rp[1:])
    rp = rp.to(torch.int32)
    col = torch.randint(0, 5000, (nnz,), generator=g, device="cuda", dtype=torch.int32)
    v = torch.rand(nnz, generator=g, device="cuda", dtype=torch.float64) - 0.5
    x = torch.rand(5000, generator=g, device="cuda", dtype=torch.float64) - 0.5
    want = sss.Plan(m, 5000, nnz, W=W, S=S).execute(rp, col, v, x)
    other = sss.Plan(m, 5000, nnz, W=16, S=3).execute(rp, col, v, x)
    assert not torch.equal(other, want)  # (the bits do tell schedules apart)
    for call in (sss.csr_spmv, sss.csr_spmv_noalloc):
        assert torch.equal(call(rp, col, v, x, torch.empty_like(want)), want)
    sss.csr_spmv_cache_clear()


@pytest.mark.parametrize("kind", DTYPES)
@pytest.mark.parametrize("W,S", [(4, 1), (8, 2), (16, 1)])
def test_short_crossing_rows_beside_long_ones(kind, W, S):
    """One row that the carry launch is made for: it then also completes the
    rows that cross by 1 to 64 entries, bound, searched and in batches, with the
    two stages' bits."""
    import torch
    from paper_1504_06474_amd import sss
    vt, yt = torch_types(kind)
    note(f"[gpu-test] crossing rows {kind} W={W} S={S}")
    SWT = 64 * W * S
    lens = [SWT - 1, 2, SWT - 65, 64 + 64, SWT - 63 - 64, 63 + 1, 0, 0, SWT - 1] + [37] * 200 + [64, 65, 63, 1] * 30
    for long_row in ([], [3 * SWT], [SWT + 65], [17 * SWT + 3]):
        for order in (lens + long_row, long_row + lens):
            A, x = csr_from_lengths(order, 30_000, seed=len(order), int_valued=False)
            d = to_dev_precision(A, x, kind)[:4]
            bits = run(sss.Plan(A.m, A.n, A.nnz, dtype=vt, W=W, S=S, debug=True), *d, A.m, yt)
            for bind in (True, False):
                plan = sss.Plan(A.m, A.n, A.nnz, dtype=vt, W=W, S=S, row_ptr=d[0], bind_rows=bind)
                assert torch.equal(run(plan, *d, A.m, yt), bits), bind
            for persistent in (False, True):
                ys = [torch.full((A.m,), float("nan"), dtype=yt, device="cuda") for _ in range(2)]
                sss.BatchPlan([(*d, y, A.n) for y in ys], dtype=vt, W=W, S=S, persistent=persistent).execute()
                for y in ys:
                    assert torch.equal(y.cpu(), bits), persistent
