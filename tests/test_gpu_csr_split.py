"""How a CSR matrix' row blocks are shared out (from a trace of the kernels): a
wave streams a block of a large matrix, a workgroup takes one of a small or
skewed matrix, of rows beyond 1024 entries unless there are many, and of rows
scattered over x up to 16M entries; and the streamed rows at the edges of
batches and blocks, with infinities and NaN beside them."""
import numpy as np
import pytest

import oracle
import paper_2209_06478_amd as dsm
from gpu_common import ctx, log, row_scaled_err, torch_dev
from kernel_trace import kernels
from test_gpu_csr_rows import EDGES

pytestmark = pytest.mark.gpu


def near(lens, gap=3):
    """Rows of the given lengths whose first columns lie close to each other's."""
    lens = np.asarray(lens, np.int64)
    nc = int(lens.max()) * gap + lens.size // 64 + 1
    rp = np.concatenate([[0], np.cumsum(lens)])
    k = np.arange(rp[-1]) - np.repeat(rp[:-1], lens)
    col = np.repeat(np.arange(lens.size) // 64, lens) + k * gap
    return lens.size, nc, rp.astype(np.int32), col.astype(np.int32)


def apart(n, per, jump, nc):
    """n rows of `per` columns, each row's first one `jump` columns past the one before (cyclic)."""
    base = np.arange(n, dtype=np.int64) * jump % (nc - 2 * per)
    col = base[:, None] + 2 * np.arange(per)
    return n, nc, (np.arange(n + 1) * per).astype(np.int32), col.reshape(-1).astype(np.int32)


CASES = {
    "few blocks": (lambda: near(np.full(200_000, 20)), False),
    "many blocks": (lambda: near(np.full(230_000, 20)), True),
    "few long rows": (lambda: near(np.full(9_000, 1100), 1), False),
    "many long rows": (lambda: near(np.full(16_500, 1100), 1), True),
    "rows 1000 apart": (lambda: apart(1_100_000, 5, 1000, 300_000), True),
    "rows 1100 apart": (lambda: apart(1_100_000, 5, 1100, 300_000), False),
    "rows far apart, many entries": (lambda: apart(1_100_000, 16, 99_991, 300_000), True),
    "mostly empty": (lambda: near(np.where(np.arange(1_200_000) % 50 == 0, 5, 0)), True),
}


@pytest.mark.parametrize("name", list(CASES))
def test_route(name):
    torch, dev = torch_dev()
    make, streams = CASES[name]
    nr, nc, rp, col = make()
    val = np.random.default_rng(3).standard_normal(col.size)
    x = np.random.default_rng(4).random(nc)
    yref, scale = oracle.spmv_csr_ref(rp, col, val, x)
    A = dsm.Matrix.from_csr(ctx(), nr, nc, rp, col, val)
    xt = torch.from_numpy(x).to(dev)
    y = A.spmv(xt)
    names = kernels(lambda: A.spmv(xt, out=y))
    log(f"[split] {name}: {names[:80]}")
    assert ("k_csr_stream" in names) == streams
    assert ("k_csr_adaptive" in names) != streams
    assert row_scaled_err(y.cpu().numpy(), yref, scale) <= 1e-14
    A.close()


@pytest.mark.parametrize("kind", ["edges", "empty"])
def test_streamed_rows(kind):
    """FP64 row-scaled 1e-14; bfloat16 values with FP32 vectors within (length + 2) 2^-24 of the row
    scale; y += A x equals y + A x; non-finite entries of x reach the rows that store their columns."""
    torch, dev = torch_dev()
    rng = np.random.default_rng(5)
    if kind == "edges":
        lens = rng.integers(4, 11, 720_001)
        lens[1000 + 1777 * np.arange(20 * len(EDGES))] = np.tile(EDGES, 20)
        lens[-3:] = [2500, 0, 0]
    else:
        lens = np.where(rng.random(1_200_000) < 0.02, 5, 0)
        lens[500_000:600_000] = 0
    nr, nc, rp, col = near(lens)
    val = rng.standard_normal(col.size)
    x = rng.random(nc) + 0.5
    x32 = x.astype(np.float32).astype(np.float64)
    vb = oracle.bf16_to_f64(oracle.cast_bf16(val))
    yref, scale = oracle.spmv_csr_ref(rp, col, val, x)
    yref32, scale32 = oracle.spmv_csr_ref(rp, col, vb, x32)
    tol32 = (np.diff(rp) + 2) * 2.0 ** -24 * scale32
    rows = np.repeat(np.arange(nr), np.diff(rp))
    bad = np.unique(np.concatenate([col[[0, -1]], col[rp[1:][np.diff(rp) > 0][::99_991] - 1]]))
    xb = x.copy()
    xb[bad] = np.resize([np.inf, np.nan, -np.inf], bad.size)
    hit = np.isin(col, bad)
    touched = np.zeros(nr, bool)
    touched[rows[hit]] = True
    sums = np.zeros(nr)
    with np.errstate(invalid="ignore"):
        np.add.at(sums, rows[hit], val[hit] * xb[col[hit]])
    assert touched.any() and not touched.all()
    A = dsm.Matrix.from_csr(ctx(), nr, nc, rp, col, val)
    B = dsm.Matrix.from_csr(ctx(), nr, nc, rp, col, val).convert("csr", value_dtype="bf16")
    xt, x32t, xbt = (torch.from_numpy(v).to(dev) for v in (x, x32.astype(np.float32), xb))
    for v in (0, 7, 8, 15):
        A.variant = B.variant = v
        y = A.spmv(xt)
        assert row_scaled_err(y.cpu().numpy(), yref, scale) <= 1e-14, v
        y32 = B.spmv(x32t).cpu().numpy().astype(np.float64)
        assert np.all(np.abs(y32 - yref32) <= tol32), v
        acc = torch.ones(nr, dtype=torch.float64, device=dev)
        A.spmv_accumulate(xt, acc)
        assert torch.equal(acc, 1 + y), v
        yb = A.spmv(xbt).cpu().numpy()
        assert row_scaled_err(yb[~touched], yref[~touched], scale[~touched]) <= 1e-14, v
        assert np.array_equal(yb[touched], sums[touched], equal_nan=True), v
    A.close()
    B.close()
