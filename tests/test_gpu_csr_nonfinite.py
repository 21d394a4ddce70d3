"""Infinities and NaN in x and in stored values reach exactly the rows that
store an entry there, also where a wave streams a row block (4096 row blocks and
more: batches repeat their last entry past a block's end) and where a workgroup
takes one (skewed matrices)."""
import numpy as np
import pytest

import oracle
import paper_2209_06478_amd as dsm
from gpu_common import ctx, row_scaled_err, torch_dev
from test_gpu_csr_rows import matrix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["x", "values"])
@pytest.mark.parametrize("kind", ["edges", "empty", "skewed"])
def test_nonfinite(kind, where):
    torch, dev = torch_dev()
    nr, nc, rp, col, val = matrix(kind)
    x = np.random.default_rng(7).random(nc) + 0.5
    rows = np.repeat(np.arange(nr), np.diff(rp))
    clean_x, clean_v = x.copy(), val.copy()
    if where == "x":
        # columns of the last entries of some rows (what a batch repeats) and of first ones
        bad = {int(col[rp[i + 1] - 1]): v for i, v in zip(np.flatnonzero(np.diff(rp) > 0)[::9973][:24],
                                                          8 * [np.inf, -np.inf, np.nan])}
        bad[int(col[0])] = np.nan
        for c, v in bad.items():
            x[c], clean_x[c] = v, 0.0
        hit = np.isin(col, list(bad))
    else:
        at = np.concatenate([[0, val.size - 1], np.arange(3, val.size, val.size // 40)])
        val[at] = np.resize([np.inf, np.nan, -np.inf], at.size)
        clean_v[at] = 0.0
        hit = np.zeros(val.size, bool)
        hit[at] = True
    touched = np.zeros(nr, bool)
    touched[rows[hit]] = True
    assert touched.any() and not touched.all()
    yref, scale = oracle.spmv_csr_ref(rp, col, clean_v, clean_x)
    with np.errstate(invalid="ignore"):
        prod = val[hit] * x[col[hit]]
        sums = np.zeros(nr)
        np.add.at(sums, rows[hit], np.where(np.isfinite(prod), 0.0, prod))  # +-inf or NaN per touched row
    A = dsm.Matrix.from_csr(ctx(), nr, nc, rp, col, val)
    xt = torch.from_numpy(x).to(dev)
    for v in (0, 7, 8, 15):
        A.variant = v
        y = A.spmv(xt).cpu().numpy()
        assert np.all(np.isfinite(y[~touched])), v
        assert row_scaled_err(y[~touched], yref[~touched], scale[~touched]) <= 1e-14, v
        assert np.array_equal(y[touched], sums[touched], equal_nan=True), v
    A.close()
