"""The least HBM budget a call fits in: the matrices, the documented vectors
and partial sums, and no more.  Buffers that only make a call faster are done
without when the budget has no room for them, with results as close."""
import numpy as np
import pytest

import inputs
import oracle
import paper_2209_06478_amd as dsm
from gpu_common import torch_dev

pytestmark = pytest.mark.gpu


def r256(b):
    return (b + 255) // 256 * 256


def payload_bytes(p, fmt, vdt="f64", **kw):
    c = dsm.Context(0)
    A = dsm.Matrix.from_csr(c, p.nrows, p.ncols, p.row_ptr, p.col, p.val)
    csr = c.bytes_in_use()
    A.convert(fmt, value_dtype=vdt, **kw)
    n = c.bytes_in_use()
    A.close()
    c.close()
    return csr, n


@pytest.mark.parametrize("n", [1, 40, 300, 70001])
def test_cg_workspace(n):
    """Six FP64 vectors, three sets of partial sums and 2 KiB."""
    torch, dev = torch_dev()
    p = inputs.banded_spd(n, 3, seed=n)
    csr, _ = payload_bytes(p, "csr")
    b = torch.from_numpy(p.b).to(dev)
    need = 6 * r256(8 * n) + 3 * r256(8 * max(n // 256 + 2, 512)) + 8 * 256
    c = dsm.Context(0, hbm_budget=csr + need)
    A = dsm.Matrix.from_csr(c, p.nrows, p.ncols, p.row_ptr, p.col, p.val)
    for rep in range(2):
        x, res = A.cg(b, tol=1e-10)
        assert res["status"] == "converged"
        assert oracle.true_relres(p.row_ptr, p.col, p.val, p.b, x.cpu().numpy()) <= 1.5e-10
    assert c.bytes_in_use() == csr + need
    A.close()
    c.close()
