"""Which kernel multigrid PCG multiplies with (from a trace of the kernels): the
LDS-staged DIA sweep by itself, the caller's where a variant has been set."""
import re

import pytest

import inputs
from gpu_common import torch_dev
from kernel_trace import kernels
from test_gpu_mg import build

pytestmark = pytest.mark.gpu


def test_product_kernel(monkeypatch):
    torch, dev = torch_dev()
    monkeypatch.setenv("DSM_CG_GRAPH", "0")  # the loop's kernels one by one
    L = inputs.hpcg27_levels(24, 2)
    mg, mats = build(L, "dia")
    b = torch.from_numpy(L[0]["problem"].b).to(dev)

    def product():
        # with the dot of the loop (the true residual's product, without it, keeps the matrix' variant)
        names = kernels(lambda: mg.pcg(b, tol=1e-8))
        assert "k_pmg_update_p" in names, names
        return tuple(re.search(k + r"<double, double, (false|true), (false|true), \d, (false|true), true", names) is not None
                     for k in ("k_dia_lds", "k_dia"))

    assert product() == (True, False)
    for v, lds in [(0, False), (16, True), (4, False), (22, True)]:
        mats[0].variant = v
        assert product() == (lds, not lds), v
    mg.close()
    [A.close() for A in mats]
