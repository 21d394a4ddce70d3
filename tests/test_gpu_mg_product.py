"""Which kernel multigrid PCG multiplies with (from a trace of the kernels): the
LDS-staged DIA sweep by itself, the caller's where a variant has been set."""
import pytest

import inputs
from gpu_common import torch_dev
from test_gpu_mg import build

pytestmark = pytest.mark.gpu


def test_product_kernel(monkeypatch):
    torch, dev = torch_dev()
    from torch.profiler import ProfilerActivity, profile
    monkeypatch.setenv("DSM_CG_GRAPH", "0")  # the loop's kernels one by one
    L = inputs.hpcg27_levels(24, 2)
    mg, mats = build(L, "dia")
    b = torch.from_numpy(L[0]["problem"].b).to(dev)

    def kernels():
        mg.pcg(b, tol=1e-8)
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            _, res = mg.pcg(b, tol=1e-8)
            torch.cuda.synchronize()
        assert res["status"] == "converged"
        # (the true residual at the end is one product with the variant as it is)
        names = [e.key for e in prof.key_averages() if e.count > 2]
        assert any("k_pmg_update_p" in k for k in names), names
        return any("k_dia_lds<" in k for k in names), any("k_dia<" in k for k in names)

    assert kernels() == (True, False)
    for v, lds in [(0, False), (16, True), (4, False), (22, True)]:
        mats[0].variant = v
        assert kernels() == (lds, not lds), v
    mg.close()
    [A.close() for A in mats]
