"""Which CG loop a solve takes, from a trace of the kernels: the one launch
where a system fits it, steps after it has been given up, the loop of one
launch per step for systems too large or switched off."""
import pytest

from gpu_common import make_matrix, torch_dev
from test_gpu_cg_resident import _problem

pytestmark = pytest.mark.gpu


def test_routes(monkeypatch):
    torch, dev = torch_dev()
    from torch.profiler import ProfilerActivity, profile

    def route(A, b, **kw):
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            _, res = A.cg(b, tol=1e-9, **kw)
            torch.cuda.synchronize()
        assert res["status"] == "converged"
        count = {k: sum(e.count for e in prof.key_averages() if k in e.key)
                 for k in ("k_slots_clear", "k_cg_persist", "k_cgp_scalars", "k_cg_update_r")}
        return tuple(count.values()), res

    monkeypatch.setenv("DSM_CG_GRAPH", "0")
    for kind, n, fits in [("tri", 300, {"csr", "dia", "ell"}), ("hpcg", 40, {"csr", "dia", "ell"}),
                          ("hpcg", 70, {"dia", "ell"}), ("hpcg", 80, set())]:
        p = _problem(kind, n)
        b = torch.from_numpy(p.b).to(dev)
        for fmt in ("csr", "dia", "ell"):
            for mode in ("f64", "jacobi"):
                A = make_matrix(p)
                A.convert(fmt)
                A.cg(b, maxit=1)
                got, res = route(A, b, mode=mode)
                if fmt in fits:
                    assert got == (1, 1, 0, 0), (kind, n, fmt, mode, got)
                else:
                    assert got[:3] == (0, 0, 0) and got[3] >= res["iters"], (kind, n, fmt, mode, got)
                monkeypatch.setenv("DSM_CG_RESIDENT", "0")
                got, _ = route(A, b, mode=mode)
                assert got[:3] == (0, 0, 0) and got[3] > 0
                monkeypatch.delenv("DSM_CG_RESIDENT")
                if fmt in fits:
                    monkeypatch.setenv("DSM_CG_GIVE_UP", "1")
                    got, res = route(A, b, mode=mode, check_every=2)
                    assert got[0] == 2 and got[2] > 2 * (res["iters"] - 2) and got[3] == 0, got
                    monkeypatch.delenv("DSM_CG_GIVE_UP")
                    got, res = route(A, b, mode=mode)  # the next solves of the handle
                    assert got[0] == 0 and got[2] > 2 * res["iters"] and got[3] == 0, got
                A.close()
