"""Which CG loop a solve takes, from a trace of the kernels: the one launch
where a system fits it, steps after it has been given up, the loop of one
launch per step for systems too large or switched off."""
import pytest

from gpu_common import make_matrix, torch_dev
from kernel_trace import kernels
from test_gpu_cg_resident import _problem

pytestmark = pytest.mark.gpu


def test_routes(monkeypatch):
    torch, dev = torch_dev()

    def route(A, b, **kw):
        """Which of the kernels ran."""
        def solve():
            assert A.cg(b, tol=1e-9, **kw)[1]["status"] == "converged"
        names = kernels(solve)
        return tuple(k in names for k in ("k_slots_clear", "k_cg_persist", "k_cgp_scalars", "k_cg_update_r"))

    monkeypatch.setenv("DSM_CG_GRAPH", "0")
    for kind, n, fits in [("tri", 300, {"csr", "dia", "ell"}), ("hpcg", 40, {"csr", "dia", "ell"}),
                          ("hpcg", 70, {"dia", "ell"}), ("hpcg", 80, set())]:
        p = _problem(kind, n)
        b = torch.from_numpy(p.b).to(dev)
        for fmt in ("csr", "dia", "ell"):
            for mode in ("f64", "jacobi"):
                A = make_matrix(p)
                A.convert(fmt)
                one = (True, True, False, False) if fmt in fits else (False, False, False, True)
                assert route(A, b, mode=mode) == one, (kind, n, fmt, mode)
                monkeypatch.setenv("DSM_CG_RESIDENT", "0")
                assert route(A, b, mode=mode) == (False, False, False, True), (kind, n, fmt, mode)
                monkeypatch.delenv("DSM_CG_RESIDENT")
                if fmt in fits:  # a launch that is given up, then the next solves of the handle
                    monkeypatch.setenv("DSM_CG_GIVE_UP", "1")
                    assert route(A, b, mode=mode, check_every=2) == (True, True, True, False), (kind, n, fmt, mode)
                    monkeypatch.delenv("DSM_CG_GIVE_UP")
                    assert route(A, b, mode=mode) == (False, True, True, False), (kind, n, fmt, mode)
                A.close()
