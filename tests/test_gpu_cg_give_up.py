"""The one-launch CG loop: which systems take it (its sums run in another order
than those of the loop of one launch per step, so the bits tell them apart),
and launches that are given up, at the start of a solve and in the middle: the
solve goes on by steps with the bits it has otherwise, and so do the solves
after it."""
import numpy as np
import pytest

from gpu_common import log, make_matrix, torch_dev
from test_gpu_cg_resident import _problem

pytestmark = pytest.mark.gpu


def _bits(x):
    return x.cpu().numpy().view(np.uint64)


# far: 12000 rows whose columns reach across the matrix do not fit
@pytest.mark.parametrize("kind,n,fits", [("tri", 63, True), ("tri", 65537, True), ("spd", 1000, True), ("hpcg", 40, True),
                                         ("far", 12000, False), ("hpcg", 80, False)])
def test_which_loop(kind, n, fits, monkeypatch):
    torch, dev = torch_dev()
    p = _problem(kind, n)
    b = torch.from_numpy(p.b + 0.25 * (np.arange(p.nrows) % 5)).to(dev)
    A = make_matrix(p)
    for fmt in ("csr", "dia", "ell"):
        if kind == "far" and fmt == "dia":
            continue
        A.convert(fmt, max_pad_ratio=1e4)
        for mode in ("f64", "jacobi"):
            monkeypatch.setenv("DSM_CG_RESIDENT", "0")
            x0 = _bits(A.cg(b, tol=1e-10, mode=mode)[0])
            monkeypatch.delenv("DSM_CG_RESIDENT")
            x1 = _bits(A.cg(b, tol=1e-10, mode=mode)[0])
            log(f"[which] {kind} {n} {fmt} {mode}: {int((x0 != x1).sum())} entries differ")
            assert np.array_equal(x0, x1) != fits, (fmt, mode)
    A.close()


@pytest.mark.parametrize("mode,vdt", [("f64", "f64"), ("jacobi", "f64"), ("f64", "f32"), ("jacobi", "bf16"),
                                      ("ir", "f32"), ("ir_cont", "bf16")])
@pytest.mark.parametrize("kind,n", [("tri", 200), ("tri", 70001), ("hpcg", 24)])
def test_given_up(kind, n, mode, vdt, monkeypatch):
    torch, dev = torch_dev()
    p = _problem(kind, n)
    b = torch.from_numpy(p.b + 0.25 * (np.arange(p.nrows) % 5)).to(dev)
    x0 = torch.from_numpy(0.5 * np.cos(np.arange(p.nrows))).to(dev)
    for fmt in ("csr", "dia", "ell"):
        for start in ("zero", "x0"):
            def solve(A, **kw):
                x = None if start == "zero" else x0.clone()
                x, res = A.cg(b, x=x, tol=1e-11, mode=mode, **kw)
                assert res["status"] == "converged"
                return _bits(x), res
            A = make_matrix(p)
            A.convert(fmt, value_dtype=vdt)
            monkeypatch.delenv("DSM_CG_GIVE_UP", raising=False)
            want, res = solve(A)
            for launch in (0, 1, 2, 3):
                log(f"[give up] {kind} {n} {mode} {vdt} {fmt} {start}: launch {launch}")
                B = make_matrix(p)  # (a handle that has not given up before)
                B.convert(fmt, value_dtype=vdt)
                monkeypatch.setenv("DSM_CG_GIVE_UP", str(launch))
                for kw in ({"check_every": 3}, {}, {"check_every": 1}):  # (the later two go by steps as a whole)
                    x, r = solve(B, **kw)
                    assert r == res, (fmt, launch, kw)
                    assert np.array_equal(x, want), (fmt, launch, kw)
                B.close()
            A.close()


def test_given_up_limit_breakdown_and_nonfinite(monkeypatch):
    torch, dev = torch_dev()
    p = _problem("tri", 700)
    bad = p.b.copy()
    bad[333] = np.nan
    cases = [dict(b=p.b, tol=0.0, maxit=7), dict(b=bad), dict(b=0 * p.b)]
    for d in (1.0, -1.0):
        def solves():
            A = make_matrix(p)
            A.set_diagonal(torch.full((700,), 2.5 * d, dtype=torch.float64, device=dev))
            out = []
            for c in cases:
                kw = {k: v for k, v in c.items() if k != "b"}
                x, r = A.cg(torch.from_numpy(c["b"]).to(dev), **kw)
                out.append((_bits(x), r))
            A.close()
            return out
        monkeypatch.delenv("DSM_CG_GIVE_UP", raising=False)
        want = solves()
        monkeypatch.setenv("DSM_CG_GIVE_UP", "0")
        for (x, r), (y, q) in zip(solves(), want):
            assert np.array_equal(x, y) and repr(r) == repr(q)
