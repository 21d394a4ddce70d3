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


def test_batch_arena():
    """Three FP64 vectors a system, 184 bytes for its descriptor and result, 1536 for the batch: systems
    whose vectors lie in LDS and in memory (beyond 8000 rows in CSR, 19000 in DIA and ELL)."""
    torch, dev = torch_dev()
    # (the conversions first: they need room for both formats)
    probs = [(inputs.banded_spd(n, 4, seed=n), f) for n, f in
             [(32000, "dia"), (20480, "ell"), (1024, "dia"), (96, "ell"), (9984, "csr"), (7936, "csr"), (1, "csr")]]

    def solve(budget):
        c = dsm.Context(0, hbm_budget=budget)
        mats = [dsm.Matrix.from_csr(c, p.nrows, p.ncols, p.row_ptr, p.col, p.val).convert(f) for p, f in probs]
        held = c.bytes_in_use()
        xs = [torch.zeros(p.nrows, dtype=torch.float64, device=dev) for p, _ in probs]
        res = dsm.cg_batched(mats, [torch.from_numpy(p.b).to(dev) for p, _ in probs], xs, tol=1e-9)
        for A in mats:
            A.close()
        c.close()
        return held, xs, res

    held, xs, res = solve(0)
    for (p, f), x, r in zip(probs, xs, res):
        assert r["status"] == "converged"
        assert oracle.true_relres(p.row_ptr, p.col, p.val, p.b, x.cpu().numpy()) <= 1.5e-9
    need = 1536 + sum(3 * r256(8 * p.nrows) + 184 for p, _ in probs)
    _, ys, qs = solve(held + need)
    assert qs == res and all(torch.equal(x, y) for x, y in zip(xs, ys))


@pytest.mark.parametrize("name", ["zipf", "spd"])
def test_creation_and_hyb(name):
    """A matrix fits in its row pointers, entries and row blocks, with its flags and their prefix sums
    during creation; HYB holds its ELL slots and overflow entries only.  Products are as close without the
    overflow's row groups."""
    torch, dev = torch_dev()
    p = inputs.zipf(nrows=50000, seed=5) if name == "zipf" else inputs.banded_spd(20000, 5, seed=1)
    n, nnz = p.nrows, p.col.size
    csr, hyb = payload_bytes(p, "hyb")
    c = dsm.Context(0, hbm_budget=csr + 4 * (2 * n + 1) + 16 * (2 * (n // 4096 + 1) + 1))
    A = dsm.Matrix.from_csr(c, p.nrows, p.ncols, p.row_ptr, p.col, p.val)
    assert c.bytes_in_use() == csr
    A.close()
    c.close()
    c = dsm.Context(0, hbm_budget=1 << 30)
    A = dsm.Matrix.from_csr(c, p.nrows, p.ncols, p.row_ptr, p.col, p.val)
    A.convert("hyb")
    i = A.info()
    slots = i["ell_width"] * i["pitch"]
    assert c.bytes_in_use() == i["bytes"] == max(4 * slots, 16) + max(8 * slots, 16) + 2 * max(4 * i["coo_nnz"], 16) + max(
        8 * i["coo_nnz"], 16)
    x = np.cos(np.arange(p.ncols))
    yref, scale = oracle.spmv_csr_ref(p.row_ptr, p.col, p.val, x)
    y = A.spmv(torch.from_numpy(x).to(dev)).cpu().numpy()
    assert np.max(np.abs(y - yref) / np.maximum(scale, 1e-300)) <= 1e-14
    A.close()
    c.close()


@pytest.mark.parametrize("fmt", ["csr", "dia"])
def test_hierarchy(fmt):
    """What a hierarchy holds: per level the rows by colour, the colours' starts and the diagonal (and, DIA,
    the other offsets, the diagonals by colour and the records of the LDS sweep); r and x of the coarser
    levels; five vectors, partial sums and the state of the solve.  Level 0 (110,592 rows) would be parted
    without a budget."""
    from test_gpu_mg import oracle_levels
    torch, dev = torch_dev()
    L = inputs.hpcg27_levels(48, 3)
    ns = [lv["problem"].nrows for lv in L]

    def hierarchy(budget):
        c = dsm.Context(0, hbm_budget=budget)
        mats = []
        for lv in L:
            p = lv["problem"]
            A = dsm.Matrix.from_csr(c, p.nrows, p.ncols, p.row_ptr, p.col, p.val)
            mats.append(A.convert(fmt) if fmt != "csr" else A)
        held = c.bytes_in_use()
        mg = dsm.Multigrid(c, mats, [lv["f2c"] for lv in L[:-1]], [lv["colour"] for lv in L])
        return c, mats, mg, held

    c, mats, mg, held = hierarchy(0)
    p = L[0]["problem"]
    b = torch.from_numpy(p.b).to(dev)
    _, want = mg.pcg(b, tol=1e-9)
    mg.close()
    [A.close() for A in mats]
    c.close()
    need = 0
    for l, (lv, n) in enumerate(zip(L, ns)):
        nc = int(lv["colour"].max()) + 1
        need += 4 * n + 8 * (nc + 1) + 8 * n
        if fmt == "dia":
            need += 4 * 26 + 8 * 27 * ((n + 63) // 64 * 64)
            if np.bincount(lv["colour"]).max() <= 512 and n <= 8192:
                need += 8 * n * 28
        need += 16 * n if l else 0
        need += 4 * ns[l + 1] if l + 1 < len(L) else 0
    need += 5 * 8 * ns[0] + 3 * 8 * max(ns[0] // 256 + 2, 512) + 72
    # (converting to DIA needs room for both formats, more than the hierarchy does)
    c, mats, mg, h = hierarchy(held + need if fmt == "csr" else 1 << 30)
    assert h == held and c.bytes_in_use() == held + need
    z = mg.apply(b)
    zr = oracle.mg(oracle_levels(L), p.b)
    assert np.max(np.abs(z.cpu().numpy() - zr)) <= 1e-12 * np.max(np.abs(zr))
    _, res = mg.pcg(b, tol=1e-9)
    assert res["status"] == want["status"] == "converged" and abs(res["iters"] - want["iters"]) <= 1
    mg.close()
    [A.close() for A in mats]
    c.close()
