"""Batched CG at the sizes where the threads of a launch change (64, 128, 256,
512 and 1024 rows): a system's result has the same bits alone, among systems of
its size and in a batch with a larger one, and meets the oracle."""
import pytest

import inputs
import oracle
import paper_2209_06478_amd as dsm
from gpu_common import ctx, log, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["csr", "dia", "ell"])
def test_batched_sizes(fmt):
    torch, dev = torch_dev()
    sizes = [1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2049]
    probs = [inputs.banded_spd(n, min(9, max(n - 1, 1)), seed=100 + n) for n in sizes]
    mats = [dsm.Matrix.from_csr(ctx(), p.nrows, p.ncols, p.row_ptr, p.col, p.val).convert(fmt, max_pad_ratio=1e3)
            for p in probs]
    bs = [torch.from_numpy(p.b).to(dev) for p in probs]

    def solve(ks):
        xs = [torch.zeros(probs[k].nrows, dtype=torch.float64, device=dev) for k in ks]
        res = dsm.cg_batched([mats[k] for k in ks], [bs[k] for k in ks], xs, tol=1e-9)
        return dict(zip(ks, zip(xs, res)))

    alone = {k: solve([k])[k] for k in range(len(sizes))}
    for k, (x, r) in alone.items():
        p = probs[k]
        log(f"[sizes] {fmt} {sizes[k]}: {r['iters']} iterations")
        _, it, _, _ = oracle.cg(p.row_ptr, p.col, p.val, p.b, tol=1e-9)
        assert r["status"] == "converged" and abs(r["iters"] - it) <= 1
        assert oracle.true_relres(p.row_ptr, p.col, p.val, p.b, x.cpu().numpy()) <= 1.5e-9
    # every prefix of the sizes is a batch of the launch its largest system takes
    for end in range(1, len(sizes) + 1):
        for k, (x, r) in solve(list(range(end))).items():
            assert torch.equal(x, alone[k][0]) and r == alone[k][1], (sizes[k], sizes[end - 1])
    for A in mats:
        A.close()
