"""Conversions of matrices with more rows than a launch of several threads a
row could cover at once."""
import pytest

import paper_2209_06478_amd as dsm
from gpu_common import ctx, log, torch_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _give_memory_back():
    yield
    torch_dev()[0].cuda.empty_cache()


@pytest.mark.parametrize("fmt", ["dia", "ell", "hdc"])
def test_more_than_2_30_rows(fmt):
    torch, dev = torch_dev()
    n = 2 ** 30 + 1000
    rows = torch.cat([torch.arange(0, 40, device=dev), torch.arange(63, n - 200, 10 ** 7 + 1, device=dev),
                      torch.arange(n - 100, n, device=dev)])
    cols = torch.stack([rows, (rows + 3) % n], 1)
    cols = torch.where(rows.view(-1, 1) + 3 < n, cols, torch.sort(cols, 1).values)
    counts = torch.zeros(n + 1, dtype=torch.int32, device=dev)
    counts[rows + 1] = 2
    rp = torch.cumsum(counts, 0, dtype=torch.int32)
    del counts
    val = torch.arange(1, 2 * rows.numel() + 1, dtype=torch.float64, device=dev)
    A = dsm.Matrix.from_csr(ctx(), n, n, rp, cols.reshape(-1).to(torch.int32), val)
    del rp
    x = torch.ones(n, dtype=torch.float32, device=dev)
    y = torch.empty(n, dtype=torch.float32, device=dev)
    want = val.view(-1, 2).sum(1).float()
    for f in (fmt, "csr"):
        A.convert(f, max_pad_ratio=1e9)
        log(f"[limits] {n} rows, {f}: {A.info()['bytes']} bytes")
        y.fill_(-1.0)
        A.spmv(x, out=y)
        assert torch.equal(y[rows], want), f
        assert int(torch.count_nonzero(y)) == rows.numel(), f
    A.close()
