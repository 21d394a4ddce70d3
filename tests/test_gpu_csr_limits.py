"""Row-block CSR products at the ends of the index range: entry and row counts
within a batch of 2^31."""
import pytest

import paper_2209_06478_amd as dsm
from gpu_common import ctx, log, torch_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _give_memory_back():
    yield
    torch_dev()[0].cuda.empty_cache()


TOP = 2 ** 31 - 2  # the largest count a matrix may have


@pytest.mark.parametrize("nnz", [TOP, TOP - 383])
def test_entries_up_to_the_limit(nnz):
    """Rows of 120 entries, the last one short: sums of small whole numbers, exact in FP32."""
    torch, dev = torch_dev()
    per, nc = 120, 1 << 20
    n = (nnz + per - 1) // per
    rp = torch.clamp(torch.arange(n + 1, dtype=torch.int64, device=dev) * per, max=nnz).to(torch.int32)
    col = torch.empty(n * per, dtype=torch.int32, device=dev)
    torch.add((torch.arange(n, dtype=torch.int32, device=dev) % 4096 * 250).view(-1, 1),
              torch.arange(per, dtype=torch.int32, device=dev), out=col.view(n, per))
    val = torch.ones(nnz, dtype=torch.float64, device=dev)
    A = dsm.Matrix.from_csr(ctx(), n, nc, rp, col[:nnz], val)
    del val, col
    x = torch.ones(nc, dtype=torch.float32, device=dev)
    want = (rp[1:] - rp[:-1]).to(torch.float32)
    for v in (0, 8):
        A.variant = v
        log(f"[limits] {nnz} entries, variant {v}")
        assert torch.equal(A.spmv(x), want)
    A.close()


def test_rows_up_to_the_limit():
    """Empty rows but for a few, the last ones among them."""
    torch, dev = torch_dev()
    rows = torch.tensor([0, 1, 255, 256, 10 ** 9, TOP - 65, TOP - 64, TOP - 63, TOP - 2, TOP - 1], device=dev)
    counts = torch.zeros(TOP + 1, dtype=torch.int32, device=dev)
    counts[rows + 1] = 3
    rp = torch.cumsum(counts, 0, dtype=torch.int32)
    del counts
    nnz = 3 * rows.numel()
    col = torch.arange(3, dtype=torch.int32, device=dev).repeat(rows.numel())
    val = torch.arange(1, nnz + 1, dtype=torch.float64, device=dev)
    A = dsm.Matrix.from_csr(ctx(), TOP, 3, rp, col, val)
    del rp
    x = torch.tensor([1.0, 2.0, 4.0], dtype=torch.float32, device=dev)
    y = torch.full((TOP,), -1.0, dtype=torch.float32, device=dev)
    for v in (0, 7):
        A.variant = v
        log(f"[limits] {TOP} rows, variant {v}")
        y.fill_(-1.0)
        A.spmv(x, out=y)
        assert torch.equal(y[rows], (val.view(-1, 3) * x).sum(1).float())
        assert int(torch.count_nonzero(y)) == rows.numel()
    A.close()
