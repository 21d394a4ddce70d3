"""Matrices whose one-thread-per-slot or several-threads-per-row kernels need
more threads than one launch can count."""
import pytest

import paper_2209_06478_amd as dsm
from gpu_common import ctx, log, torch_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _give_memory_back():
    yield
    torch_dev()[0].cuda.empty_cache()


def _sparse(n, rows, per, val, torch, dev):
    counts = torch.zeros(n + 1, dtype=torch.int32, device=dev)
    counts[rows + 1] = per
    rp = torch.cumsum(counts, 0, dtype=torch.int32)
    col = torch.arange(per, dtype=torch.int32, device=dev).repeat(rows.numel())
    return dsm.Matrix.from_csr(ctx(), n, per, rp, col, val)


@pytest.mark.parametrize("lanes_log", [5, 6])
def test_csr_vector_kernels(lanes_log):
    """2^28 rows of 32 and 64 lanes: 2^33 and 2^34 threads."""
    torch, dev = torch_dev()
    n = 2 ** 28 + 7
    rows = torch.cat([torch.arange(0, n - 100, 10 ** 6 + 1, device=dev), torch.arange(n - 50, n, device=dev)])
    val = torch.arange(1, 3 * rows.numel() + 1, dtype=torch.float64, device=dev)
    A = _sparse(n, rows, 3, val, torch, dev)
    A.variant = lanes_log
    x = torch.tensor([1.0, 2.0, 4.0], dtype=torch.float32, device=dev)
    y = torch.full((n,), -1.0, dtype=torch.float32, device=dev)
    log(f"[large] vector kernel, {1 << lanes_log} lanes, {n} rows")
    A.spmv(x, out=y)
    assert torch.equal(y[rows], (val.view(-1, 3) * x).sum(1).float())
    assert int(torch.count_nonzero(y)) == rows.numel()
    A.close()


def test_values_exact_looks_at_every_slot():
    """5.4e9 ELL slots, the last ones of which hold a value that FP32 does not."""
    torch, dev = torch_dev()
    n = 2 ** 30 + 1000
    rows = torch.tensor([5, n - 1], device=dev)
    val = torch.ones(10, dtype=torch.float64, device=dev)
    for last, exact in ((1.0, True), (0.1, False)):
        val[9] = last
        A = _sparse(n, rows, 5, val, torch, dev)
        A.convert("ell", max_pad_ratio=1e10)
        log(f"[large] {A.info()['bytes']} bytes")
        assert A.values_exact("f32") == exact
        A.close()
