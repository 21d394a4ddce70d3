"""Two threads ingest and convert handles of one context on their per-thread
default streams (one stream handle for both): scratch that one call freed must
not reach the other while its kernels still use it."""
import threading

import numpy as np
import pytest

import inputs
import paper_2209_06478_amd as dsm
from gpu_common import torch_dev

pytestmark = pytest.mark.gpu
PER_THREAD = 2  # hipStreamPerThread


def test_per_thread_streams():
    torch, dev = torch_dev()
    c = dsm.Context(0)
    probs = [inputs.banded(nrows=60000, seed=31), inputs.banded(nrows=60000, seed=32)]
    rng = np.random.default_rng(8)
    data = []
    for p in probs:
        perm = rng.permutation(p.col.size)
        rows = np.repeat(np.arange(p.nrows, dtype=np.int32), np.diff(p.row_ptr))
        data.append([torch.from_numpy(np.ascontiguousarray(a[perm])).to(dev) for a in (rows, p.col, p.val)])
    torch.cuda.synchronize()
    bad, done = [], []

    def work(k):
        p = probs[k]
        for rep in range(6):
            A = dsm.Matrix.from_coo(c, p.nrows, p.ncols, *data[k], sorted=False, stream=PER_THREAD)
            for fmt in ("csr", "dia", "csr") if rep % 2 else ("csr", "hyb", "csr"):
                A.convert(fmt, max_pad_ratio=1e6, stream=PER_THREAD)
            e = A.export(stream=PER_THREAD)
            if not (np.array_equal(e["row_ptr"], p.row_ptr) and np.array_equal(e["col"], p.col)
                    and np.array_equal(e["val"], p.val)):
                bad.append((k, rep))
            A.close()
        done.append(k)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    [t.start() for t in ts]
    [t.join(60) for t in ts]
    assert sorted(done) == [0, 1] and not bad, (done, bad)
    assert c.bytes_in_use() == 0
    c.close()
