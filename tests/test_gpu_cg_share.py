"""A one-launch CG solve whose stream is still busy with earlier work does not
keep a solve of another thread from the device meanwhile."""
import threading
import time

import pytest

import inputs
import paper_2209_06478_amd as dsm
from gpu_common import log, torch_dev

pytestmark = pytest.mark.gpu


def test_a_busy_stream_holds_no_share():
    torch, dev = torch_dev()
    p = inputs.hpcg27(40)  # 250 workgroups
    c = [dsm.Context(0) for _ in range(2)]
    A = [dsm.Matrix.from_csr(k, p.nrows, p.ncols, p.row_ptr, p.col, p.val) for k in c]
    b = torch.from_numpy(p.b).to(dev)
    for M in A:
        assert M.cg(b)[1]["status"] == "converged"
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    cycles = 100_000_000  # one wave that counts; about 0.05 s at 2 GHz and 1 s at 100 MHz
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    torch.cuda._sleep(cycles)
    torch.cuda.synchronize()
    reps = max(1, round(1.0 / (time.perf_counter() - t0)))
    done, waiting = {}, threading.Event()

    def solve(k):
        with torch.cuda.stream(streams[k]):
            if k == 0:
                for _ in range(reps):
                    torch.cuda._sleep(cycles)
                waiting.set()
            res = A[k].cg(b)[1]
            done[k] = time.perf_counter(), res["status"]

    ts = [threading.Thread(target=solve, args=(k,)) for k in range(2)]
    ts[0].start()
    waiting.wait(30)
    time.sleep(0.05)  # the first solve is under way, behind its stream's work
    t0 = time.perf_counter()
    ts[1].start()
    [t.join(60) for t in ts]
    took = [done[k][0] - t0 for k in range(2)]
    log(f"[share] behind a busy stream {took[0]:.3f} s, beside it {took[1]:.3f} s")
    assert done[0][1] == done[1][1] == "converged"
    assert took[1] < 0.5 * took[0]
    for M in A:
        M.close()
    [k.close() for k in c]
