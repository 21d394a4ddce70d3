"""Smoother sweeps of one hierarchy that run at the same time on two streams,
with vectors of their own, beside each other and beside a V-cycle: each has the
bits it has alone (a sweep by itself uses nothing of the hierarchy but its
values)."""
import pytest

import inputs
from gpu_common import torch_dev
from test_gpu_mg import build
from test_gpu_mg_parted import levels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("beside", ["sweep", "cycle"])
@pytest.mark.parametrize("kind", ["lattice", "seven"])
def test_sweeps_side_by_side(kind, beside):
    torch, dev = torch_dev()
    L = levels(kind)
    mg, mats = build(L, "dia")
    n = L[0]["problem"].nrows
    r = [torch.from_numpy(inputs.uniform_vector(n, seed=50 + k) - 0.5).to(dev) for k in range(2)]
    x0 = [torch.from_numpy(inputs.uniform_vector(n, seed=60 + k)).to(dev) for k in range(2)]
    reps = 12
    want = []
    for k in range(2):
        x = x0[k].clone()
        for _ in range(reps):
            mg.symgs(0, r[k], x)
        want.append(x)
    zwant = mg.apply(r[1])
    torch.cuda.synchronize()
    st = [torch.cuda.Stream(), torch.cuda.Stream()]
    for _ in range(4):
        x = [v.clone() for v in x0]
        z = torch.empty_like(x[1])
        torch.cuda.synchronize()
        for _ in range(reps):
            with torch.cuda.stream(st[0]):
                mg.symgs(0, r[0], x[0])
            with torch.cuda.stream(st[1]):
                if beside == "sweep":
                    mg.symgs(0, r[1], x[1])
                else:
                    mg.apply(r[1], out=z)
        torch.cuda.synchronize()
        assert torch.equal(x[0], want[0])
        assert torch.equal(x[1], want[1]) if beside == "sweep" else torch.equal(z, zwant)
    mg.close()
    for A in mats:
        A.close()
