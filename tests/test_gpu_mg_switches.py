"""DSM_MG_ND=0 takes the runtime-length colour sweep (seen in a trace of the
kernels) on levels of every kind, parted ones among them, with the same bits."""
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.gpu

PROGRAM = """
import sys
import numpy as np
sys.path[:0] = [{root!r}, {tests!r}]
import inputs
from gpu_common import torch_dev
from kernel_trace import kernels
from test_gpu_mg import build
from test_gpu_mg_parted import levels
torch, dev = torch_dev()
L = levels({kind!r})
mg, mats = build(L, "dia")
n = L[0]["problem"].nrows
r = torch.from_numpy(inputs.uniform_vector(n, seed=41) - 0.5).to(dev)
x = torch.from_numpy(inputs.uniform_vector(n, seed=42)).to(dev)
mg.symgs(0, r, x)
z = mg.apply(r)
names = kernels(lambda: mg.apply(r))
np.savez({out!r}, x=x.cpu().numpy(), z=z.cpu().numpy(), lists="k_symgs_list" in names, runtime="k_symgs_dia<" in names)
"""


@pytest.mark.parametrize("kind", ["lattice", "seven", "mixed"])
def test_runtime_length_sweep(kind, tmp_path):
    got = {}
    for nd in ("1", "0"):
        out = str(tmp_path / f"nd{nd}.npz")
        code = PROGRAM.format(root=ROOT, tests=os.path.join(ROOT, "tests"), kind=kind, out=out)
        r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, DSM_MG_ND=nd), capture_output=True,
                           text=True, timeout=100)
        if "Skipped" in r.stderr:
            pytest.skip("the profiler recorded no kernels")
        assert r.returncode == 0, r.stderr[-3000:]
        got[nd] = np.load(out)
        assert bool(got[nd]["lists"]) == (nd == "1") and bool(got[nd]["runtime"]) == (nd == "0")
    for k in ("x", "z"):
        assert np.array_equal(got["0"][k].view(np.uint64), got["1"][k].view(np.uint64)), k
