"""The names of the kernels that a piece of a test launches, from torch's trace
of the device (it sees every kernel of the process)."""
import pytest


def kernels(work, repeats=4):
    """Runs work() `repeats` times (a trace may lack some of the launches) and
    returns the names of the kernels seen, in one string; skips the test where
    no trace can be taken."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        for _ in range(repeats):
            work()
        torch.cuda.synchronize()
    names = " ".join(e.key for e in prof.key_averages())
    if not names:
        pytest.skip("the profiler recorded no kernels")
    return names
