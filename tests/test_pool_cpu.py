"""When a context hands a kept device block out without waiting for the work
queued before it was freed (pure bookkeeping), built with g++ under
AddressSanitizer and UndefinedBehaviorSanitizer: known streams, the per-thread
default stream (one handle for many streams), unknown ones, device-wide waits."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_kept_blocks(tmp_path):
    exe = tmp_path / "pool_driver"
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-Wall", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-o", str(exe), os.path.join(ROOT, "tests", "c", "pool_driver.cpp")]
    subprocess.check_call(cmd)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout[-4000:] + r.stderr[-4000:]
    assert "pool driver ok" in r.stdout
