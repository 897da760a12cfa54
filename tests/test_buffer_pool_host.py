"""The pool of idle device buffers on the host (no GPU), over a memory of a given
size with injected failures: what is handed out again, the bounds on number and
bytes, release and retry when memory is out, buffers given back before the device
is idle, several threads; nothing leaks and nothing is freed twice."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2304_01841_amd", "csrc")


def test_pool_over_an_injected_memory(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "pool")
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-g", "-pthread", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all", "-I", CSRC,
                           os.path.join(HERE, "buffer_pool_driver.cpp"), "-o", exe])
    env = dict(os.environ, ASAN_OPTIONS="verify_asan_link_order=0")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "buffer pool ok" in r.stdout
