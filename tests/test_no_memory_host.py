"""No C++ exception crosses the C ABI where the host runs out of memory while a
plane is made: libwcsim's allocations fail from the k-th on, for every k, on a
host without a GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_plane_creation_without_host_memory(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    from paper_2304_01841_amd import wcsim
    exe = str(tmp_path / "no_memory")
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-g", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                           os.path.join(HERE, "no_memory_driver.cpp"), wcsim.LIB_PATH, "-ldl",
                           "-Wl,-rpath," + os.path.dirname(wcsim.LIB_PATH),
                           "-Wl,-rpath-link,/opt/rocm/lib", "-o", exe])
    env = dict(os.environ, LD_LIBRARY_PATH="/opt/rocm/lib:" + os.environ.get("LD_LIBRARY_PATH", ""),
               HIP_VISIBLE_DEVICES="-1")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "without memory ok" in r.stdout
