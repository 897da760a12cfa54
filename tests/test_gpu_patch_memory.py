"""What the library holds of a device after patch sets are destroyed: at most 256
MiB over all planes, handed from plane to plane, and nothing once they are gone.
In a process of its own, where no other test's planes keep the device's pool."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.gpu


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def check():
    from paper_2304_01841_amd import wcsim
    from paper_2304_01841_amd import workloads as W
    phys = W.physics(False)
    phys["nsigma"] = 5.0
    R = W.response("unipolar", Rp=21, Rt=40, r0=10)
    dep = torch.from_numpy(W.uniform_depos(np.random.default_rng(1), 100_000, (0.0, 500.0),
                                           (0.0, 500.0), max_drift_time=2000.0)).cuda()
    planes = [wcsim.Plane(W.plane(100, 1000, plane_id=k), phys, R, r0=10) for k in range(6)]
    sets = [wcsim.rasterize(planes[0], dep, 1)]  # (every kernel is loaded)
    nbytes = 4 * sets[0].nvalues
    assert 100 << 20 < nbytes < 250 << 20
    sets.pop().destroy()
    before = _free()
    sets = [wcsim.rasterize(P, dep, 1) for P in planes]
    print("set of %.0f MiB, %d of them" % (nbytes / 2**20, len(sets)), flush=True)
    assert before - _free() >= 5 * nbytes
    for pt in sets:
        pt.destroy()
    held = before - _free()
    print("held when all are destroyed: %.0f MiB more" % (held / 2**20), flush=True)
    assert held <= 256 << 20
    # the next plane's set takes what another's left
    quiet = _free()
    pt = wcsim.rasterize(planes[3], dep, 2)
    assert quiet - _free() < nbytes
    pt.destroy()
    for P in planes[:-1]:
        P.destroy()
    last = wcsim.rasterize(planes[-1], dep, 3)
    planes[-1].destroy()
    with_set = _free()
    last.destroy()
    assert _free() - with_set >= nbytes
    print("memory ok", flush=True)


def test_idle_memory_is_bounded_over_planes():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    r = subprocess.run([sys.executable, os.path.abspath(__file__)], capture_output=True, text=True,
                       timeout=100, env=dict(os.environ, PYTHONPATH=ROOT))
    print(r.stdout, flush=True)
    assert r.returncode == 0 and "memory ok" in r.stdout, r.stdout + r.stderr


if __name__ == "__main__":
    check()
