"""Scatter-add of patch sets on both sides of its rules: counts around 4,096
(patches summed in LDS from there on, where neighbours lie together), 49,152 and
98,304 (more patches a wavefront), neighbours together, apart, half and half, and
in another order; grids against the oracle within 1e-5 of their maximum.  And
patches that share no cell run side by side: a set costs about what one patch
does while the chip is not full."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2304_01841_amd import workloads as W

pytestmark = pytest.mark.gpu


def _depos(kind, n):
    rng = np.random.default_rng(n)
    apart = W.uniform_depos(rng, n, (0.0, 300.0), (0.0, 400.0), max_drift_time=40.0)
    along = apart.copy()  # tracks of 256 depos, 0.02 mm and 0.01 us apart
    step = np.arange(n) % 256
    first = np.arange(n) - step
    along[:, 0] = apart[first, 0]
    along[:, 2] = apart[first, 2] + 0.02 * step
    along[:, 3] = apart[first, 3] + 0.01 * step
    if kind == "together":
        return along
    if kind == "mixed":
        return np.concatenate([along[:n // 2], apart[n // 2:]])
    if kind == "shuffled":
        return along[rng.permutation(n)]
    return apart


@pytest.mark.parametrize("kind", ["together", "apart", "mixed", "shuffled"])
@pytest.mark.parametrize("n", [9, 4095, 4096, 49151, 49153, 98305])
def test_grid_of_sets(n, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_01841_amd import wcsim
    pl, phys = W.plane(60, 800), W.physics(False)
    P = wcsim.Plane(pl, phys, W.response("unipolar", Rp=21, Rt=40, r0=10), r0=10)
    dep = np.ascontiguousarray(_depos(kind, n))
    print("scatter: %s, %d depos" % (kind, n), flush=True)
    pt = wcsim.rasterize(P, torch.from_numpy(dep).cuda(), 1)
    G = torch.full((P.npitch, P.nticks), 7.0, device="cuda")
    wcsim.scatter_add(P, pt, G)
    ometa, ovals, _ = O.rasterize(dep, phys, pl, 1)
    ref = O.scatter(ometa, ovals, pl)
    assert np.abs(G.cpu().numpy() - ref).max() <= 1e-5 * ref.max()
    wcsim.scatter_add(P, pt, G, zero_first=False)
    assert np.abs(G.cpu().numpy() - 2 * ref).max() <= 2e-5 * ref.max()
    pt.destroy()
    P.destroy()


def _time(wcsim, phys, n, arrival):
    P = wcsim.Plane(W.plane(960, 6000), phys, W.response("unipolar", Rp=21, Rt=40, r0=10), r0=10)
    dep = W.uniform_depos(np.random.default_rng(n), n, (500.0, 4300.0), (400.0, 2600.0))
    dep[:, 3] += dep[:, 0] / W.DRIFT_SPEED - arrival
    dep[:, 0] = arrival * W.DRIFT_SPEED
    pt = wcsim.rasterize(P, torch.from_numpy(dep).cuda(), 1)
    G = torch.zeros((P.npitch, P.nticks), device="cuda")
    times = []
    for _ in range(9):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            wcsim.scatter_add(P, pt, G, zero_first=False)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) / 20 * 1e3)
    pt.destroy()
    P.destroy()
    t = float(np.median(times))
    print("%d patches: %.1f us" % (n, t), flush=True)
    return t


@pytest.mark.parametrize("diffusion,many", [(100.0, 16), (1.0, 1000)])
def test_separate_patches_run_side_by_side(diffusion, many):
    """Sixteen windows of some 20,000 bins, or 1,000 ordinary ones, in less than
    twice the time of one."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_01841_amd import wcsim
    phys = W.physics(False)
    phys["DT"] *= diffusion
    phys["DL"] *= diffusion
    assert _time(wcsim, phys, many, 1500.0) < 2.0 * _time(wcsim, phys, 1, 1500.0)
