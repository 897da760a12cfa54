"""Patch sets from a handful of depos to tens of thousands, of ordinary windows
and of windows beyond a wavefront's reach: counts where a wavefront takes one more
patch (8,192, 16,384 and 32,768 depos) and where large patches change their
workgroup (1,024), windows and offsets bit for bit and values within 1e-5 of each
patch's maximum against the oracle (float32 products and draws of FP64 weights).
And what a set costs per value does not grow with its windows."""
import time

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2304_01841_amd import workloads as W

pytestmark = pytest.mark.gpu


def _plane(wcsim, phys, wires, ticks):
    pl = W.plane(wires, ticks)
    return pl, wcsim.Plane(pl, phys, W.response("unipolar", Rp=21, Rt=40, r0=10), r0=10)


def _check(dep, phys, wires, ticks, ev):
    from paper_2304_01841_amd import wcsim
    pl, P = _plane(wcsim, phys, wires, ticks)
    print("rasterize %d depos" % len(dep), flush=True)
    pt = wcsim.rasterize(P, torch.from_numpy(np.ascontiguousarray(dep)).cuda(), ev)
    meta, offs, vals = pt.to_host()
    pt.destroy()
    P.destroy()
    ometa, ovals, _ = O.rasterize(dep, phys, pl, ev)
    assert np.array_equal(meta, ometa[:, :4])
    assert np.array_equal(offs[:-1], ometa[:, 4]) and offs[-1] == ovals.size
    some = ometa[:, 2] * ometa[:, 3] > 0
    top = np.maximum.reduceat(ovals, ometa[some, 4])
    err = np.maximum.reduceat(np.abs(vals - ovals), ometa[some, 4])
    assert (err <= 1e-5 * top).all()
    return ometa


@pytest.mark.parametrize("fluct", [False, True])
@pytest.mark.parametrize("n", [2, 8191, 8192, 16383, 16385, 32768])
def test_patches_per_wavefront(n, fluct):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dep = W.uniform_depos(np.random.default_rng(n), n, (0.0, 200.0), (0.0, 250.0),
                          max_drift_time=400.0)
    _check(dep, W.physics(fluct), 40, 500, 7)


@pytest.mark.parametrize("large", [0, 1, 1024, 1025, 3000])
def test_large_patches_among_others(large):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(large)
    phys = W.physics(True)
    phys["DT"] *= 9.0
    phys["DL"] *= 9.0
    dep = W.uniform_depos(rng, 500 + large, (0.0, 200.0), (0.0, 250.0), max_drift_time=200.0)
    T = rng.uniform(2000.0, 2300.0, large)
    at = rng.permutation(len(dep))[:large]
    dep[at, 3] += dep[at, 0] / W.DRIFT_SPEED - T
    dep[at, 0] = T * W.DRIFT_SPEED
    m = _check(dep, phys, 40, 500, 9)
    nq = ((m[:, 1] + m[:, 3] - 1) >> 2) - (m[:, 1] >> 2) + 1
    beyond = (m[:, 2] + m[:, 3] + 2 > 64) | (m[:, 2] * nq > 192)
    assert beyond.sum() == large


def test_wide_windows_cost_no_more_per_value():
    """60,000 uniform depos whose windows hold 160 or 1,500 bins on average: a
    value of the wide set, most of whose patches are beyond a wavefront, costs no
    more than one of the other (about 0.6 of it)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_01841_amd import wcsim
    n, cost = 60_000, []
    for nsigma, factor in ((3.0, 1.0), (5.0, 4.0)):
        phys = W.physics(True)
        phys["nsigma"] = nsigma
        phys["DT"] *= factor
        phys["DL"] *= factor
        _, P = _plane(wcsim, phys, 480, 6000)
        dep = torch.from_numpy(W.uniform_depos(np.random.default_rng(3), n, (0.0, 2400.0),
                                               (0.0, 3000.0))).cuda()
        times, nvalues = [], 0
        for _ in range(12):
            torch.cuda.synchronize()
            t = time.perf_counter()
            pt = wcsim.rasterize(P, dep, 1)
            times.append(time.perf_counter() - t)
            nvalues = pt.nvalues
            pt.destroy()
        cost.append(np.median(times[2:]) / nvalues)
        print("nsigma %g: %.3g values, %.0f us" % (nsigma, nvalues, np.median(times[2:]) * 1e6),
              flush=True)
        P.destroy()
    assert cost[1] <= cost[0]
