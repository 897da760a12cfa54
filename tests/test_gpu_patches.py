"""Patch values by wavefront and the staged scatter at the sizes where they can
go wrong: windows of one bin, around the 64 window edges and 192 items that a
wavefront holds (beyond them the generic kernel), patch counts around a
wavefront's eight and the scatter's sixteen, patches on one spot, along a track,
far apart, across and outside the grid.  Windows bit for bit and values within
1e-5 of each patch's maximum (float32 products and draws of FP64 weights, as the
repository's patch tests); the grid within 1e-5 of its maximum."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2304_01841_amd import workloads as W

pytestmark = pytest.mark.gpu


def _check(dep, phys, pl, ev, label):
    from paper_2304_01841_amd import wcsim
    P = wcsim.Plane(pl, phys, W.response("unipolar", Rp=21, Rt=40, r0=10), r0=10)
    print("patches: %s, %d depos" % (label, len(dep)), flush=True)
    pt = wcsim.rasterize(P, torch.from_numpy(np.ascontiguousarray(dep)).cuda(), ev)
    meta, offs, vals = pt.to_host()
    ometa, ovals, _ = O.rasterize(dep, phys, pl, ev)
    assert np.array_equal(meta, ometa[:, :4]), label
    for d in range(len(dep)):
        o, m = ometa[d, 4], ometa[d, 2] * ometa[d, 3]
        if m:
            ref = ovals[o:o + m]
            assert np.abs(vals[offs[d]:offs[d] + m] - ref).max() <= 1e-5 * max(ref.max(), 1e-300), (label, d)
    G = torch.full((P.npitch, P.nticks), 7.0, device="cuda")
    wcsim.scatter_add(P, pt, G)
    ref = O.scatter(ometa, ovals, pl)
    assert np.abs(G.cpu().numpy() - ref).max() <= 1e-5 * max(ref.max(), 1e-300), label
    wcsim.scatter_add(P, pt, G, zero_first=False)
    assert np.abs(G.cpu().numpy() - 2 * ref).max() <= 2e-5 * max(ref.max(), 1e-300), label
    pt.destroy()
    P.destroy()


@pytest.mark.parametrize("fluct", [False, True])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 16, 17, 33])
def test_patch_counts_and_places(n, fluct):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(n)
    phys = W.physics(fluct)
    pl = W.plane(12, 301)
    spot = W.uniform_depos(rng, n, (30.0, 30.2), (70.0, 70.5), max_drift_time=2000.0)
    track = W.track_depos(rng, 1, per_seg=n, box=(3000.0, 100.0, 60.0), step=0.5)
    track[:, 3] = 60.0 - track[:, 0] / W.DRIFT_SPEED + np.arange(n) * 0.3
    far = W.uniform_depos(rng, n, (-8.0, 68.0), (-20.0, 170.0), max_drift_time=2400.0)
    still = far.copy()
    still[:, 0] = 0.0
    for label, dep in (("spot", spot), ("track", track), ("far", far), ("no drift", still)):
        _check(dep, phys, pl, 3 + n, label)


@pytest.mark.parametrize("fluct", [False, True])
def test_windows_around_a_wavefronts_reach(fluct):
    """Drift times and diffusion spread so that n_p + n_t + 2 passes 64 and the
    items pass 192, among ordinary patches; some draws all zero."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(8)
    pl = W.plane(20, 500)
    phys = W.physics(fluct)
    phys["DT"] *= 6.0
    phys["DL"] *= 4.0
    phys["lifetime"] = 4000.0
    dep = W.uniform_depos(rng, 300, (-5.0, 105.0), (-10.0, 260.0), max_drift_time=3000.0)
    dep[::7, 4] = rng.uniform(0.0, 3.0, dep[::7].shape[0])
    ometa, _, _ = O.rasterize(dep, phys, pl, 5)
    edges = ometa[:, 2] + ometa[:, 3] + 2
    assert (edges > 64).sum() > 20 and (edges <= 64).sum() > 20
    _check(dep, phys, pl, 5, "mixed")


def test_kept_buffers_serve_one_set_at_a_time():
    """Sets of one plane made after others were destroyed: smaller, larger, two
    alive together, host depos, several threads, and a set that outlives its
    plane.  Every set holds its own values."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import threading
    from paper_2304_01841_amd import wcsim
    pl, phys = W.plane(12, 301), W.physics(True)
    P = wcsim.Plane(pl, phys, W.response("unipolar", Rp=21, Rt=40, r0=10), r0=10)

    def depos(seed, n):
        return W.uniform_depos(np.random.default_rng(seed), n, (0.0, 60.0), (0.0, 150.0))

    def same(pt, dep, ev):
        meta, offs, vals = pt.to_host()
        ometa, ovals, _ = O.rasterize(dep, phys, pl, ev)
        assert np.array_equal(meta, ometa[:, :4]) and np.array_equal(offs[:-1], ometa[:, 4])
        assert np.abs(vals - ovals).max() <= 1e-5 * ovals.max()

    for n in (200, 150, 900, 20, 900):
        dep = depos(n, n)
        pt = wcsim.rasterize(P, dep if n == 150 else torch.from_numpy(dep).cuda(), n)
        same(pt, dep, n)
        pt.destroy()
    a, b = depos(1, 300), depos(2, 280)
    pa = wcsim.rasterize(P, torch.from_numpy(a).cuda(), 1)
    pb = wcsim.rasterize(P, torch.from_numpy(b).cuda(), 2)
    same(pa, a, 1)
    same(pb, b, 2)
    pa.destroy()
    pb.destroy()
    failed = []

    def worker(seed):
        try:
            s = torch.cuda.Stream()
            for r in range(4):
                dep = depos(10 * seed + r, 100 + 30 * seed)
                dd = torch.from_numpy(dep).cuda()
                torch.cuda.current_stream().synchronize()
                pt = wcsim.rasterize(P, dd, r, stream=s)
                same(pt, dep, r)
                pt.destroy()
        except Exception as e:  # noqa: BLE001 (reported below)
            failed.append(e)

    ts = [threading.Thread(target=worker, args=(k,)) for k in range(3)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not failed, failed
    last = wcsim.rasterize(P, torch.from_numpy(a).cuda(), 1)
    P.destroy()
    same(last, a, 1)
    last.destroy()
