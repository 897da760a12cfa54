"""Which events the allocation-free entry point takes does not depend on the
chunk width that the library chooses: the limit of 64 MiB counts the spectra of
such a plane in chunks of eight columns, for a plane of its own and for one that
shares a larger plane's response spectrum.  The largest event is taken and agrees
with wcsim_simulate_event; one depo more than fits is refused.  A width that the
caller asks for counts as it is."""
import numpy as np
import pytest
import torch

from paper_2304_01841_amd import workloads as W

pytestmark = pytest.mark.gpu

CONV_TOL = 1e-4  # normwise, the bar of the convolved output


def _most(wcsim, P, kind):
    """Most depos whose workspace (as P counts it) is within the limit."""
    lo, hi = 0, 1 << 20
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if wcsim._lib.wcsim_simulate_workspace_bytes(P.handle, mid, kind) <= wcsim.NOALLOC_SCRATCH_BYTES:
            lo = mid
        else:
            hi = mid
    return lo


@pytest.mark.parametrize("wires,ticks", [(100, 6000), (130, 4000), (60, 9000), (480, 1050)])
def test_limit_is_that_of_eight_columns(wires, ticks):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_01841_amd import wcsim
    pl, phys, R = W.plane(wires, ticks), W.physics(False), W.response("bipolar")
    donor = wcsim.Plane(W.plane(960, ticks), phys, R)
    own = wcsim.Plane(pl, phys, R)
    shared = wcsim.Plane(pl, phys, R, share=donor)
    eight = wcsim.Plane(pl, phys, R, schedule={"freq_chunk": 8})
    wide = wcsim.Plane(pl, phys, R, schedule={"freq_chunk": 16})
    kind = wcsim.OUT_WIRE
    n = _most(wcsim, eight, kind)
    box = (0.0, wires * W.PITCH), (0.0, ticks * W.TICK)
    dep = torch.from_numpy(W.uniform_depos(np.random.default_rng(wires), n + 1, *box)).cuda()
    ref = wcsim.simulate_event(eight, dep[:n], 3).cpu().numpy()
    for name, P in (("own", own), ("shared", shared)):
        print("case: %s, %d wires x %d ticks, %d depos" % (name, wires, ticks, n), flush=True)
        out = torch.full((P.nwires, P.nticks), float("nan"), device="cuda")
        got = wcsim.simulate_event_noalloc(P, dep[:n], 3, out).cpu().numpy()
        assert np.abs(got - ref).max() <= CONV_TOL * np.abs(ref).max(), name
        with pytest.raises(wcsim.WcsimError) as ei:
            wcsim.simulate_event_noalloc(P, dep, 3, out)
        assert ei.value.status == wcsim.E_INVALID
    most = _most(wcsim, wide, kind)
    assert most < n
    out = torch.empty((pl["nwires"], ticks), device="cuda")
    wcsim.simulate_event_noalloc(wide, dep[:most], 3, out)
    with pytest.raises(wcsim.WcsimError):
        wcsim.simulate_event_noalloc(wide, dep[:most + 1], 3, out)
    for P in (donor, own, shared, eight, wide):
        P.destroy()
