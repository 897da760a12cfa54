"""The chunk width that the library chooses does not depend on the wires: planes
of one readout and response share a batch class and a response spectrum whatever
their wire counts, and a plane that shares another's spectrum gets the width it
would have had alone, so that nothing depends on which plane came first."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2304_01841_amd import workloads as W

pytestmark = pytest.mark.gpu

WIRES = (24, 100, 480, 800, 960)


def _chunks(wcsim, planes):
    p = (ctypes.c_void_p * len(planes))(*[x.handle.value for x in planes])
    n = (ctypes.c_int64 * len(planes))(*[1000] * len(planes))
    return wcsim._lib.wcsim_batch_chunk_count(p, n, len(planes), wcsim.OUT_WIRE)


# (953 and 3257 ticks: 1152- and 3456-point transforms, the longest below 1200 and
# 3600)
@pytest.mark.parametrize("det", [0, 1])
@pytest.mark.parametrize("ticks", [300, 953, 954, 2000, 3000, 3257, 3258, 6000])
def test_one_class_of_any_wire_count(ticks, det):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_01841_amd import wcsim
    phys, R = W.physics(True), W.response("bipolar")
    sched = {"deterministic": det}
    planes = [wcsim.Plane(W.plane(w, ticks), phys, R, schedule=sched) for w in WIRES]
    widths = {p.info["freq_chunk"] for p in planes}
    assert widths == {16 if ticks >= (3258 if det else 954) else 8}
    assert _chunks(wcsim, planes) == 1
    for donor in (planes[0], planes[-1]):
        for w in WIRES:
            q = wcsim.Plane(W.plane(w, ticks), phys, R, share=donor)
            assert q.info["freq_chunk"] == donor.info["freq_chunk"]
            assert _chunks(wcsim, planes + [q]) == 1
            q.destroy()
    # short responses have 16 columns at any length
    short = wcsim.Plane(W.plane(24, ticks), phys, W.response("bipolar", Rp=21, Rt=20, r0=10), r0=10)
    assert short.info["freq_chunk"] == 16
    for p in planes + [short]:
        p.destroy()


def test_default_mixed_batch_agrees_with_single_events():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_01841_amd import wcsim
    phys, R, ticks = W.physics(True), W.response("unipolar"), 4000
    planes = [wcsim.Plane(W.plane(w, ticks), phys, R) for w in (24, 300, 960)]
    deps = [torch.from_numpy(W.uniform_depos(np.random.default_rng(w.nwires), 3000,
                                             (0.0, w.nwires * W.PITCH), (0.0, ticks * W.TICK))).cuda()
            for w in planes]
    outs = [torch.full((p.nwires, ticks), float("nan"), device="cuda") for p in planes]
    wcsim.simulate_batch(planes, deps, [1, 2, 3], outs)
    for p, d, e, o in zip(planes, deps, (1, 2, 3), outs):
        ref = wcsim.simulate_event(p, d, e)
        assert (o - ref).abs().max() <= 1e-5 * ref.abs().max()
        p.destroy()
