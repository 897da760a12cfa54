"""Tick-axis transforms of every kind of length: each single-pass radix, plans
of several passes, several rows per workgroup with a remainder, the longest
lengths, odd readouts.  The convolution against the oracle's library FFT.

Tolerance: a float32 transform of n points loses about eps log2(n) of its
largest value (6e-8 * 15 for the longest here); two transforms per axis and a
spectrum product make that about 4e-6 of the output's maximum, so 1e-5."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2304_01841_amd import workloads as W

pytestmark = pytest.mark.gpu

SINGLE = [2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16]          # one pass
MULTI = [18, 25, 48, 60, 81, 160, 250, 512, 864, 1125]  # several rows per workgroup
LONG = [1600, 1875, 2187, 4096, 4608, 6561, 9720, 10000]


@pytest.mark.parametrize("n2", SINGLE + MULTI + LONG)
def test_tick_transform_lengths(n2):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_01841_amd import wcsim
    rng = np.random.default_rng(n2)
    Rt = 2 if n2 < 32 else 21
    nt = 2 * n2 + 1 - Rt  # the largest readout of this transform (odd for Rt = 2)
    nt -= (n2 % 3 == 0 and nt > 3)  # and a shorter one
    pl = W.plane(3, nt, nimpact=5)  # 15 rows: a remainder for 2, 4 and 8 rows a workgroup
    R = W.random_response(rng, 7, Rt)
    P = wcsim.Plane(pl, W.physics(False), R, r0=3, schedule={"fft_ticks": 2 * n2})
    assert P.info["fft_ticks"] == 2 * n2
    G = rng.standard_normal((15, nt)).astype(np.float32)
    ref = O.convolve(G, R.astype(np.float64), 3)
    for kind, want in ((wcsim.OUT_PITCH, ref), (wcsim.OUT_WIRE, O.wire_rows(ref, 5))):
        got = wcsim.convolve(P, torch.from_numpy(G).cuda(), kind=kind).cpu().numpy()
        err = np.abs(got - want).max() / np.abs(ref).max()
        print("N2 %d nt %d kind %d err %.2g" % (n2, nt, kind, err), flush=True)
        assert err <= 1e-5
    P.destroy()


@pytest.mark.parametrize("nt", [100, 101, 1000, 6000])
def test_a_grid_at_any_float(nt):
    """A grid that starts one float into its storage gives the aligned grid's
    output bit for bit (the same arithmetic on the same values)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_01841_amd import wcsim
    P = wcsim.Plane(W.plane(5, nt), W.physics(False), W.response("bipolar"), r0=105)
    g = torch.Generator(device="cuda").manual_seed(nt)
    G = torch.rand((50, nt), generator=g, device="cuda")
    off = torch.zeros(50 * nt + 1, device="cuda")[1:].view(50, nt)
    off.copy_(G)
    for kind in (wcsim.OUT_WIRE, wcsim.OUT_PITCH):
        assert torch.equal(wcsim.convolve(P, G, kind=kind), wcsim.convolve(P, off, kind=kind))
    P.destroy()
