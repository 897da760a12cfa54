"""Polyphase wire pass with its phases cut over groups: phase counts around
multiples of two and five groups, wires around a block, one to several blocks,
both chunk widths, launches small enough for five groups, for two, and planes of
reproducible sums (one group).  Against the oracle's library FFT; tolerance as in
the tick transform tests, 1e-5 of the output's maximum."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2304_01841_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nimpact", [2, 3, 4, 5, 6, 10, 11])
@pytest.mark.parametrize("wires,ticks", [(3, 120), (108, 150), (230, 1400)])
def test_phases_over_groups(nimpact, wires, ticks):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_01841_amd import wcsim
    rng = np.random.default_rng(nimpact * 1000 + wires)
    Rp = min(21 * nimpact, 60)
    R = W.random_response(rng, Rp, 30)
    pl = W.plane(wires, ticks, nimpact=nimpact)
    G = rng.standard_normal((wires * nimpact, ticks)).astype(np.float32)
    ref = O.wire_rows(O.convolve(G, R.astype(np.float64), Rp // 3, workers=8), nimpact)
    Gt = torch.from_numpy(G).cuda()
    for F in (8, 16):
        for det in (0, 1):
            P = wcsim.Plane(pl, W.physics(False), R, r0=Rp // 3,
                            schedule={"freq_chunk": F, "wire_mode": 1, "deterministic": det})
            got = wcsim.convolve(P, Gt).cpu().numpy()
            again = wcsim.convolve(P, Gt).cpu().numpy()
            err = np.abs(got - ref).max() / np.abs(ref).max()
            print("nimpact %d wires %d F %d det %d err %.2g" % (nimpact, wires, F, det, err),
                  flush=True)
            assert err <= 1e-5 and np.array_equal(got, again)
            P.destroy()


@pytest.mark.parametrize("wires,ticks,nimpact", [(700, 1400, 3), (430, 2600, 5)])
def test_two_groups_of_sixteen_columns(wires, ticks, nimpact):
    """More than one workgroup per CU and at most four: two groups, 16 columns."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_01841_amd import wcsim
    rng = np.random.default_rng(wires)
    Rp = 21 * nimpact - 1
    R = W.random_response(rng, Rp, 30)
    P = wcsim.Plane(W.plane(wires, ticks, nimpact=nimpact), W.physics(False), R, r0=Rp // 2,
                    schedule={"freq_chunk": 16, "wire_mode": 1})
    wgs = 8 * -(-P.info["nchunks"] // 8) * P.info["wire_blocks"]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert cus < wgs <= 4 * cus
    G = rng.standard_normal((wires * nimpact, ticks)).astype(np.float32)
    ref = O.wire_rows(O.convolve(G, R.astype(np.float64), Rp // 2, workers=8), nimpact)
    got = wcsim.convolve(P, torch.from_numpy(G).cuda()).cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()
    P.destroy()


@pytest.mark.parametrize("nimpact", [2, 5, 10, 11])
@pytest.mark.parametrize("wires,ticks", [(3, 2000), (110, 1000), (240, 900), (330, 1000)])
def test_halves_of_sixteen_columns(wires, ticks, nimpact):
    """Chunks of sixteen columns, one to three blocks of wires, on both sides of
    the launches that take them by halves, alone and in a batch."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_01841_amd import wcsim
    rng = np.random.default_rng(wires + nimpact)
    Rp = min(21 * nimpact, 60)
    R = W.random_response(rng, Rp, 30)
    P = wcsim.Plane(W.plane(wires, ticks, nimpact=nimpact), W.physics(False), R, r0=Rp // 3,
                    schedule={"freq_chunk": 16, "wire_mode": 1})
    G = rng.standard_normal((wires * nimpact, ticks)).astype(np.float32)
    ref = O.wire_rows(O.convolve(G, R.astype(np.float64), Rp // 3, workers=8), nimpact)
    got = wcsim.convolve(P, torch.from_numpy(G).cuda()).cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()
    dep = torch.from_numpy(W.uniform_depos(rng, 500, (0.0, wires * W.PITCH), (0.0, ticks * W.TICK))).cuda()
    alone = wcsim.simulate_event(P, dep, 5)
    for n in (1, 2, 6):
        outs = [torch.full((wires, ticks), float("nan"), device="cuda") for _ in range(n)]
        wcsim.simulate_batch([P] * n, [dep] * n, [5] * n, outs)
        for o in outs:
            assert (o - alone).abs().max() <= 1e-5 * alone.abs().max()
    P.destroy()
