"""Owner flush of tiles with one work item (a wavefront's) and with several (a
workgroup's): depo counts around multiples of an item's 32 depos and of a
workgroup's wavefronts, many of each kind in every colour.  The grid repeats bit
for bit, in a batch too, and agrees with the oracle (1e-5 of its maximum, the
repository's grid tolerance)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2304_01841_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [0, 1, 2])
@pytest.mark.parametrize("count", [1, 32, 33, 64, 191, 193, 400])
def test_light_and_heavy_tiles(tile, count):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_01841_amd import wcsim
    rng = np.random.default_rng(count)
    pl, phys = W.plane(24, 300), W.physics(True)
    spots = [(y, t) for y in range(3) for t in range(4)]
    parts = []
    for k, (y, t) in enumerate(spots):  # heavy and light tiles beside each other
        n = count if k % 2 == 0 else 1 + k
        z, a = 10.0 + 40.0 * y, 12.0 + 33.0 * t
        parts.append(W.uniform_depos(rng, n, (z, z + 2.0), (a, a + 1.0), max_drift_time=150.0))
    dep = np.concatenate(parts)
    dep = np.ascontiguousarray(dep[rng.permutation(len(dep))])
    dd = torch.from_numpy(dep).cuda()
    P = wcsim.Plane(pl, phys, W.response("unipolar", Rp=21, Rt=40, r0=10), r0=10,
                    schedule={"deterministic": 1, "tile": tile})
    outs = []
    for _ in range(2):
        ws = wcsim.simulate_workspace(P, len(dep), wcsim.OUT_PITCH)
        ws.fill_(0xFF)
        out = wcsim.simulate_event(P, dd, 17, kind=wcsim.OUT_PITCH, workspace=ws)
        outs.append((out.clone(), wcsim.workspace_grid(P, ws, len(dep)).clone()))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    both = [torch.empty_like(outs[0][0]) for _ in range(3)]
    wcsim.simulate_batch([P] * 3, [dd] * 3, [17, 18, 17], both, kind=wcsim.OUT_PITCH)
    assert torch.equal(both[0], outs[0][0]) and torch.equal(both[2], outs[0][0])
    G = O.grid(dep, phys, pl, 17)
    assert np.abs(outs[0][1].cpu().numpy() - G).max() <= 1e-5 * G.max()
    P.destroy()
