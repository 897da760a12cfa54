"""Coloured noise on rows shorter than the filter: the codes equal the oracle's,
whatever the taps that reach past the row hold, and those taps cost nothing."""
import numpy as np
import pytest
import torch

from oracle import oracle as O

pytestmark = pytest.mark.gpu

SEED = 0x1234_5678_9ABC


def _digitize(wave, fir):
    from paper_2304_01841_amd import wcsim
    out = torch.zeros(wave.shape, dtype=torch.int16, device="cuda")
    wcsim.digitize(wave, 1.25, 700.0, 3.0, 13, SEED, 4, out=out, fir=fir)
    return out


@pytest.mark.parametrize("ncols", [1, 7, 8, 9, 64, 255, 257, 511, 513])
def test_codes_of_short_rows(ncols):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(ncols)
    w = (rng.standard_normal((6, ncols)) * 400.0).astype(np.float32)
    for nfir in (ncols, ncols + 1, ncols + 7, 1000):
        f = (rng.standard_normal(nfir) / np.sqrt(nfir)).astype(np.float32)
        print("%d columns, %d taps" % (ncols, nfir), flush=True)
        ref = O.digitize(w, 1.25, 700.0, 3.0, 13, SEED, 4, fir=f.astype(np.float64))
        wd = torch.from_numpy(w).cuda()
        got = _digitize(wd, torch.from_numpy(f).cuda()).cpu().numpy().view(np.uint16)
        assert np.array_equal(got, ref)
        if nfir > ncols:  # (no column reaches back that far)
            f[ncols:] = np.inf
            same = _digitize(wd, torch.from_numpy(f).cuda()).cpu().numpy().view(np.uint16)
            assert np.array_equal(same, ref)


def test_taps_past_the_row_cost_nothing():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = torch.randn((960, 64), device="cuda") * 400.0
    times = []
    for nfir in (64, 1000):
        f = torch.randn(nfir, device="cuda")
        v = []
        for _ in range(9):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                _digitize(w, f)
            b.record()
            torch.cuda.synchronize()
            v.append(a.elapsed_time(b) / 20 * 1e3)
        times.append(float(np.median(v)))
        print("%d taps: %.1f us" % (nfir, times[-1]), flush=True)
    assert times[1] < 1.5 * times[0]


@pytest.mark.parametrize("rows,ncols,nfir", [(1, 1001, 1), (3, 3001, 32), (3, 3001, 33), (512, 1000, 33),
                                             (513, 1000, 33), (768, 1001, 32), (769, 1001, 32),
                                             (300, 2049, 5), (1, 513, 513), (1280, 1001, 9),
                                             (1281, 1001, 9)])
def test_codes_of_few_and_many_workgroups(rows, ncols, nfir):
    """On both sides of the launch sizes where a workgroup gets more threads or
    fewer columns; whole and ragged groups of eight columns."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(rows)
    w = (rng.standard_normal((rows, ncols)) * 400.0).astype(np.float32)
    f = (rng.standard_normal(nfir) / np.sqrt(nfir)).astype(np.float32)
    ref = O.digitize(w, 1.25, 700.0, 3.0, 13, SEED, 4, fir=f.astype(np.float64))
    got = _digitize(torch.from_numpy(w).cuda(), torch.from_numpy(f).cuda())
    assert np.array_equal(got.cpu().numpy().view(np.uint16), ref)
