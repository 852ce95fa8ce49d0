"""The pattern tile (partial sums of 8 channels shared between trials) is
bit-exact where it can go wrong: channel counts around whole groups of 8,
trial counts around its tiles, outputs around its 512-sample tiles, every
downsampling it takes, saturated input, either band order."""
import numpy as np
import pytest

import oracle
from paper_2110_12749_amd import synth
from tests._util import say

pytestmark = pytest.mark.gpu


def _check(nchan, nsamp, segs, tpw=None, tsamp=98.304e-6, f_lo=1000.0, f_hi=1500.0, descending=False,
           saturated=False):
    """Every row with the pattern tile (tpw: trials per wave forced; None: the
    default) against the oracle; outputs prefilled with a sentinel."""
    import torch
    from paper_2110_12749_amd import gsp
    w = synth.small(nchan=nchan, nsamp=nsamp, segments=segs, tsamp=tsamp, f_lo=f_lo, f_hi=f_hi, n_pulses=1)
    X, freqs = w.generate(), w.freqs
    if saturated:
        X[:] = 255
        X[::3] = 0
    if descending:
        X, freqs = np.ascontiguousarray(X[:, ::-1]), freqs[::-1].copy()
    ref = oracle.dedisperse(X, freqs, w.tsamp, w.segments)
    desc = gsp.plan_shape(w.nsamp, freqs, w.tsamp, w.segments)
    ctx = gsp.Context(0)
    try:
        for s in range(desc.n_seg):
            if tpw is not None:
                ctx.set_row_shape(freqs, desc, s, 4, tpw, 8, 16, 4)
            shape = ctx.row_shape(freqs, desc, s)
            say(f"[case] row {s}: {shape}, {desc.n_out[s]} outputs")
            assert shape[4] == 4
        fb = torch.from_numpy(X).to("cuda")
        dmt = ctx.dedisperse(fb, freqs, desc, out=torch.full((desc.total,), -1, dtype=torch.int32, device="cuda"))
        for s, v in enumerate(gsp.segment_views(desc, dmt)):
            bad = np.argwhere(v.cpu().numpy() != ref[s])
            assert len(bad) == 0, f"row {s}: {len(bad)} mismatches, first {bad[:5].tolist()}"
    finally:
        torch.cuda.synchronize()
        ctx.close()


@pytest.mark.parametrize("tpw", [12, 8])
@pytest.mark.parametrize("nchan,descending", [(128, False), (203, True)])
def test_every_downsampling(dev, tpw, nchan, descending):
    _check(nchan, 12000, [(0.0, 0.3, 133, 1), (39.9, 0.8, 65, 2), (91.9, 1.5, 20, 3), (121.9, 2.0, 15, 8)], tpw,
           f_lo=1400.0, descending=descending)


@pytest.mark.parametrize("nchan", [1, 7, 8, 9])
def test_few_channels(dev, nchan):
    _check(nchan, 5000, [(0.0, 0.2, 5, 1), (1.0, 0.3, 3, 4)], 12)


@pytest.mark.parametrize("n_dm", [1, 95, 96, 97])
def test_trial_tile_edges(dev, n_dm):
    _check(128, 6000, [(0.0, 0.3, n_dm, 1)], 12, f_lo=1400.0)


@pytest.mark.parametrize("extra", [1, 255, 256, 257, 511, 512, 513])
def test_output_tile_edges(dev, extra):
    """Rows of exactly `extra` outputs past one whole tile less 512."""
    from paper_2110_12749_amd import gsp
    segs = [(0.0, 0.4, 40, 1)]
    w = synth.small(nchan=64, nsamp=8000, segments=segs, tsamp=98.304e-6)
    delay = 8000 - gsp.plan_shape(w.nsamp, w.freqs, w.tsamp, segs).n_out[0]
    _check(64, delay + extra, segs, 12)


@pytest.mark.parametrize("D", [1, 8])
def test_saturated(dev, D):
    """The largest sums: every 16-bit half is carried before it overflows."""
    _check(1024, 9000 * D, [(0.0, 1.0, 24, D)], 12, tsamp=196.608e-6, saturated=True)


def test_wide_band(dev):
    """Delays inside a group span many shifts: patterns fall into subgroups."""
    _check(512, 40000, [(0.0, 0.1, 100, 1)], 8, tsamp=196.608e-6, f_lo=270.0, f_hi=1620.0)


def test_default_where_it_fills_the_chip(dev):
    _check(96, 140000, [(0.0, 0.3, 100, 1)], f_lo=1400.0)
