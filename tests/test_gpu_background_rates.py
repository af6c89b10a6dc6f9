"""FP32-mixed: the Faraday rate of a loaded background that is nearly, but not,
free of curl.  The interior's rate lies below 1e-9 of max |E| over the first
cell, the outer boundary's (where E_theta ends) far above it; both act."""
import numpy as np
import pytest

from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["everywhere", "inner rows", "one row"])
def test_small_background_rate_is_integrated(where):
    """B_phi starts at zero and grows by -dt (curl E)_phi a step, so the FP32
    path must show the whole of it: the rate is held to 6e-8, the FP64 path's
    own rounding of the curl is 1e-16 E / dr a step against a rate of
    1e-10 E / dr, and E follows B_phi by 1e-2 of a step's change in four steps,
    in both paths alike: 1e-4 of the largest."""
    w = W.tiny_dipole(16)
    w.nr, w.nth = 96, 80
    sims = {}
    for prec in (W.FP64, W.FP32_MIXED):
        d = w.desc()
        d["precision"] = prec
        sims[prec] = ffpic.Sim(d, capacity=[16, 16])
    a, b = sims[W.FP64], sims[W.FP32_MIXED]
    e = a.field(ffpic.ETH)
    er = a.field(ffpic.ER)
    peak = max(np.abs(e).max(), np.abs(er).max())
    i = np.arange(97.0)[:, None]
    j = np.arange(81.0)[None, :]
    shape = {"everywhere": i < 96, "inner rows": i < 40, "one row": i == 30}[where]
    # of alternating sign from row to row, so that the curl is 2e-10 E / dr
    e = e + np.where(shape, 1e-10 * peak * np.sin(0.3 * j) * (-1.0) ** i, 0.0)
    e[:, 80] = 0.0
    for s in (a, b):
        s.load_fields(ffpic.ETH, e)
        s.step(4)
    x, y = a.field(ffpic.BPH)[:80], b.field(ffpic.BPH)[:80]
    assert 0.0 < np.abs(x).max() < 1e-8 * peak
    assert np.abs(x - y).max() < 1e-4 * np.abs(x).max()
