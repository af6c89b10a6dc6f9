"""FP64 field step where the node quotients change form: B^2 inside the range
that the stored reciprocals take, below it, and zero.  Every operation is
rounded as the oracle's or to one unit in the last place, so each component
agrees to 1e-12 of its largest value, as at ordinary field strengths."""
import numpy as np
import pytest

import oracle
from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W
from parity_util import rel

pytestmark = pytest.mark.gpu

FIELDS = [(ffpic.ER, oracle.ER), (ffpic.ETH, oracle.ETH), (ffpic.EPH, oracle.EPH),
          (ffpic.BR, oracle.BR), (ffpic.BTH, oracle.BTH), (ffpic.BPH, oracle.BPH)]


@pytest.mark.parametrize("scale", [1.0, 1e-100, 1e-136, 1e-150, 1e-200])
def test_field_step_at_any_strength_fp64(scale):
    oracle.build(force=False)
    w = W.tiny_open_dipole(16, steps=4)
    w.nr, w.nth = 37, 260
    w.mu = scale
    psi_pc = w.mu / w.r_lc
    w.psi_thr = (0.85 * psi_pc, 0.9 * psi_pc, 2.3 * psi_pc, 2.4 * psi_pc)
    d = w.desc()
    d["precision"] = W.FP64
    sim = ffpic.Sim(d, capacity=[1] * d["nspec"])
    ora = oracle.Oracle(d)
    sim.step(4)
    ora.step(4)
    for g, o in FIELDS:
        a, b = sim.field(g), ora.field(o)
        assert np.all(np.isfinite(a))
        # the norm squares the values: scaled back to ordinary ones first
        assert rel(a / scale, b / scale) < 1e-12, g
