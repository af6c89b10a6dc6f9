"""FP32 field step where the rows without a Faraday rate of the background are
read as one row: a corotating background (a rate in the last row only), one
whose rate reaches every row (an E0 of the toroidal component), and one loaded
into a context that has already captured its steps as a graph.  Against the
oracle in FP64 to 2e-5 of each field group's largest value, as the other
comparisons of the FP32 step over some ten steps."""
import numpy as np
import pytest

import oracle
from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W
from parity_util import rel_grouped

pytestmark = pytest.mark.gpu

E = [(ffpic.ER, oracle.ER, "Er"), (ffpic.ETH, oracle.ETH, "Eth"), (ffpic.EPH, oracle.EPH, "Eph")]
B = [(ffpic.BR, oracle.BR, "Br"), (ffpic.BTH, oracle.BTH, "Bth"), (ffpic.BPH, oracle.BPH, "Bph")]


@pytest.mark.parametrize("toroidal,before", [(False, 0), (True, 0), (True, 6)])
def test_background_rate_rows_fp32(toroidal, before):
    oracle.build(force=False)
    w = W.tiny_open_dipole(16, steps=8)
    w.nr, w.nth = 45, 300
    d = w.desc()
    d["precision"] = W.FP32_MIXED
    d["sort_interval"] = 2
    sim, ora = ffpic.Sim(d, capacity=[1] * d["nspec"]), oracle.Oracle(d)
    sim.step(before)
    ora.step(before)
    if toroidal:
        e = ora.field(oracle.EPH)
        i, j = np.meshgrid(np.arange(w.nr + 1), np.arange(w.nth + 1), indexing="ij")
        e = e + 1e-3 * np.abs(ora.field(oracle.ER)).max() * np.sin(np.pi * j / w.nth) ** 2 * (i > 0)
        e[:, [0, -1]] = 0.0
        # (all six, as a restart from files would: the background is then the
        # loaded state)
        fields = {g: ora.field(o) for g, o, _ in E + B}
        fields[ffpic.EPH] = e
        for g, o, _ in E + B:
            sim.load_fields(g, fields[g])
            ora.set_field(o, fields[g])
    sim.step(8)
    ora.step(8)
    for group in (E, B):
        errs = rel_grouped([(n, sim.field(g), ora.field(o)) for g, o, n in group])
        assert max(errs.values()) < 2e-5, errs
