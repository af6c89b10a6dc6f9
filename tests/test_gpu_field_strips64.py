"""FP64 field step where its strips of columns end: strips of 128 and of 256
threads (122 and 250 owned columns), full last strips and ones of one or a few
columns, slabs of one row and, on the tall grid, of several.  Every operation
is rounded as the oracle's or to one unit in the last place, so each component
agrees to 1e-12 of its largest value."""
import pytest

import oracle
from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W
from parity_util import rel
from test_gpu_fields64 import FIELDS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,nth", [(23, 8), (23, 121), (23, 122), (23, 243), (23, 249), (23, 250),
                                    (23, 365), (23, 366), (23, 487), (23, 500), (3001, 130)])
def test_field_step_strip_edges_fp64(nr, nth):
    oracle.build(force=False)
    w = W.tiny_open_dipole(16, steps=4)
    w.nr, w.nth = nr, nth
    d = w.desc()
    d["precision"] = W.FP64
    sim = ffpic.Sim(d, capacity=[1] * d["nspec"])
    ora = oracle.Oracle(d)
    sim.step(4)
    ora.step(4)
    for g, o in FIELDS:
        assert rel(sim.field(g), ora.field(o)) < 1e-12, g
