"""Flux function, blending function and kill flags from one kernel, whose
blocks overlap by one radial row: grids whose last block holds one row of cells
or a full set, for the 4 to 12 rows of single launches and the 16 of grouped
ones, and columns around the tile of 256.  The flux function is a
sum in a fixed order and the rest are choices made from it, so everything is
bit for bit the oracle's (FP32: the single context's)."""
import math

import numpy as np
import pytest

import oracle
from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W
from test_gpu_parity import kill_cells

pytestmark = pytest.mark.gpu


def dipole(nr, nth, precision):
    w = W.tiny_open_dipole(nr * nth)
    w.nr, w.nth = nr, nth
    d = w.desc()
    d["precision"] = precision
    d["sort_interval"] = 1000
    d["ff_enable"] = 1
    return d


@pytest.mark.parametrize("nr,nth", [(43, 255), (44, 256), (45, 257), (45, 513), (2047, 6),
                                    (2050, 257), (2051, 8), (2052, 6), (2057, 40)])
def test_flux_mask_and_kill_flags(nr, nth):
    oracle.build(force=False)
    d = dipole(nr, nth, W.FP64)
    sim, ora = ffpic.Sim(d, capacity=[nr * nth] * d["nspec"]), oracle.Oracle(d)
    # one particle at the centre of each cell: those that the load keeps
    i, j = np.meshgrid(np.arange(nr), np.arange(nth), indexing="ij")
    r = np.exp((i + 0.5) * (math.log(d["rmax"]) / nr)).reshape(-1)
    z = np.zeros_like(r)
    p = dict(r=r, th=((j + 0.5) * math.pi / nth).reshape(-1), ur=z, uth=z, uph=z)
    sim.load_particles(0, p)
    ora.load(0, p)
    assert np.array_equal(sim.field(ffpic.PSI), ora.field(oracle.PSI))
    assert np.array_equal(sim.field(ffpic.F), ora.field(oracle.F))
    cells = sim.particles(0)["cell"]
    assert 0 < len(cells) < nr * nth
    assert np.array_equal(cells, ora.particles(0)["cell"])
    assert not kill_cells(sim, nr, nth)[cells].any()


@pytest.mark.parametrize("nr,nth", [(768, 20), (769, 20), (771, 600), (1276, 8), (1281, 8),
                                    (1289, 300), (1793, 6), (1794, 257), (2816, 6), (2817, 6),
                                    (2824, 260)])
def test_flux_mask_and_kill_flags_by_rows(nr, nth):
    test_flux_mask_and_kill_flags(nr, nth)


def test_flux_and_mask_grouped():
    shapes = [(44, 256), (45, 257), (46, 30), (60, 513), (61, 255)]
    descs = [dipole(nr, nth, W.FP32_MIXED) for nr, nth in shapes]
    batch = ffpic.Batch(descs, [[1] * d["nspec"] for d in descs])
    batch.step(3)
    batch.sync()
    for k, d in enumerate(descs):
        sim = ffpic.Sim(d, capacity=[1] * d["nspec"])
        sim.step(3)
        for c in (ffpic.PSI, ffpic.F):
            assert np.array_equal(batch.view(k).field(c), sim.field(c)), (k, c)
