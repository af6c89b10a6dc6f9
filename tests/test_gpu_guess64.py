"""FP64 push on grids where its single-precision guess of a radial cell is no
guide: shells whose cells are thinner than a float resolves, and radii beyond a
float's range.  Particles in a few cells would fit the LDS patches of their
guesses' box; the cells they are in lie anywhere.

In the thin shell a unit in the last place of r (2.2e-16) is 2.2e-8 of a cell,
moves are a few tenths of one, and polar moves 1e-8 with units of 2.2e-16:
currents agree to 2e-6 of the largest.  At 1e39 they are as on any grid of this
size (1e-12, as in the tests of the push's instances)."""
import math

import numpy as np
import pytest

import oracle
from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W
from parity_util import rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,rmin,ratio,tol", [
    (64, 1.0, 64e-8, 2e-6), (500, 1.0, 500e-8, 2e-6), (64, 1e39, math.log(10.0), 1e-12),
    (64, 1e-39, math.log(10.0), 1e-12)])
@pytest.mark.parametrize("n,few", [(3000, True), (3000, False), (1, False)])
def test_push64_where_the_guess_is_no_guide(nr, rmin, ratio, tol, n, few):
    oracle.build(force=False)
    w = W.tiny_dipole(n)
    w.nr, w.nth, w.rmin = nr, 96, rmin
    w.rmax = w.r_abs = rmin * math.exp(ratio)
    w.r_lc = 3.0 * rmin
    w.qm, w.weight = (1.0,), (1e-4,)
    d = w.desc()
    d["precision"], d["init"] = W.FP64, W.INIT_ZERO
    g = np.random.Generator(np.random.PCG64(nr + n))
    lo, hi = (0.4, 0.4 + 3.0 / nr) if few else (0.05, 0.95)
    r = rmin * np.exp(g.uniform(lo, hi, n) * ratio)
    th = g.uniform(1.4, 1.45, n) if few else g.uniform(0.2, 2.9, n)
    u = g.normal(0.0, 3.0, (3, n))
    p = dict(r=r, th=th, ur=u[0], uth=u[1], uph=u[2])
    sim, ora = ffpic.Sim(d, capacity=[n]), oracle.Oracle(d)
    sim.load_particles(0, p)
    ora.load(0, p)
    for _ in range(2):
        sim.run_phases(ffpic.PHASE_PUSH)
        ora.phases(oracle.PHASE_PUSH)
    a, b = sim.particles(0), ora.particles(0)
    assert np.sum(a["cell"] != b["cell"]) <= n // 1000
    for x, y in ((ffpic.JR, oracle.JR), (ffpic.JTH, oracle.JTH), (ffpic.JPH, oracle.JPH)):
        assert rel(sim.field(x), ora.field(y)) < tol
