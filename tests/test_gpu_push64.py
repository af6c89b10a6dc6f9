"""FP64 push kernel instances against the oracle: every particles-per-thread
setting (chosen by the species' size), the remainders of its chunks, the
series and the library forms of the logarithm and arctangent (chosen by the
grid's spacings, at 1/16), and boxes too large for the LDS patches.

Tolerances: positions and momenta are formed by the oracle's operations, each
rounded to within one unit in the last place (2.2e-16), in a chain of a few
tens for the momenta (1e-13) and of the last few for r and theta (4 units);
currents are sums of the particles' in-cell displacements, whose offsets
carry one unit of r or theta over a cell (2.2e-16 / 0.06 relative to a cell)
against displacements of about a tenth of a cell: 1e-12 of the largest.
"""
import math

import numpy as np
import pytest

import oracle
from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W
from parity_util import rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build(force=False)
    ffpic.lib()


def scattered(w, n, seed, spread):
    """n particles over the domain (spread) or in a few cells, isotropic."""
    g = np.random.Generator(np.random.PCG64(seed))
    lo, hi = (1.05 * w.rmin, 0.98 * w.r_abs) if spread else (2.0, 2.3)
    t0, t1 = (0.0, math.pi) if spread else (1.4, 1.5)
    r = np.exp(g.uniform(math.log(lo), math.log(hi), n))
    th = g.uniform(t0, t1, n)
    if spread:
        th[: n // 50] *= 1e-4                      # next to the axes
        th[n // 50: n // 25] = math.pi - 1e-4 * th[n // 50: n // 25]
    u = g.normal(0.0, 3.0, (3, n))
    return dict(r=r, th=th, ur=u[0], uth=u[1], uph=u[2])


# grid spacings: 64 x 96; on either side of 1/16 in theta (nth 50, 51) and in
# log r (nr 36, 37 over ln 10); sizes: one slot, a chunk's edges, and past the
# sizes where a thread takes two (2^21) and eight (2^22) particles
@pytest.mark.parametrize("nr,nth,n,spread", [
    (64, 96, 1, True), (64, 96, 255, True), (64, 96, 257, True), (64, 96, 40_001, True),
    (64, 96, 40_000, False), (37, 51, 20_003, True), (36, 51, 20_003, True),
    (37, 50, 20_003, True), (12, 9, 5_000, True),
    (300, 517, (1 << 21) + 1, True), (300, 517, (1 << 22) + 7, True),
    (300, 517, (1 << 22) + 300, False)])
def test_push64_instances(nr, nth, n, spread):
    w = W.tiny_open_dipole(n)
    w.nr, w.nth = nr, nth
    w.rr_coef = 0.02
    w.shell_r = 1.5
    w.qm, w.weight = (1.0,), (1e-4,)
    d = w.desc()
    sim, ora = ffpic.Sim(d, capacity=[n]), oracle.Oracle(d)
    p = scattered(w, n, nr + nth + n, spread)
    sim.load_particles(0, p)
    ora.load(0, p)
    sim.run_phases(ffpic.PHASE_PUSH)
    ora.phases(oracle.PHASE_PUSH)
    g, o = sim.particles(0), ora.particles(0)
    live = o["r"] > 0
    assert np.array_equal(g["cell"], o["cell"])
    for k in ("r", "th"):
        assert np.allclose(g[k][live], o[k][live], rtol=4 * 2.2e-16, atol=1e-18), k
    for k in ("ur", "uth", "uph"):
        scale = np.abs(o[k][live]).max(initial=1.0)
        assert np.abs(g[k][live] - o[k][live]).max(initial=0.0) < 1e-13 * scale, k
    for a, b in ((ffpic.JR, oracle.JR), (ffpic.JTH, oracle.JTH), (ffpic.JPH, oracle.JPH)):
        assert rel(sim.field(a), ora.field(b)) < 1e-12
    assert np.array_equal(sim.diagnostics(0)["removed"][0], ora.removed(0))
