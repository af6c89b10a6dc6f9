"""Grids of more than 32768 radial rows (65535 are accepted): a cell packed as
(row << 16) | column fills the sign bit there.  The push, its deposit through
the LDS patches (particles in a few cells) and straight to the grid (scattered
ones), in-cell and crossing moves, and the node charges, against the oracle.

A cell is 5.8e-5 of its radius thick, so one unit in the last place of r
(2.2e-16 of it) is 4e-12 of a cell; a step moves a particle by up to 0.1 of
one.  FP64 currents therefore agree to 4e-12 / 0.1 with a few such units in
either end, 2e-10 of the largest entry."""
import math

import numpy as np
import pytest

import oracle
from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W
from parity_util import rel

pytestmark = pytest.mark.gpu

NR = 40_000


def tall(nth, n, few, seed, precision):
    w = W.tiny_open_dipole(n)
    w.nr, w.nth = NR, nth
    w.qm, w.weight = (1.0,), (1e-4,)
    d = w.desc()
    d["precision"], d["ff_enable"] = precision, 0
    g = np.random.Generator(np.random.PCG64(seed))
    dlog = math.log(w.rmax / w.rmin) / NR
    top = math.log(0.99 * w.r_abs / w.rmin) / dlog
    # cells on both sides of row 32768, or the outer quarter of the rows
    xi = g.uniform(32766.0, 32771.0, n) if few else g.uniform(30000.0, top, n)
    assert top > 32771.0
    r = w.rmin * np.exp(xi * dlog)
    th = g.uniform(1.4, 1.5, n) if few else g.uniform(0.1, 3.0, n)
    u = g.normal(0.0, 3.0, (3, n))
    return w, d, dict(r=r, th=th, ur=u[0], uth=u[1], uph=u[2])


@pytest.mark.parametrize("nth,n,few", [(64, 3000, True), (8, 3000, True), (64, 5000, False),
                                       (8, 257, False)])
def test_fp64_rows_past_32768(nth, n, few):
    oracle.build(force=False)
    w, d, p = tall(nth, n, few, nth + n, W.FP64)
    sim, ora = ffpic.Sim(d, capacity=[n]), oracle.Oracle(d)
    sim.load_particles(0, p)
    ora.load(0, p)
    for _ in range(2):
        sim.run_phases(ffpic.PHASE_PUSH)
        ora.phases(oracle.PHASE_PUSH)
    g, o = sim.particles(0), ora.particles(0)
    assert (o["cell"] // nth >= 32768).sum() > n // 10
    assert np.array_equal(g["cell"], o["cell"])
    currents = [(ffpic.JR, oracle.JR), (ffpic.JPH, oracle.JPH)]
    # columns coarser than 1/16 take the device library's arctangent, a unit of
    # theta from the host's for every fourth particle, and a move there is 1e-5
    # of a column: J_theta compares the two libraries (1e-9, on any row)
    if nth > 50:
        currents.append((ffpic.JTH, oracle.JTH))
    for a, b in currents:
        assert rel(sim.field(a), ora.field(b)) < 2e-10
    # what the node charges add to the Gauss residual: rho of the particles
    assert rel(sim.field(ffpic.GAUSS), ora.gauss()) < 1e-9


@pytest.mark.parametrize("nth,n,few", [(64, 3000, True), (64, 5000, False), (8, 257, False)])
def test_fp32_rows_past_32768(nth, n, few):
    """FP32-mixed, whose state holds the packed cell: load, export, the sorts
    (full, incremental, placed by the push), push, counts and node charges.
    Offsets carry 6e-8 of a cell, so a particle within 1e-3 of them of an edge
    may lie on its other side, a radial move (a tenth of a cell) is known to
    1e-6 and J_r and J_phi to 2e-5; a polar move is 1e-4 of a column, known to
    1e-3 of itself, and J_theta to 1e-2."""
    oracle.build(force=False)
    w, d, p = tall(nth, n, few, nth + n, W.FP32_MIXED)
    d["sort_interval"] = 1
    sim, ora = ffpic.Sim(d, capacity=[n]), oracle.Oracle(d)
    sim.load_particles(0, p)
    ora.load(0, p)
    g, o = sim.particles(0), ora.particles(0)
    assert (o["cell"] // nth >= 32768).sum() > n // 10
    assert np.array_equal(g["cell"], o["cell"])
    assert sim.n(0) == n and sim.diagnostics(ffpic.DIAG_MOMENTS)["alive"] == [n]
    assert rel(sim.field(ffpic.GAUSS), ora.gauss()) < 1e-6
    sim.run_phases(ffpic.PHASE_PUSH)
    ora.phases(oracle.PHASE_PUSH)
    g, o = sim.particles(0), ora.particles(0)
    assert np.sum(g["cell"] != o["cell"]) <= max(1, 1e-3 * n)
    currents = [(ffpic.JR, oracle.JR, 2e-5), (ffpic.JPH, oracle.JPH, 2e-5)]
    if nth > 50:
        currents.append((ffpic.JTH, oracle.JTH, 1e-2))
    for a, b, tol in currents:
        assert rel(sim.field(a), ora.field(b)) < tol
    sim.step(3)
    ora.step(3)
    g, o = sim.particles(0), ora.particles(0)
    assert sim.diagnostics(ffpic.DIAG_MOMENTS)["alive"] == [n]
    assert np.sum(np.sort(g["cell"]) != np.sort(o["cell"])) <= max(1, 4e-3 * n)
