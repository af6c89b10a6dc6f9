"""Pushes of particles that cross or land next to the polar axis."""
import math

import numpy as np
import pytest

import oracle
from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W

pytestmark = pytest.mark.gpu


def free(precision, n, scale=1.0, **over):
    """No fields, one species without charge: straight lines."""
    w = W.tiny_dipole(n)
    w.rmin, w.rmax, w.r_abs, w.r_lc = 1.0 * scale, 10.0 * scale, 9.0 * scale, 3.0 * scale
    w.qm, w.weight = (1.0,), (0.0,)
    for k, v in over.items():
        setattr(w, k, v)
    d = w.desc()
    d["precision"], d["init"] = precision, W.INIT_ZERO
    return w, d


@pytest.mark.parametrize("precision", [W.FP32_MIXED, W.FP64])
@pytest.mark.parametrize("scale,start", [(1.0, 1.0), (1.0, 1.5), (1e-6, 1.5)])
def test_momentum_kept_on_landing_on_the_axis(precision, scale, start):
    """Particles that move in their meridional plane towards the axis, their
    speeds so close to the one that ends on it that in FP32 some end at a
    distance of exactly zero (from r = 1, where r sin theta is not rounded):
    the momentum keeps its size (2e-6: some ten roundings of 6e-8 and the
    rotation's series)."""
    n = 200_000
    w, d = free(precision, n, scale)
    dt, dth = oracle.timestep(d), math.pi / w.nth
    r, th, vr = start * scale, 0.1 * dth, 0.05
    # r sin th + dt (vr sin th + vth cos th) = 0, within 3e-6
    vth = -(r / dt + vr) * math.tan(th) * (1.0 + np.linspace(-3e-6, 3e-6, n))
    v2 = vr * vr + vth * vth
    assert v2.max() < 0.8
    ur, uth = vr / np.sqrt(1.0 - v2), vth / np.sqrt(1.0 - v2)
    zero = np.zeros(n)
    sim = ffpic.Sim(d, capacity=[n])
    sim.load_particles(0, dict(r=zero + r, th=zero + th, ur=ur, uth=uth, uph=zero))
    sim.run_phases(ffpic.PHASE_PUSH)
    p = sim.particles(0)
    assert len(p["r"]) == n and (p["cell"] >= 0).all()
    size = np.sqrt(p["ur"] ** 2 + p["uth"] ** 2 + p["uph"] ** 2)
    # (one cell: the load's sort keeps the order)
    assert np.abs(size / np.hypot(ur, uth) - 1.0).max() < 2e-6


@pytest.mark.parametrize("nth", [51, 128, 1024])
def test_polar_angle_next_to_the_axis(nth):
    """FP64: the new angle of particles that end in the first column is the
    rounded angle of the end point, as the oracle's arctangent gives it, however
    close to the axis they end.  Both round the same end point, so they differ by
    one unit in the last place at most, but where the sine or cosine of the old
    angle was rounded differently (a few in a thousand, and the difference grows
    as the end nears the axis): 99 % within a unit."""
    oracle.build(force=False)
    n = 100_000
    w, d = free(W.FP64, n, nr=nth, nth=nth)
    g = np.random.Generator(np.random.PCG64(nth))
    dt, dth = oracle.timestep(d), math.pi / nth
    th = g.uniform(0.0, min(2.0, 2.0 * dt / (1.1 * dth)) * dth, n)
    u = g.normal(0.0, 3.0, (3, n))
    u[2, : n // 2] = 0.0                       # in the meridional plane
    p = dict(r=np.exp(g.uniform(math.log(1.1), math.log(1.5), n)), th=th, ur=u[0], uth=u[1],
             uph=u[2])
    sim, ora = ffpic.Sim(d, capacity=[n]), oracle.Oracle(d)
    sim.load_particles(0, p)
    ora.load(0, p)
    sim.run_phases(ffpic.PHASE_PUSH)
    ora.phases(oracle.PHASE_PUSH)
    a, b = sim.particles(0), ora.particles(0)
    first = (b["r"] > 0) & (b["th"] < dth)
    units = np.abs(a["th"] - b["th"])[first] / np.spacing(b["th"][first])
    assert first.sum() > n // 4
    assert (units > 1.0).mean() < 0.01, (units > 1.0).mean()
