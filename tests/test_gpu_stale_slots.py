"""Slots between the device's count of a species and the host's bound on it:
they hold no particle of the species, whatever their memory holds."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W

pytestmark = pytest.mark.gpu


def leaving(n, precision):
    """A 512^2 dipole with n chargeless particles per species (so that the
    fields of two runs cannot differ by the order of the deposit's additions),
    a tenth of which leave through r_abs within a few steps."""
    w = W.tiny_open_dipole(n)
    w.nr = w.nth = 512
    d = w.desc()
    d["precision"], d["sort_interval"], d["weight"] = precision, 8, [0.0, 0.0]
    parts = []
    for s in range(2):
        p = w.particles(s)
        k = n // 10
        p["r"][:k] = w.r_abs * (1.0 - 1e-4)
        p["ur"][:k] = 10.0
        parts.append(p)
    return d, parts


def fill_and_free(nbytes):
    """Device memory filled with bytes that read as cells far outside the grid
    (row and column 16191), and given back."""
    hip, p = ffpic.lib(), C.c_void_p()
    assert hip.hipMalloc(C.byref(p), C.c_size_t(nbytes)) == 0
    assert hip.hipMemset(p, 0x3f, C.c_size_t(nbytes)) == 0
    assert hip.hipDeviceSynchronize() == 0
    assert hip.hipFree(p) == 0


def same(a, b):
    for s in range(2):
        pa, pb = a.particles(s), b.particles(s)
        assert len(pa["r"]) == len(pb["r"]) > 0
        live = pb["cell"] >= 0
        assert np.array_equal(pa["cell"], pb["cell"])
        for k in ("r", "th", "ur", "uth", "uph"):
            assert np.array_equal(pa[k][live], pb[k][live]), (s, k)
    assert (a.diagnostics(ffpic.DIAG_MOMENTS)["removed"] ==
            b.diagnostics(ffpic.DIAG_MOMENTS)["removed"])


@pytest.mark.parametrize("precision", [W.FP32_MIXED, W.FP64])
def test_restored_with_dead_slots(precision):
    """A checkpoint with dead slots, restored into a new context: its first
    sort drops them, and the second state buffer beyond has never been
    written.  The sorts after it (radix form, placed by the push) keep to the
    slots before the sort."""
    n = (1 << 21) + 300
    d, parts = leaving(n, precision)
    a = ffpic.Sim(d, capacity=[n, n])
    for s in range(2):
        a.load_particles(s, parts[s])
    a.step(3)
    assert (a.particles(0)["cell"] < 0).sum() > n // 100
    image = a.save()
    # memory that the new context's buffers may come from: cells far outside
    fill_and_free(1 << 30)
    b = ffpic.Sim(d, capacity=[n, n])
    b.restore(image)
    for _ in range(3):
        a.step(8)
        b.step(8)
        same(a, b)


@pytest.mark.parametrize("precision", [W.FP64, W.FP32_MIXED])
def test_load_after_removals(precision):
    """A second load after steps whose sorts dropped particles, with the export
    (which lends itself a state buffer) in between: the live particles and the
    new ones, and none of those that had left."""
    oracle.build(force=False)
    n = 6000
    w = W.tiny_open_dipole(n)
    d = w.desc()
    d["precision"], d["sort_interval"] = precision, 2
    d["qm"], d["weight"], d["nspec"] = [1.0], [0.0], 1
    sim, ora = ffpic.Sim(d, capacity=[2 * n]), oracle.Oracle(d)
    p = w.particles(0)
    p["r"][: n // 3] = w.r_abs * (1.0 - 1e-3)
    p["ur"][: n // 3] = 10.0
    first = {k: v[: n - 500] for k, v in p.items()}
    second = {k: v[n - 500:] for k, v in p.items()}
    sim.load_particles(0, first)
    ora.load(0, first)
    sim.step(7)
    ora.step(7)
    before = sim.particles(0)
    assert 0 < (before["cell"] >= 0).sum() < 0.9 * n
    sim.load_particles(0, second)
    ora.load(0, second)
    for steps in (0, 4):
        sim.step(steps)
        ora.step(steps)
        g, o = sim.particles(0), ora.particles(0)
        gl, ol = g["cell"] >= 0, o["cell"] >= 0
        assert gl.sum() == ol.sum()
        assert sim.diagnostics(ffpic.DIAG_MOMENTS)["alive"] == [int(ol.sum())]
        gu, ou = (np.sort(x["ur"][m]) for x, m in ((g, gl), (o, ol)))
        # eleven FP32 steps, some ten roundings of 6e-8 each; FP64: 1e-16
        tol = 1e-5 if precision == W.FP32_MIXED else 1e-12
        assert np.abs(gu - ou).max() < tol * np.abs(ou).max()
        if precision == W.FP64:
            assert np.array_equal(np.sort(g["cell"][gl]), np.sort(o["cell"][ol]))
