"""Slots between the device's count of a species and the host's bound on it:
they hold no particle of the species, whatever their memory holds."""
import ctypes as C

import numpy as np
import pytest

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
