"""FP32 push against the oracle at the sizes that choose its chunks (one, two,
four and eight particles per thread, at 1536, 4096 and 24576 rounds of 256
slots), their remainders, boxes within and beyond the LDS patches (in parts and
from device memory), next to the axes, with the shell and radiation reaction.

Tolerances are those of one FP32 push: offsets are held to 2^-24 of a cell, so
a particle within rounding of an edge may lie on its other side (1e-3 of
them at most), momenta carry some ten roundings of 6e-8 and the fields' and
positions' rounding (1e-5 of the largest), and currents, sums of moves of about
a tenth of a cell known to 1e-6, agree to 2e-5 of the largest."""
import math

import numpy as np
import pytest

import oracle
from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W
from parity_util import rel
from test_gpu_push64 import scattered

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,nth,n,spread", [
    (64, 96, 1, True), (64, 96, 255, True), (64, 96, 257, False), (12, 9, 5_000, True),
    (300, 517, 40_001, True),                  # boxes beyond the patches
    (64, 96, 1536 * 256 + 3, False), (300, 517, 1536 * 256 + 3, True),
    (64, 96, 4096 * 256 + 259, True),
    (300, 517, 24576 * 256 + 5, True),         # chunks in parts where a row ends
])
def test_push32_chunks(nr, nth, n, spread):
    oracle.build(force=False)
    w = W.tiny_open_dipole(n)
    w.nr, w.nth = nr, nth
    w.rr_coef = 0.02
    w.shell_r = 1.5
    w.qm, w.weight = (1.0,), (1e-4,)
    d = w.desc()
    d["precision"] = W.FP32_MIXED
    sim, ora = ffpic.Sim(d, capacity=[n]), oracle.Oracle(d)
    p = scattered(w, n, nr + nth + n, spread)
    sim.load_particles(0, p)
    ora.load(0, p)
    sim.run_phases(ffpic.PHASE_PUSH)
    ora.phases(oracle.PHASE_PUSH)
    g, o = sim.particles(0), ora.particles(0)
    assert len(g["r"]) == len(o["r"])
    assert np.sum(g["cell"] != o["cell"]) <= 1e-3 * len(o["r"])
    same = (o["cell"] >= 0) & (g["cell"] == o["cell"])
    cell = math.log(w.rmax / w.rmin) / nr, math.pi / nth
    assert np.abs(np.log(g["r"][same] / o["r"][same])).max(initial=0.0) < 1e-5 * cell[0]
    assert np.abs(g["th"][same] - o["th"][same]).max(initial=0.0) < 1e-5 * cell[1]
    for k in ("ur", "uth", "uph"):
        scale = np.abs(o[k][same]).max(initial=1.0)
        assert np.abs(g[k][same] - o[k][same]).max(initial=0.0) < 1e-5 * scale, k
    for a, b in ((ffpic.JR, oracle.JR), (ffpic.JTH, oracle.JTH), (ffpic.JPH, oracle.JPH)):
        assert rel(sim.field(a), ora.field(b)) < 2e-5
    removed = np.abs(sim.diagnostics(0)["removed"][0] - np.asarray(ora.removed(0)))
    assert removed.max() <= 1e-5 * n + 1
