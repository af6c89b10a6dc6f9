"""The two forms of the incremental sort (buckets up to 2^21 slots, radix
passes above) against the stable order of the cells: the line between
them, buckets that are counted and ones that are sorted, a single particle.
The order is exact, so nothing is allowed to differ."""
import numpy as np
import pytest

from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W
from test_gpu_parity import check_incremental_sort

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [W.FP32_MIXED, W.FP64])
@pytest.mark.parametrize("nr,nth,n", [
    (24, 24, 2),                  # one particle of each species
    (24, 24, 150_000),            # a few cells hold all: buckets of thousands
    (61, 33, 200_000),            # buckets on both sides of 1024 movers
    (256, 512, 2 * ((1 << 21) - 5)),   # just below the line
    (256, 512, 2 * ((1 << 21) + 1)),   # above it: radix passes
])
def test_incremental_sort_forms(precision, nr, nth, n):
    ffpic.lib()
    w = W.tiny_dipole(n // 2)
    w.nr, w.nth = nr, nth
    w.sheet_rmin, w.sheet_rmax = 1.05, 1.6
    check_incremental_sort(w, precision, moved=(0.0, 1.0))


@pytest.mark.parametrize("nr,n", [(96, 50_001), (512, (1 << 21) + 3)])
def test_sort_placed_by_the_push_fp64(nr, n):
    """In a step that sorts and pushes, the FP64 push writes its particles in
    the sorted order too (buckets, radix passes).  A twin takes the sort as a
    phase of its own, so that the sort places them: bit for bit the same.  The
    particles carry no charge, so the order of the deposit's additions cannot
    make the fields differ."""
    w = W.tiny_open_dipole(n)
    w.nr = w.nth = nr
    w.sheet_rmin, w.sheet_rmax = 1.05, 4.0
    d = w.desc()
    d["precision"] = W.FP64
    d["sort_interval"] = 2
    d["weight"] = [0.0, 0.0]
    a = ffpic.Sim(d, capacity=[n, n])
    b = ffpic.Sim(d, capacity=[n, n])
    for sim in (a, b):
        sim.record_sort(True)
        for s in range(2):
            sim.load_particles(s, w.particles(s))
    rest = (ffpic.PHASE_INJECT | ffpic.PHASE_EXTRACT | ffpic.PHASE_PUSH | ffpic.PHASE_PAIRS |
            ffpic.PHASE_FIELDS)
    for cycle in range(3):
        a.step(2)
        b.run_phases(ffpic.PHASE_MASK)
        b.run_phases(ffpic.PHASE_SORT)
        b.run_phases(rest)
        b.run_phases(ffpic.PHASE_MASK | rest)
        for s in range(2):
            pa, pb = a.particles(s), b.particles(s)
            assert len(pa["r"]) == len(pb["r"]) > 0
            live = pb["r"] > 0
            assert np.array_equal(pa["r"], pb["r"])
            for k in ("cell", "th", "ur", "uth", "uph"):
                assert np.array_equal(pa[k][live], pb[k][live]), (cycle, s, k)
            assert np.array_equal(a.sort_permutation(s), b.sort_permutation(s)), (cycle, s)
        for c in (ffpic.ER, ffpic.BTH, ffpic.EPH):
            assert np.array_equal(a.field(c), b.field(c))
