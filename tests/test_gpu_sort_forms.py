"""The two forms of the incremental sort (buckets up to 2^21 slots, radix
passes above) against the stable order of the cells: the line between
them, buckets that are counted and ones that are sorted, a single particle.
The order is exact, so nothing is allowed to differ."""
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
