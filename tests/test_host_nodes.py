"""The FP64 push forms the polar nodes it settles cells by as j dth, the sort and
the export read them from the table: the two are equal bit for bit (CPU only)."""
import math

import numpy as np
import pytest

from paper_2406_14512_amd import ffpic
from paper_2406_14512_amd import workloads as W


@pytest.mark.parametrize("nth", [2, 3, 7, 50, 51, 96, 300, 517, 1024, 4096, 30_011, 65_535])
def test_polar_nodes_are_products(nth):
    w = W.tiny_dipole(10)
    w.nr, w.nth = 4, nth
    thn = ffpic.host_table(w.desc(), ffpic.TAB_THN)
    assert np.array_equal(thn, np.arange(nth + 1) * (math.pi / nth))
