"""Moments brought to the host for any of the four fields, through pinned memory and past it, against
all four: the same bits, and nothing written for a field that is not asked for."""
import numpy as np
import pytest

from paper_2504_20169_amd import lbm
from paper_2504_20169_amd import workloads as wl
from _helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(40, 33), (300, 120), (500, 300)])
def test_any_fields(nx, ny):
    say("moment subsets", nx, ny)
    r = lbm.Run(nx, ny, 0.8, 1.0, 0.05, 0.01, 1.0, lattice=17)
    r.init(*wl.noisy_state(nx, ny, 3, 1.0, 0.05, 0.01, 1.0).as_tuple())
    r.step(3)
    want = r.moments()
    for mask in range(16):
        got = np.full((4, ny, nx), np.nan)
        ptr = [got[k].ctypes.data if mask >> k & 1 else None for k in range(4)]
        assert lbm.load().lbm_moments(r.h, *ptr, 0) == lbm.LBM_OK
        for k in range(4):
            assert np.array_equal(got[k], want[k]) if mask >> k & 1 else np.isnan(got[k]).all(), (mask, k)
    r.close()
