"""Moments, error norms and the health check brought to the host (through pinned memory up to a
size, straight into the caller's arrays above it) against the same fields on the device: the same
bits, at grids on both sides of the line (32 KiB nodes of four moments; 43688 nodes of three
references) and on one run that grows and shrinks what it brings."""
import numpy as np
import pytest

from paper_2504_20169_amd import lbm
from paper_2504_20169_amd import workloads as wl
from _helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(8, 8), (256, 128), (331, 99), (344, 127), (331, 132), (400, 120)])
def test_host_results_equal_device_results(nx, ny):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("PyTorch in this process sees no HIP device")
    say("host copies", nx, ny)
    r = lbm.Run(nx, ny, 0.8, 1.0, 0.05, 0.01, 1.0)
    r.set_bc(15, "periodic")
    state = wl.noisy_state(nx, ny, 7, 1.0, 0.05, 0.01, 1.0)
    r.init(*state.as_tuple())
    refs = [np.ascontiguousarray(a) for a in (state.rho, state.ux, state.T)]
    rdev = [torch.from_numpy(a).cuda() for a in refs]
    for _ in range(2):
        r.step(3)
        assert r.check() == lbm.LBM_OK
        dev = [torch.full((ny, nx), float("nan"), dtype=torch.float64, device="cuda") for _ in range(4)]
        norms = torch.full((3,), float("nan"), dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        r.moments_device(*[d.data_ptr() for d in dev])
        r.error_norms_noalloc(*[d.data_ptr() for d in rdev], norms.data_ptr())
        r.synchronize()
        assert np.array_equal(r.error_norms(*refs), norms.cpu().numpy())
        for got, want in zip(r.moments(), dev):
            assert np.array_equal(got, want.cpu().numpy())
    r.close()
