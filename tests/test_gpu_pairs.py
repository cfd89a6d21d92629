"""What two-step passes (the default schedule of large FP64 and FP32 runs) leave behind and meet beside
the plain runs: checkpoints after an odd number of passes."""
import struct

import numpy as np
import pytest

from paper_2504_20169_amd import lbm
from paper_2504_20169_amd import workloads as wl
from _helpers import say

pytestmark = pytest.mark.gpu


def _make(lattice, storage, nx, ny, bcx, bcy, W, seed, overlap=2, outlet=None, terms=0):
    r = lbm.Run(nx, ny, 0.8, 1.0, 0.05, 0.01, 1.0, storage=storage, lattice=lattice)
    r.set_bc(lbm.LBM_XMIN | lbm.LBM_XMAX, bcx)
    r.set_bc(lbm.LBM_YMIN | lbm.LBM_YMAX, bcy)
    if outlet:
        r.set_bc(lbm.LBM_XMAX, outlet)
    mask = (3 if bcx != "periodic" else 0) | (12 if bcy != "periodic" else 0)
    if W and mask:
        r.set_pml(mask, W, 0.002)
    if terms:
        r.set_nrbc_pml_terms(terms)
    r.set_launch(overlap=overlap)
    Nx, Ny = r.grid()
    r.init(*wl.noisy_state(Nx, Ny, seed, 1.0, 0.05, 0.01, 1.0).as_tuple())
    return r


def _state(r):
    return list(r.moments()) + [r.populations(), r.pml_q()]


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


def _paired(r, storage):
    """The run alone takes its steps in pairs (by its interior and frame nodes)."""
    interior, frame = r.node_classes()[:2]
    return interior >= (400000 + frame if storage == "f64" else 800000 + 5 * frame)


@pytest.mark.parametrize("steps", [5, 7, 10, 12])
def test_checkpoint_has_one_parity(tmp_path, steps):
    """After an odd number of two-step passes (7 and 12 steps: 3 passes and a step, 5 and two) the
    population buffers have changed roles another number of times than the moment strips.  The
    file still names one buffer for both, the one of the step's parity, and a run that loads it
    goes on with the same bits."""
    say("checkpoint after", steps, "steps")
    a = _make(9, "f64", 690, 671, "nrbc", "nrbc", 9, seed=8)
    assert _paired(a, "f64")
    a.step(steps)
    a.save(tmp_path / "c")
    head = (tmp_path / "c").read_bytes()[:88]
    assert struct.unpack_from("<q", head, 80)[0] == steps
    assert struct.unpack_from("<i", head, 60)[0] == steps & 1
    b = _make(9, "f64", 690, 671, "nrbc", "nrbc", 9, seed=9)
    b.step(4)
    b.load(tmp_path / "c")
    assert b.step_count == steps and _same(_state(a), _state(b))
    for r in (a, b):
        r.step(9)
    assert _same(_state(a), _state(b))
    a.close()
    b.close()
