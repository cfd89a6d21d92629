"""Boundary launches that split a node's populations over four waves (taken while their blocks are
all on the device at once) against those of whole nodes: the same expressions in the same order, so
the same bits.  A small run alone takes the split kernels, the same run in a group with a larger one
the others; rings and frames here end within a block, just past one, and fill a few exactly."""
import numpy as np
import pytest

from paper_2504_20169_amd import lbm
from paper_2504_20169_amd import workloads as wl
from _helpers import say

pytestmark = pytest.mark.gpu

# nx, ny, edges along x and y, PML width, options
SMALL = [
    (8, 9, "zg", "zg", 0, {}),
    (64, 7, "periodic", "nrbc", 0, {}),
    (32, 32, "nrbc", "nrbc", 6, {}),
    (47, 21, "nrbc", "zg", 3, {}),
    (7, 128, "nrbc", "periodic", 20, {}),
    (61, 40, "nrbc", "nrbc", 9, dict(outlet="nrbc_a")),
    (40, 33, "nrbc", "nrbc", 8, dict(terms=2)),
]
# side of a run whose boundary alone is past the line
LARGE = {(37, "f64"): 470, (37, "f32"): 900, (37, "f16"): 900, (17, "f64"): 700, (17, "f32"): 1000, (17, "f16"): 1000}


def _run(lattice, storage, nx, ny, bcx, bcy, W, kw, seed, overlap):
    r = lbm.Run(nx, ny, 0.8, 1.0, 0.05, 0.01, 1.0, storage=storage, lattice=lattice)
    r.set_bc(lbm.LBM_XMIN | lbm.LBM_XMAX, bcx)
    r.set_bc(lbm.LBM_YMIN | lbm.LBM_YMAX, bcy)
    if "outlet" in kw:
        r.set_bc(lbm.LBM_XMAX, kw["outlet"])
    mask = (3 if bcx != "periodic" else 0) | (12 if bcy != "periodic" else 0)
    if W:
        r.set_pml(mask, W, 0.002)
    if "terms" in kw:
        r.set_nrbc_pml_terms(kw["terms"])
    r.set_launch(overlap=overlap)
    Nx, Ny = r.grid()
    r.init(*wl.noisy_state(Nx, Ny, seed, 1.0, 0.05, 0.01, 1.0).as_tuple())
    return r


def _state(r):
    return list(r.moments()) + [r.populations(), r.pml_q()]


@pytest.mark.parametrize("lattice,storage", list(LARGE), ids=lambda v: str(v))
@pytest.mark.parametrize("overlap", [0, 2])
def test_split_boundary_equals_whole_nodes(lattice, storage, overlap):
    alone = []
    for k, c in enumerate(SMALL):
        say("small boundary", lattice, storage, overlap, c)
        r = _run(lattice, storage, *c, seed=60 + k, overlap=overlap)
        r.step(5)
        alone.append(_state(r))
        r.close()
    g = lbm.Group()
    side = LARGE[lattice, storage]
    runs = [_run(lattice, storage, *c, seed=60 + k, overlap=2) for k, c in enumerate(SMALL)]
    runs.append(_run(lattice, storage, side, side, "nrbc", "nrbc", 20, {}, seed=59, overlap=2))
    for r in runs:
        g.add(r)
    g.step(nsteps=5)
    g.synchronize()
    for r, a, c in zip(runs, alone, SMALL):
        assert all(np.array_equal(x, y) for x, y in zip(_state(r), a)), c
    g.close()
