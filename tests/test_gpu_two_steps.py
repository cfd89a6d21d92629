"""Two-step passes (the default schedule of large FP64 and FP32 runs) against single steps: the same
expressions in the same order, so the same bits in the moments, the populations and the PML field,
for every stencil, edge kind and step count, at grids whose last strip, last tile and last turn are
full, ragged or one node wide; in a group, where small members take pairs with a large one and stop
at their own counts; and across a checkpoint."""
import numpy as np
import pytest

from paper_2504_20169_amd import lbm
from paper_2504_20169_amd import workloads as wl
from _helpers import say

pytestmark = pytest.mark.gpu

# (lattice, storage, nx, ny, bcx, bcy, W, step calls)
CASES = [
    (37, "f64", 700, 641, "nrbc", "nrbc", 9, (1, 2, 3, 6, 37)),
    (37, "f64", 4300, 103, "zg", "periodic", 20, (5, 4)),     # the lowest interior taken in pairs, nearly
    (37, "f64", 102, 4200, "periodic", "nrbc", 0, (35,)),
    (37, "f64", 681, 702, "periodic", "periodic", 0, (7, 64)),
    (37, "f64", 672, 701, "zg", "nrbc", 1, (33,)),
    (37, "f32", 1024, 903, "nrbc", "zg", 3, (3, 34)),
    (37, "f32", 1001, 997, "periodic", "zg", 0, (64, 1, 3)),
    (17, "f64", 731, 653, "nrbc", "nrbc", 16, (3, 65)),
    (17, "f32", 1107, 1003, "zg", "zg", 4, (12,)),
    (9, "f64", 701, 689, "nrbc", "periodic", 12, (6, 31)),
    (9, "f32", 1203, 909, "nrbc", "nrbc", 5, (37,)),
]


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


@pytest.mark.parametrize("case", CASES, ids=lambda c: "q%d-%s-%dx%d-%s-%s-W%d" % c[:7])
def test_pairs_equal_single_steps(case):
    say("two-step case", case)
    out = []
    for overlap in (0, 2):
        r = _make(*case[:7], seed=5, overlap=overlap)
        for n in case[7]:
            r.step(n)
        assert r.check() == lbm.LBM_OK
        out.append(_state(r))
        r.close()
    assert _same(*out), case


@pytest.mark.parametrize("lattice", [37, 17, 9])
def test_small_members_of_a_paired_group_equal_alone(lattice):
    """Interiors of 96 cells and up beside a large run: strips and tiles a few nodes wide, CBC (A) and
    PML-moment targets, and stops close together and far apart."""
    cases = [(700, 650, "zg", "zg", 4, {}, 40), (96, 104, "nrbc", "nrbc", 6, {}, 17),
             (161, 97, "periodic", "nrbc", 5, {}, 9), (109, 155, "zg", "periodic", 1, {}, 40),
             (120, 131, "nrbc", "nrbc", 8, dict(outlet="nrbc_a"), 16),
             (113, 99, "nrbc", "nrbc", 7, dict(terms=2), 0), (102, 102, "periodic", "periodic", 0, {}, 1)]
    alone = []
    for k, (nx, ny, bx, by, W, kw, n) in enumerate(cases):
        r = _make(lattice, "f64", nx, ny, bx, by, W, 30 + k, overlap=0, **kw)
        r.step(n + 5)
        alone.append(_state(r))
        r.close()
    g = lbm.Group()
    runs = [_make(lattice, "f64", nx, ny, bx, by, W, 30 + k, **kw)
            for k, (nx, ny, bx, by, W, kw, n) in enumerate(cases)]
    for r in runs:
        g.add(r)
    say("paired group", lattice)
    g.step(steps=np.array([c[-1] for c in cases]))
    g.step(nsteps=5)
    g.synchronize()
    for r, a, c in zip(runs, alone, cases):
        assert r.step_count == c[-1] + 5
        assert _same(_state(r), a), c
    g.close()


def test_checkpoint_between_pairs(tmp_path):
    """A call of odd length leaves the population buffers and the moment strips out of step with
    each other; a checkpoint carries both."""
    a = _make(37, "f64", 700, 641, "nrbc", "nrbc", 9, seed=8)
    a.step(5)
    a.save(tmp_path / "c")
    a.step(12)
    b = _make(37, "f64", 700, 641, "nrbc", "nrbc", 9, seed=9)
    b.load(tmp_path / "c")
    assert b.step_count == 5
    b.step(12)
    assert _same(_state(a), _state(b))
    a.close()
    b.close()
