"""What two-step passes (the default schedule of large FP64 and FP32 runs) leave behind and meet beside
the plain runs: thin grids, targets formed ahead, small members of a group, checkpoints after an odd
number of passes, the NaN canary.  That the cases do take
pairs is asked of the host's schedule in test_host_runtime.py."""
import struct

import numpy as np
import pytest

from paper_2504_20169_amd import lbm
from _helpers import say
from pair_cases import GROUP, SINGLE, make

pytestmark = pytest.mark.gpu


def _state(r):
    return list(r.moments()) + [r.populations(), r.pml_q()]


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("steps", [5, 7, 10, 12])
def test_checkpoint_has_one_parity(tmp_path, steps):
    """After an odd number of two-step passes (7 and 12 steps: 3 passes and a step, 5 and two) the
    population buffers have changed roles another number of times than the moment strips.  The
    file still names one buffer for both, the one of the step's parity, and a run that loads it
    goes on with the same bits."""
    say("checkpoint after", steps, "steps")
    a = make(9, "f64", 690, 671, "nrbc", "nrbc", 9, {}, seed=8)
    a.step(steps)
    a.save(tmp_path / "c")
    head = (tmp_path / "c").read_bytes()[:88]
    assert struct.unpack_from("<q", head, 80)[0] == steps
    assert struct.unpack_from("<i", head, 60)[0] == steps & 1
    b = make(9, "f64", 690, 671, "nrbc", "nrbc", 9, {}, seed=9)
    b.step(4)
    b.load(tmp_path / "c")
    assert b.step_count == steps and _same(_state(a), _state(b))
    for r in (a, b):
        r.step(9)
    assert _same(_state(a), _state(b))
    a.close()
    b.close()


def _ids(c):
    return "q%d-%s-%dx%d-%s-%s-W%d%s" % (c[:7] + ("".join("-%s%s" % kv for kv in c[7].items()),))


@pytest.mark.parametrize("case", SINGLE, ids=_ids)
def test_canary_in_pairs_leaves_the_bits(case):
    """Every buffer that a two-step pass or one of its steps writes in full, the bands of the level
    between among them, filled with NaN before: the same bits as without, and finite."""
    say("canary in pairs", case)
    out = []
    for flags in (0, lbm.LBM_DEBUG_POISON):
        r = make(*case, seed=12)
        r.set_debug(flags)
        r.step(7)
        assert r.check() == lbm.LBM_OK
        out.append(_state(r))
        r.close()
    assert all(np.isfinite(x).all() for x in out[1])
    assert _same(*out)


def test_canary_in_a_paired_group():
    out = []
    for flags in (0, lbm.LBM_DEBUG_POISON):
        g = lbm.Group()
        runs = [make(37, "f64", *c, seed=40 + k) for k, (c, n) in enumerate(GROUP)]
        runs[2].set_debug(flags)
        for r in runs:
            g.add(r)
        say("canary in a paired group", flags)
        g.step(steps=np.array([n for c, n in GROUP]))
        g.synchronize()
        assert not g.check().any()
        out.append([_state(r) for r in runs])
        g.close()
        for r in runs:
            r.close()
    for a, b in zip(*out):
        assert all(np.isfinite(x).all() for x in b) and _same(a, b)


@pytest.mark.parametrize("case", SINGLE, ids=_ids)
def test_pairs_equal_single_steps_for_thin_grids_and_formed_targets(case):
    say("pairs against single steps", case)
    out = []
    for overlap in (0, 2):
        r = make(*case, seed=13, overlap=overlap)
        for n in (6, 35):
            r.step(n)
        assert r.check() == lbm.LBM_OK
        out.append(_state(r))
        r.close()
    assert _same(*out)


@pytest.mark.parametrize("lattice", [37, 17, 9])
def test_members_of_a_paired_group_equal_alone(lattice):
    """Strips and tiles a few nodes wide beside a large run's, stops close together and far apart."""
    alone = []
    for k, (c, n) in enumerate(GROUP):
        r = make(lattice, "f64", *c, seed=30 + k, overlap=0)
        r.step(n + 23)
        alone.append(_state(r))
        r.close()
    g = lbm.Group()
    runs = [make(lattice, "f64", *c, seed=30 + k) for k, (c, n) in enumerate(GROUP)]
    for r in runs:
        g.add(r)
    say("members of a paired group", lattice)
    g.step(steps=np.array([n for c, n in GROUP]))
    g.step(nsteps=23)
    g.synchronize()
    for r, a, (c, n) in zip(runs, alone, GROUP):
        assert r.step_count == n + 23 and _same(_state(r), a), c
    g.close()
    for r in runs:
        r.close()
