"""The library's host side on the CPU, under a stand-in for the HIP runtime (tests/host/fake_hip.cpp)
that counts memory and logs launches, copies and graphs instead of running kernels: what it does
when device memory runs out, that it waits before it frees, and which kernels a schedule has."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_2504_20169_amd import lbm

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists(lbm.LIB_PATH),
                                reason="g++ or the library is missing")

PRELUDE = """
import ctypes, sys
sys.path[:0] = [%r, %r]
import numpy as np
from paper_2504_20169_amd import lbm
F = ctypes.CDLL(%r)
F.fake_log.restype = ctypes.c_char_p
F.fake_used.restype = F.fake_pinned.restype = ctypes.c_size_t
F.fake_limit.argtypes = [ctypes.c_size_t]
F.fake_refuse.argtypes = [ctypes.c_size_t, ctypes.c_size_t]
log = lambda: F.fake_log().decode().split("\\n")
def run(nx, ny, W=0, bc="periodic", **kw):
    r = lbm.Run(nx, ny, 0.8, **kw)
    r.set_bc(15, bc)
    if W:
        r.set_pml(15, W, 0.01)
    return r
def init(r):
    r.init(1.0, 0.0, 0.0, 1.0)
    return r
def pairs(n=8, of=None):
    log()
    (of.step(nsteps=n) if isinstance(of, lbm.Group) else of.step(n))
    return sum("k_core" in l for l in log())
"""


@pytest.fixture(scope="session")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "host", "fake_hip.cpp")],
                   check=True)
    return so


def _play(fake, code):
    res = subprocess.run([sys.executable, "-c", PRELUDE % (ROOT, HERE, fake) + code + "\nprint('played')"],
                         env=dict(os.environ, LD_PRELOAD=fake), capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and res.stdout.endswith("played\n"), res.stdout[-1500:] + res.stderr[-3000:]


def test_bands_are_taken_last_and_only_where_pairs_are(fake):
    """A run that pairs alone holds bands, one that does not holds what its footprint without them
    says; with memory for all but the bands it initialises, takes single steps, and later calls see
    no error of the refused allocation."""
    _play(fake, """
a = init(run(6500, 103, W=4, bc="zg"))
with_bands = F.fake_used()
assert pairs(of=a) == 3 and a.footprint() + 8192 >= with_bands
a.close()
assert F.fake_used() == 0
r = run(6500, 103, W=4, bc="zg")
peak = r.footprint()
F.fake_limit(with_bands - 1)         # the staging of the fields is less than the bands
r.init(1.0, 0.0, 0.0, 1.0)
assert r.footprint() < peak and F.fake_used() < with_bands
assert pairs(of=r) == 0
r.close()
for spare in (0, 1000, 1 << 24):     # the bands fit until the staging is asked for, or beside it
    F.fake_limit(with_bands + spare)
    r = init(run(6500, 103, W=4, bc="zg"))
    assert F.fake_used() == with_bands and pairs(of=r) == 3
    r.close()
F.fake_limit(1 << 62)
b = init(run(1024, 1024, W=32, bc="nrbc", storage="f32"))     # no pairs by itself
assert F.fake_used() <= b.footprint() - 4 * 8 * 1088 * 1088 + 8192
assert pairs(of=b) == 0
""")


def test_a_result_makes_bands_give_way(fake):
    """Device scratch of a call that finds no memory takes that of the bands: what fitted without
    them still does."""
    _play(fake, """
a = init(run(6500, 103, W=4, bc="zg"))
assert pairs(of=a) == 3
F.fake_limit(F.fake_used())          # nothing left
a.moments()
assert pairs(of=a) == 0 and a.footprint() >= F.fake_used()
a.moments()
""")


def test_bands_of_a_group(fake):
    """Members that do not pair alone hold bands while they are in a group that does, and none after;
    if one of them finds no memory for its bands the group takes single steps."""
    _play(fake, """
big = init(run(720, 700, lattice=9))
small = init(run(120, 110, lattice=9))
alone = F.fake_used()
g = lbm.Group()
g.add(big); g.add(small)
assert pairs(of=g) == 3 and F.fake_used() > alone
assert pairs(of=g) == 3
held = F.fake_used()
g.remove(small)
assert F.fake_used() < held and pairs(of=g) == 3
g.add(small)
F.fake_refuse(20000, 1 << 62)        # no more bands
assert pairs(of=g) == 0
F.fake_refuse(1 << 62, 1 << 62)
g.remove(small); g.add(small)
assert pairs(of=g) == 3
g.close()
assert pairs(of=big) == 3 and pairs(of=small) == 0
""")


def test_graphs_are_destroyed_when_they_are_done(fake):
    """A new launch configuration or debug flag drops the captured steps once those in flight have
    ended, on the run's stream; the same configuration keeps them."""
    _play(fake, """
for kw, nx in (({}, 64), (dict(lattice=9), 700)):
    r = init(run(nx, nx, **kw))
    for change in (lambda: r.set_launch(bulk_tx=128), lambda: r.set_launch(bulk_tx=128, split=2),
                   lambda: r.set_launch(graph_steps=16), lambda: r.set_debug(lbm.LBM_DEBUG_RANGES),
                   lambda: r.set_debug(0), r.close):
        r.step(70)
        assert "instantiate" in log()
        change()
        assert "GRAPH DESTROYED IN FLIGHT" not in log(), change
r = init(run(64, 64))
r.step(70)
log()
r.set_launch()
r.step(70)
assert "instantiate" not in log()
g = lbm.Group()
g.add(r)
g.step(nsteps=70)
g.set_launch(bulk_tx=256)
g.step(nsteps=70)
g.remove(r)
g.close()
assert "GRAPH DESTROYED IN FLIGHT" not in log()
""")


def test_where_boundary_launches_split_a_node(fake):
    """Single steps of thick frames around little interior take whole nodes unless a side is
    characteristic; thin frames, and those of a large interior, are split over four waves."""
    _play(fake, """
for nx, ny, bx, by, W, storage, lattice, split in (
        (591, 41, "periodic", "zg", 52, "f32", 37, False), (591, 41, "periodic", "nrbc", 52, "f32", 37, True),
        (100, 100, "zg", "zg", 60, "f16", 37, False), (100, 100, "nrbc", "nrbc", 60, "f16", 37, True),
        (156, 1183, "zg", "periodic", 15, "f32", 37, False), (350, 350, "zg", "zg", 20, "f32", 37, True),
        (300, 80, "zg", "zg", 32, "f64", 17, False), (300, 80, "nrbc", "nrbc", 32, "f64", 17, True),
        (300, 80, "zg", "zg", 32, "f16", 17, True), (156, 1183, "zg", "periodic", 15, "f16", 17, False),
        (300, 80, "zg", "zg", 32, "f64", 37, True), (156, 1183, "zg", "periodic", 15, "f64", 17, True), (500, 500, "zg", "zg", 20, "f32", 17, False),
        (600, 600, "periodic", "periodic", 0, "f64", 37, True), (800, 800, "nrbc", "nrbc", 16, "f32", 37, False),
        (800, 800, "nrbc", "nrbc", 16, "f16", 37, True), (800, 800, "nrbc", "nrbc", 10, "f32", 37, True), (100, 100, "zg", "zg", 60, "f32", 9, False)):
    r = lbm.Run(nx, ny, 0.8, storage=storage, lattice=lattice)
    r.set_bc(3, bx); r.set_bc(12, by)
    if W:
        r.set_pml(3 * (bx != "periodic") | 12 * (by != "periodic"), W, 0.01)
    init(r)
    log()
    r.step(2)
    names = " ".join(log())
    assert ("k_frame_split" in names, "k_small_step" in names) == (split, split), (nx, ny, bx, by, W, storage, lattice)
    assert ("k_phase_a_bulk" in names) == (not split)
    r.close()
""")


def test_frame_stores_stream_in_small_sets(fake):
    """The whole-node frame kernel streams FP64 always, FP32 and FP16 while the populations of the run
    or group are few, FP16 again where they are many."""
    _play(fake, """
streams = lambda: "ELb1E" in [l for l in log() if "k_frame" in l][-1]
for nx, ny, storage, lattice, want in ((65, 1311, "f32", 9, True), (700, 700, "f32", 9, True), (1200, 1200, "f32", 9, True), (1400, 1400, "f32", 9, False),
                                       (500, 1500, "f32", 9, False), (1500, 500, "f32", 9, True), (900, 900, "f64", 9, True),
                                       (500, 500, "f16", 9, True), (1100, 1100, "f16", 9, False), (1780, 1780, "f16", 37, False),
                                       (1830, 1830, "f16", 37, True), (2000, 300, "f32", 37, False)):
    r = init(run(nx, ny, W=12, bc="nrbc", storage=storage, lattice=lattice))
    r.step(1)
    assert streams() == want, (nx, ny, storage)
    r.close()
g = lbm.Group()
small = [init(run(200, 200, W=12, bc="nrbc", storage="f32", lattice=9)) for _ in range(40)]
for k, r in enumerate(small):
    g.add(r)
    g.step(nsteps=1)
    assert streams() == (k < 35), k
""")


def test_pinned_memory_is_bounded_and_moments_copy_what_is_asked(fake):
    """The runs of a process keep at most 64 MiB of pinned memory, given back with them; the others'
    results go straight to the caller's arrays; one field costs one plane."""
    _play(fake, """
runs = []
for k in range(100):
    r = init(run(300, 109, lattice=9))
    r.moments()
    runs.append(r)
    assert F.fake_pinned() <= (64 << 20) + 4096
assert F.fake_pinned() > 60 << 20
for r in runs:
    r.close()
assert F.fake_pinned() == 4096       # the page of the health check's flags
for n in ((60, 50), (400, 300)):
    r = init(run(*n, lattice=9))
    a = np.zeros((2,) + n[::-1])
    log()
    lbm.load().lbm_moments(r.h, None, a[0].ctypes.data, None, None, 0)
    assert [l for l in log() if "copy" in l] == ["copy %d" % (8 * n[0] * n[1])]
    lbm.load().lbm_moments(r.h, a[0].ctypes.data, None, None, a[1].ctypes.data, 0)
    assert sum(int(l.split()[1]) for l in log() if "copy" in l) == 16 * n[0] * n[1]
    assert lbm.load().lbm_moments(r.h, None, None, None, None, 0) == lbm.LBM_OK
    assert not any("copy" in l for l in log())
    r.close()
""")


def test_the_cases_of_the_pair_tests_take_pairs(fake):
    """Also under the NaN canary, which fills buffers before the pass and between its steps."""
    _play(fake, """
import pair_cases as pc
for c in pc.SINGLE:
    r = pc.make(*c, seed=1)
    assert pairs(7, r) == 3, c
    r.set_debug(lbm.LBM_DEBUG_POISON)
    log()
    r.step(7)
    names = " ".join(log())
    assert names.count("k_core") == 3 and names.count("k_poison") == 7, c
    r.close()
for q in (37, 17, 9):
    g = lbm.Group()
    runs = [pc.make(q, "f64", *c, seed=1) for c, n in pc.GROUP]
    for r in runs:
        g.add(r)
    log()
    # stops at 1, 9, 16, 17 and 40 steps: one step, 3 pairs and two, eight steps, 11 pairs and one
    g.step(steps=np.array([n for c, n in pc.GROUP]))
    assert sum("k_core" in l for l in log()) == 14
    runs[0].set_debug(lbm.LBM_DEBUG_POISON)
    assert pairs(8, g) == 3
    for r in runs:
        g.remove(r)
        r.close()
    g.close()
""")


def test_autotune_keeps_pairs(fake, tmp_path):
    """A run or group that pairs is tuned within the fused schedule, timed in single steps, and a cached
    line of another schedule does not switch its pairs off; one that does not pair takes any line."""
    cache = str(tmp_path / "tune")
    with open(cache, "w") as f:
        f.write("700 700 0 9 128 0 -1\n200 200 0 9 128 0 -1\n")
    _play(fake, """
cache = %r
r = init(run(700, 700, lattice=9))
log()
assert r.autotune(steps=8, cache_path=cache)["overlap"] == 2
assert not any("k_core" in l for l in log())
assert pairs(of=r) == 3
lines = open(cache).read().splitlines()
assert len(lines) == 3 and lines[2].split()[5] == "2"
again = init(run(700, 700, lattice=9))
log()
assert again.autotune(steps=8, cache_path=cache) == r.get_launch()
assert len(open(cache).read().splitlines()) == 3
small = init(run(200, 200, lattice=9))
assert small.autotune(steps=8, cache_path=cache)["overlap"] == 0
g = lbm.Group()
g.add(r)
log()
assert g.autotune(steps=8)["overlap"] == 2
assert not any("k_core" in l for l in log())
assert pairs(of=g) == 3
""" % cache)


@pytest.mark.skipif(shutil.which("c++filt") is None, reason="c++filt not found")
def test_tracked_kernels_of_the_benchmark_exist(fake):
    """The counter summary of the benchmark finds its kernels by their demangled names."""
    _play(fake, """
import subprocess
import bench
seen = set()
r = init(run(1024, 1024, W=32, bc="nrbc"))
for overlap in (2, 0):
    r.set_launch(overlap=overlap)
    log()
    r.step(6)
    seen |= set(l[4:] for l in log() if l.startswith("run "))
names = subprocess.run(["c++filt"], input="\\n".join(seen), capture_output=True, text=True, check=True).stdout.split("\\n")
assert set(bench.TRACKED.values()) <= set(names), names
""")


def test_check_allocates_nothing(fake):
    """The health check, also of lbm_step's check interval, may run while another stream of the process is
    being captured: its flag lies in one pinned page of the process, as far as that goes."""
    _play(fake, """
runs = [init(run(16, 16, lattice=9)) for _ in range(1030)]
assert F.fake_pinned() == 4096
used = F.fake_used()
for r in runs:
    assert r.check() == lbm.LBM_OK
r = runs[0]
r.set_check_interval(4)
r.step(9)
assert F.fake_used() == used and F.fake_pinned() == 4096
for r in runs:
    r.close()
assert F.fake_pinned() == 4096 and F.fake_used() == 0
""")


def test_bands_of_a_group_are_one_allocation(fake):
    """The first step of a new group that pairs allocates once for all its members' bands."""
    _play(fake, """
big = init(run(720, 700, lattice=9))
small = [init(run(120, 110, lattice=9)) for _ in range(5)]
g = lbm.Group()
for r in [big] + small:
    g.add(r)
F.fake_mallocs.restype = ctypes.c_size_t
n = F.fake_mallocs()
assert pairs(of=g) == 3
assert F.fake_mallocs() == n + 5          # the group's four arrays and the bands
F.fake_limit(F.fake_used())               # nothing left: a result of a member takes the block
small[2].moments()
assert pairs(of=g) == 0
F.fake_limit(1 << 62)
g.remove(small[0])
assert pairs(of=g) == 3
""")
