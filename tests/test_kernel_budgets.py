"""Register budgets of the two-step tiles and of the boundary kernels, every stencil (CPU: the compiler's
resource report for gfx950).  The tiles fill the LDS and registers of a compute unit, so their waves
per SIMD are those their LDS allows; what spills there is held to what it was measured with."""
import os
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2504_20169_amd import build as b
from test_kernel_resources import _resource_report

pytestmark = pytest.mark.slow

# (kernel, type of the storage, further text of the name): fewest waves per SIMD for D2Q37, D2Q17, D2Q9
BUDGET = [
    ("k_core", "d", "", (2, 4, 6)), ("k_core", "f", "", (4, 6, 8)),
    ("k_small_step", "d", "", (2, 4, None)), ("k_small_step", "f", "", (4, 5, None)),
    ("k_small_step", "DF16_", "", (4, 5, None)),
    ("k_frame_split", "d", "", (2, 4, None)), ("k_frame_split", "f", "", (4, 8, None)),
    ("k_frame_split", "DF16_", "", (4, 8, None)),
    ("k_frame", "d", "Li0E", (2, 4, 4)), ("k_frame", "f", "Li0E", (4, 5, 8)), ("k_frame", "DF16_", "Li0E", (4, 5, 8)),
    ("k_frame", "d", "Li1E", (2, 3, 4)), ("k_frame", "f", "Li1E", (3, 4, 6)),
    ("k_frame", "d", "Li2E", (2, 4, 4)), ("k_frame", "f", "Li2E", (4, 5, 8)),
    ("k_phase_a", "d", "Li1E", (3, 4, 7)), ("k_phase_a", "f", "Li1E", (3, 5, 7)),
]
SPILLED = {("k_core", "f", 0): 6}   # VGPRs, D2Q37: 28 bytes of scratch per lane


def test_budgets():
    srcs = [os.path.join(b.HERE, "csrc", n) for n in ("lbm_kernels.hip", "lbm_kernels_d2q17.hip", "lbm_kernels_d2q9.hip")]
    with ThreadPoolExecutor(3) as ex:
        reports = list(ex.map(_resource_report, srcs))
    for name, kind, more, waves in BUDGET:
        for s, (report, most) in enumerate(zip(reports, waves)):
            key = "%d%sI%s" % (len(name), name, kind)   # as the name is mangled
            found = [r for n, r in report.items() if key in n and more in n]
            assert bool(found) == (most is not None), (name, kind, s)
            for r in found:
                assert int(r["Occupancy [waves/SIMD]"]) >= most, (name, kind, more, s, r)
                assert int(r["VGPRs Spill"]) <= SPILLED.get((name, kind, s), 0), (name, kind, more, s, r)
