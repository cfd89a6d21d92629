"""Runs and a group that take two-step passes, for the bounds-checked debug build: run_all() steps
each with whichever library build is loaded, checks it (an index out of range raises in the
bounds-checked build) and returns a hash of its state.

Run as a script (python tests/bounds_pair_cases.py OUT.json) with LBM_MI355X_LIB naming the
bounds-checked build; tests/test_gpu_bounds_pairs.py compares its hashes with the normal build's."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
for p in (ROOT, os.path.join(ROOT, "tests")):
    if p not in sys.path:
        sys.path.insert(0, p)

import numpy as np  # noqa: E402
from bounds_cases import _digest  # noqa: E402
from pair_cases import GROUP, SINGLE, make  # noqa: E402


def run_all():
    from paper_2504_20169_amd import lbm
    out = {"build_flags": lbm.lbm_build_flags()}
    for c in SINGLE:
        print("bounds pair case", c, flush=True)
        r = make(*c, seed=70)
        r.step(4)            # a pair and two single steps
        out[repr(c)] = "%d %s" % (r.check(), _digest(r.populations(), *r.moments(), r.pml_q()))
        r.close()
    for q in (37, 17, 9):
        print("bounds pair group", q, flush=True)
        g = lbm.Group()
        runs = [make(q, "f64", *c, seed=80 + k) for k, (c, n) in enumerate(GROUP)]
        for r in runs:
            g.add(r)
        g.step(steps=np.array([n for c, n in GROUP], dtype=np.int64))
        flags = g.check()
        assert not (flags == 2).any(), flags   # 2: an index out of range (bounds-checked build)
        for k, r in enumerate(runs):
            out["group %d %d" % (q, k)] = "%d %s" % (flags[k], _digest(r.populations(), *r.moments(), r.pml_q()))
        g.close()
        for r in runs:
            r.close()
    return out


if __name__ == "__main__":
    import torch  # noqa: F401  (PyTorch first, as the benchmark loads it)
    res = run_all()
    with open(sys.argv[1], "w") as fh:
        json.dump(res, fh, indent=1)
    print("bounds pair cases done", len(res) - 1, flush=True)
