"""The bounds-checked debug build over two-step passes: every stencil and paired storage, thin grids,
periodic wraps, formed targets and a group of small members.  No kernel meets an index out of range,
and the results are bitwise those of the normal build."""
import json
import os
import subprocess
import sys

import pytest

from paper_2504_20169_amd import lbm

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, HERE)
import bounds_pair_cases  # noqa: E402


@pytest.mark.gpu
def test_bounds_checked_pairs_find_no_index_out_of_range(tmp_path):
    if not os.path.exists(lbm.BOUNDS_LIB_PATH):
        pytest.fail("the bounds-checked build is missing: run __graft_entry__.build()")
    out = tmp_path / "bounds_pairs.json"
    env = dict(os.environ, LBM_MI355X_LIB=lbm.BOUNDS_LIB_PATH)
    print("bounds-checked build: subprocess over pairs", flush=True)
    res = subprocess.run([sys.executable, "-u", os.path.join(HERE, "bounds_pair_cases.py"), str(out)],
                         env=env, capture_output=True, text=True, timeout=110)
    sys.stdout.write(res.stdout[-2000:])
    assert res.returncode == 0, res.stderr[-4000:]
    checked = json.load(open(out))
    assert checked.pop("build_flags") == lbm.LBM_BUILD_BOUNDS
    normal = bounds_pair_cases.run_all()
    assert normal.pop("build_flags") == 0
    assert checked.keys() == normal.keys()
    assert not [k for k in normal if normal[k] != checked[k]]
