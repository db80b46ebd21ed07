"""Forms whose index ranges are easy to leave, under the bounds-checked build: the same solves in a
process that loads it end with a check word of 0 and give, bit for bit, the points of the plain
build, which this process loads."""
import os
import subprocess
import sys

import numpy as np
import pytest

import paper_2604_23951_amd as lpg

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
sys.path.insert(0, HERE)
import checked_forms_child  # noqa: E402


@pytest.mark.parametrize("name", list(checked_forms_child.SETS))
def test_checked_build_runs_clean(name, tmp_path):
    lib = os.path.join(ROOT, "paper_2604_23951_amd", "_lib", "liblpgpu_checked.so")
    if not os.path.exists(lib):
        pytest.skip("checked build not compiled (run __graft_entry__.build())")
    out = tmp_path / "checked.npz"
    env = dict(os.environ, LPGPU_CHECKED="1", PYTHONPATH=os.pathsep.join([ROOT, HERE]))
    env.pop("LPGPU_LIB_OVERRIDE", None)
    print("checked build: child process", name, flush=True)
    r = subprocess.run([sys.executable, os.path.join(HERE, "checked_forms_child.py"), name, str(out)], env=env,
                       capture_output=True, text=True, timeout=100)
    print(r.stdout[-2000:], r.stderr[-2000:], flush=True)
    assert r.returncode == 0
    got = np.load(out)
    assert int(got["checked"]) == 1 and int(got["word"]) == 0
    assert lpg.lp_check_word(0) == (0, False)
    ref = dict(checked_forms_child.SETS[name]())
    assert set(ref) == set(got.files) - {"word", "checked"}
    for key, x in ref.items():
        np.testing.assert_array_equal(got[key], x, err_msg=key)
