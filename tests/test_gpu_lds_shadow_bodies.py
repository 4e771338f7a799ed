"""LDS race detection (the debug build libspvar_shadow.so) over what runs between and beside the
class passes of tests/test_gpu_lds_shadow.py: no conflict in any phase of
tests/lds_shadow_bodies_driver.py, every launch covered by the bitmap, results bit-exact."""
import json
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _phase(name):
    lib = os.path.join(ROOT, "paper_1706_07826_amd", "libspvar_shadow.so")
    assert os.path.exists(lib), "libspvar_shadow.so is not built (paper_1706_07826_amd/build.py builds both variants)"
    env = dict(os.environ, SPVAR_LIBRARY="shadow")
    env.pop("SPVAR_SHADOW_ALLOW_COLOUR_EDGES", None)
    p = subprocess.run([sys.executable, "-u", os.path.join(ROOT, "tests", "lds_shadow_bodies_driver.py"), name],
                       env=env, capture_output=True, text=True, timeout=110)
    print(p.stdout[-4000:], p.stderr[-4000:], flush=True)
    assert p.returncode == 0
    d = json.loads([l for l in p.stdout.splitlines() if l.startswith("{")][-1])
    assert d["write_write"] == 0 and d["read_write"] == 0 and d["uncovered"] == 0
    return d


def test_exchange():
    """A split group's boundary copy stores no byte into a word that an in-group swap of the same
    barrier interval stores whole."""
    d = _phase("exchange")
    assert d["passes"] > d["class_passes"]  # the exchanges with in-group swaps were checked too


@pytest.mark.parametrize("phase", ["records_in_lds", "held_sites"])
def test_sampling_bodies(phase):
    """The byte-parallel SA bodies, each under a switch that makes the launch take it."""
    assert _phase(phase)["passes"] > 1000
