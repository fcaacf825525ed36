"""What the resident PCG kernel does where its workgroups cannot all run or one stands still
(tests/resident_driver.cpp, built by __graft_entry__.build(), sets the limits from the host)."""
import json
import math
import os
import subprocess

import pytest

from gpu_helpers import say

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = os.path.join(ROOT, "tests", "_bin", "resident_driver")
SPINS = 1 << 24   # the library's own


def _run(shape, pe, dt, maxit, rtol, *limits):
    assert os.path.exists(DRIVER), "tests/_bin/resident_driver is missing: run __graft_entry__.build()"
    cmd = [DRIVER, *map(str, shape), str(pe), dt, str(maxit), str(rtol), *map(str, limits)]
    say("[resident limits]", *cmd[1:])
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=60)
    say(r.stdout.strip(), r.stderr.strip())
    assert r.returncode == 0, (r.returncode, r.stderr)
    return json.loads(r.stdout)


@pytest.mark.parametrize("shape,pe,dt", [((40, 44, 36), 1, "f32"), ((97, 113, 75), 2, "f32"),
                                         ((40, 37, 30), 0, "f64")])
def test_wait_given_up_shows_in_every_output(shape, pe, dt):
    """No workgroup waits for another's words: none has its neighbours' in time, so each gives up.
    The next solve on the same words is the first one again."""
    r = _run(shape, pe, dt, 6, 0.0, 0)
    ok, lost, again = r["runs"]
    assert ok["nans"] == 0 and ok["iters"] == 6
    assert lost["iters"] == -1 and math.isnan(float(lost["relres"])) and lost["nans"] > 0
    assert again == ok
