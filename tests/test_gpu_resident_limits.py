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


def _run(shape, pe, dt, maxit, rtol, spins=SPINS, most=0, grow=0, cus=0):
    assert os.path.exists(DRIVER), "tests/_bin/resident_driver is missing: run __graft_entry__.build()"
    cmd = [DRIVER, *map(str, shape), str(pe), dt, str(maxit), str(rtol), str(spins), str(most),
           str(grow), str(cus)]
    say("[resident limits]", *cmd[1:])
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=60)
    say(r.stdout.strip(), r.stderr.strip())
    assert r.returncode == 0, (r.returncode, r.stderr)
    out = json.loads(r.stdout)
    for run in out["runs"]:
        run.pop("ms")
    return out


@pytest.mark.parametrize("shape,pe,dt", [((40, 44, 36), 1, "f32"), ((97, 113, 75), 2, "f32"),
                                         ((40, 37, 30), 0, "f64")])
def test_wait_given_up_shows_in_every_output(shape, pe, dt):
    """No workgroup waits for another's words: none has its neighbours' in time, so each gives up.
    The next solve on the same words is the first one again."""
    r = _run(shape, pe, dt, 6, 0.0, spins=0)
    ok, lost, again = r["runs"]
    assert ok["nans"] == 0 and ok["iters"] == 6
    assert lost["iters"] == -1 and math.isnan(float(lost["relres"])) and lost["nans"] > 0
    assert again == ok


# Every variant of the kernel and every PE axis (FP32 units of 2, 4, 8, 12, 16 planes and 16 planes of
# three positions per thread; FP64 units of 2, 4 and 8), odd extents, and the smallest volume.
VOLUMES = [((2, 2, 1), "f32", 0), ((33, 9, 150), "f32", 0), ((97, 113, 75), "f32", 1),
           ((130, 131, 61), "f32", 2), ((144, 168, 111), "f32", 3), ((150, 190, 117), "f32", 4),
           ((201, 199, 131), "f32", 5), ((40, 37, 30), "f64", 0), ((70, 71, 50), "f64", 1),
           ((90, 90, 89), "f64", 2)]


@pytest.mark.parametrize("most,grow", [(1, 0), (3, 0), (1, 7), (100, 40)])
@pytest.mark.parametrize("pe", [0, 1, 2])
@pytest.mark.parametrize("shape,dt,tier", VOLUMES)
def test_shared_solve_gives_the_same_bits(shape, dt, tier, pe, most, grow):
    """However many workgroups take part, and when they join: x, the iterations and the residual of
    the resident solve, and the next one on the same words."""
    if shape[pe] < 2:
        shape = shape[::-1]
    r = _run(shape, pe, dt, 5, 0.0, most=most, grow=grow)
    assert r["tier"] == tier and r["role"] == pe
    first, shared, again = r["runs"]
    assert first["nans"] == 0 and first["iters"] == 5
    assert shared == first and again == first


@pytest.mark.parametrize("most", [1, 5])
def test_shared_solve_stops_early(most):
    r = _run((40, 44, 36), 1, "f32", 30, 0.05, most=most, grow=1)
    first, shared, again = r["runs"]
    assert 0 < first["iters"] < 30
    assert shared == first and again == first


@pytest.mark.parametrize("cus", [8, 16])
@pytest.mark.parametrize("shape,pe,dt", [((97, 113, 75), 2, "f32"), ((144, 168, 111), 1, "f32"),
                                         ((90, 90, 89), 0, "f64")])
def test_fewer_compute_units_than_workgroups(shape, pe, dt, cus):
    """A stream with 64 or 128 compute units: the workgroups that start share the solve."""
    r = _run(shape, pe, dt, 8, 0.0, cus=cus)
    first, shared, again = r["runs"]
    assert shared == first and again == first
