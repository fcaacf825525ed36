"""The OT start at the edges of its segments: columns at and around 8, 12 and 16 cells per segment of
16, columns shorter than the segments are many, and a number of columns that fills no tile, along each
axis, against the oracle."""
import numpy as np
import pytest
import torch

from gpu_helpers import rounded, say, to_dev, to_host
from oracle import rgp as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("real", ["f64", "f32"])
@pytest.mark.parametrize("m,pe", [(2, 0), (15, 1), (17, 2), (128, 0), (129, 1), (192, 2), (193, 0),
                                  (200, 1), (256, 2), (257, 0)])
def test_ot_segment_edges(m, pe, real):
    from paper_2403_10706_amd import rgp
    say(f"[ot edges] {m} cells, axis {pe}, {real}")
    dt = dict(f64=torch.float64, f32=torch.float32)[real]
    shape = [5, 7]
    shape.insert(pe, m)
    rng = np.random.default_rng(m)
    Ip, Im = (rounded(rng.uniform(-1, 50, shape), dt) for _ in range(2))
    h = (1.0, 1.25, 0.75)
    for guard in (True, False):
        b0, ng = rgp.ot_init(to_dev(Ip, dt), to_dev(Im, dt), pe, h, guard=guard)
        ref = orc.ot_init(Ip, Im, pe, h, eps=1e-3, guard=guard)
        err = float(np.max(np.abs(to_host(b0) - ref.b0)))
        say(f"[ot edges] guard {guard}: {err:.2e}")
        # the CDFs are FP64 in both; the start is rounded once to its type (2^-24 of 64 voxels)
        assert err <= dict(f64=1e-9 * max(1.0, m / 100.0), f32=1e-4)[real]
        if guard:
            assert int(to_host(ng)[0]) == ref.guarded_cells
