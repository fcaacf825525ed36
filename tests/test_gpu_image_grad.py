"""dJ/dI+- at the edges of its runs of 8 samples: columns of 2 to 170 cells, fields that stretch and
compress the samples close to the barrier and carry whole stretches out of the column."""
import numpy as np
import pytest
import torch

from gpu_helpers import rel2, rounded, say, to_dev, to_host
from oracle import rgp as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("real", ["f64", "f32"])
@pytest.mark.parametrize("shape,pe,amp", [
    ((2, 3, 5), 0, 0.4), ((3, 7, 65), 1, 2.5), ((5, 8, 9), 1, 3.0), ((4, 9, 64), 1, 3.0),
    ((3, 170, 70), 1, 40.0), ((33, 5, 4), 0, 60.0), ((6, 5, 31), 2, 9.0)])
def test_image_gradient_run_edges(shape, pe, amp, real):
    from paper_2403_10706_amd import rgp
    say(f"[image grad] {shape} pe {pe} amp {amp} {real}")
    dt = dict(f64=torch.float64, f32=torch.float32)[real]
    rng = np.random.default_rng(9)
    Ip, Im = (rounded(rng.uniform(0, 50, shape), dt) for _ in range(2))
    nsh = [m + (d == pe) for d, m in enumerate(shape)]
    # slopes of up to 0.95 along PE, of either sign for stretches of cells, shifted as a whole
    s = np.repeat(rng.uniform(-0.95, 0.95, [-(-n // 6) if d == pe else n for d, n in
                                            enumerate(shape)]), 6, axis=pe)
    b = np.concatenate([np.zeros([1 if d == pe else n for d, n in enumerate(shape)]),
                        np.cumsum(np.take(s, range(shape[pe]), axis=pe), axis=pe)], axis=pe)
    assert list(b.shape) == nsh
    b = rounded(b + rng.uniform(-amp, amp), dt)
    gp, gm = rgp.loss_grad_images(to_dev(Ip, dt), to_dev(Im, dt), to_dev(b, dt), pe)
    rp, rm = orc.image_gradient(Ip, Im, b, pe, (1.0, 1.0, 1.0))
    # FP32: a position of up to 200 cells is rounded by 200 * 2^-24, times the largest slope of the
    # interpolant over the typical residual
    tol = dict(f64=1e-11, f32=1e-4)[real]
    assert rel2(to_host(gp), rp) <= tol
    assert rel2(to_host(gm), rm) <= tol
