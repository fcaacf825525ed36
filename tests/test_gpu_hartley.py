"""The z-update's Hartley passes over line lengths that take each fold (odd, 2 mod 4, 0 mod 4), one
line per workgroup and tiny grids: an ADMM correction against the oracle."""
import numpy as np
import pytest
import torch

from gpu_helpers import BFINAL_ATOL, say, to_dev, to_host
from oracle import rgp as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,pe", [((1, 8, 1), 1), ((2, 8, 3), 1), ((4, 6, 5), 1), ((8, 9, 6), 1),
                                      ((66, 5, 37), 1), ((3, 10, 300), 1), ((1024, 3, 2), 1),
                                      ((1023, 3, 2), 1), ((7, 12, 14), 0), ((9, 10, 16), 2)])
@pytest.mark.parametrize("real", ["f64", "f32"])
def test_admm_line_lengths(shape, pe, real):
    from paper_2403_10706_amd import rgp
    say(f"[hartley] {shape} pe {pe} {real}")
    dt = dict(f64=torch.float64, f32=torch.float32)[real]
    rng = np.random.default_rng(2)
    Ip = 10 + rng.uniform(0, 1, shape)
    Im = 10 + rng.uniform(0, 1, shape)
    Ip, Im = (torch.as_tensor(x).to(dt).double().numpy() for x in (Ip, Im))
    opts = rgp.Options(levels=1, gn_iters=2, pcg_iters=10, pcg_rtol=0.1, solver="admm")
    out = rgp.correct(to_dev(Ip, dt), to_dev(Im, dt), pe, opts=opts, real_dtype=dt)
    ref = orc.solve(Ip, Im, pe, levels=1, gn_iters=2, pcg_iters=10, pcg_rtol=0.1, solver="admm")
    d = float(np.max(np.abs(to_host(out["b"]) - ref.b)))
    say(f"[hartley] {shape} pe {pe} {real}: max|b - b_oracle| = {d:.3e} of {np.max(np.abs(ref.b)):.2e}")
    assert d <= dict(f64=1e-8, f32=BFINAL_ATOL)[real]
