"""The least-squares correction at the edges of its register form: one, 64, 65, 128, 192, 193, 256
and 257 cells per column, fields that compress many cells into one, and columns with values that are
not finite, against the oracle (or the same column without its neighbours)."""
import numpy as np
import pytest
import torch

from gpu_helpers import DEV, rel2, rounded, say, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("real", ["f64", "f32"])
@pytest.mark.parametrize("m", [2, 63, 64, 65, 128, 192, 193, 256, 257])
def test_lsq_column_lengths(m, real):
    from oracle import lsq as olsq
    from paper_2403_10706_amd import rgp
    say(f"[lsq edges] {m} cells {real}")
    dt = dict(f64=torch.float64, f32=torch.float32)[real]
    rng = np.random.default_rng(m)
    shape, pe = (3, m, 5), 1
    Ip, Im = (rounded(rng.uniform(1, 50, shape), dt) for _ in range(2))
    # stretches of slope up to 0.9 of either sign: up to ten moved cells end in one output cell
    s = np.repeat(rng.uniform(-0.9, 0.9, (3, -(-m // 8), 5)), 8, axis=1)[:, :m]
    b = rounded(np.concatenate([np.zeros((3, 1, 5)), np.cumsum(s, axis=1)], axis=1), dt)
    maxit = 4 if m > 4 else 1   # (two unknowns are exact after two steps)
    out, it = rgp.correct_lsq(to_dev(Ip, dt), to_dev(Im, dt), to_dev(b, dt), pe, maxit=maxit,
                              rtol=0.0)
    ref = olsq.lsq_correct(Ip, Im, b, pe, maxit=maxit, rtol=0.0)[0]
    err = rel2(to_host(out), ref)
    say(f"[lsq edges] {m} cells {real}: {err:.2e}")
    # four CGLS steps multiply the rounding of a position (m 2^-24 cells) by a few
    assert err <= dict(f64=1e-10, f32=1e-3)[real]


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), 3e38])
def test_lsq_non_finite_columns_stay_apart(bad):
    from paper_2403_10706_amd import rgp
    shape, pe = (2, 40, 6), 1
    g = torch.Generator(device=DEV).manual_seed(4)
    P, M = (torch.rand(shape, device=DEV, generator=g) + 1 for _ in range(2))
    b = 0.3 * torch.rand(rgp.field_shape(shape, pe), device=DEV, generator=g)
    clean, _ = rgp.correct_lsq(P, M, b, pe, maxit=5, rtol=0.0)
    Q = P.clone()
    Q[1, 17, 2] = bad
    out, _ = rgp.correct_lsq(Q, M, b, pe, maxit=5, rtol=0.0)
    keep = torch.ones_like(P, dtype=torch.bool)
    keep[1, :, 2] = False
    assert torch.equal(out[keep], clean[keep])
    if bad != bad:   # |s|^2 is NaN, so no iteration starts from I = 0
        assert not bool(out[1, :, 2].any())
    elif bad == float("inf"):   # the first step length is inf / inf
        assert bool(out[1, :, 2].isnan().all())
