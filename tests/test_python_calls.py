"""What the Python layer does around the library's calls, without a GPU."""
import numpy as np
import pytest
import torch

from paper_2403_10706_amd import autograd as ag
from paper_2403_10706_amd import rgp


@pytest.mark.parametrize("weights", [None, [1.0], [2.0], [1.0, 1.0], [0.5, 1.0]])
def test_pyramid_objective_returns_a_scalar_of_its_own(monkeypatch, weights):
    """The objective may be added to in place, on one level as on several."""
    levels = 1 if weights is None else len(weights)
    jdsp = []

    def loss_grad(P, M, b, *args, **kwargs):
        jdsp.append(torch.arange(3.0, 7.0, dtype=torch.float64))
        return jdsp[-1], None, None, None

    monkeypatch.setattr(rgp, "loss_grad", loss_grad)
    monkeypatch.setattr(rgp, "restrict_image", lambda I, dtype: I[::2, ::2, ::2].contiguous())
    shape, fields = (4, 4, 4), []
    for l in range(levels):
        n = 4 // 2 ** l
        fields.append(torch.zeros(rgp.field_shape((n, n, n), 1), requires_grad=True))
    I = torch.ones(shape)
    J = ag.pyramid_objective(I, I, fields, 1, weights=weights)
    want = 3.0 * (sum(weights) if weights else 1.0)
    assert float(J.detach()) == want and J.requires_grad
    J += 1.0
    assert float(J.detach()) == want + 1.0
    assert all(float(x[0]) == 3.0 for x in jdsp)


def _same(g, want):
    return list(g.m) == list(want.m) and list(g.h) == list(want.h) and g.pe == want.pe


@pytest.mark.parametrize("shape,pe,h", [
    ((8, 9, 10), 1, (1.0, 0.9, 1.1)),
    ([8, 9, 10], 1, [1.0, 0.9, 1.1]),
    (torch.Size((8, 9, 10)), 1, (1, 2, 3)),
    (np.array([8, 9, 10]), np.int64(1), np.array([1.0, 0.9, 1.1])),
    ([np.array(8), np.array(9), np.array(10)], np.array(1), [np.array(1.0)] * 3),
    (torch.tensor([8, 9, 10]), torch.tensor(1), torch.tensor([1.0, 0.9, 1.1])),
    ((8.0, 9, 10), True, (1.0, 1.0, 1.0)),
])
def test_grid_of_a_call_takes_what_make_grid_takes(shape, pe, h):
    for _ in range(2):
        assert _same(rgp._grid(shape, pe, h), rgp.make_grid(shape, pe, h))
        assert rgp._need(rgp.OP_GN_HVP, shape, pe, h, torch.float32) == \
            rgp.workspace_size(rgp.OP_GN_HVP, shape, pe, h, torch.float32)


def test_grid_of_a_call_sees_values_changed_in_place():
    h, pe = torch.tensor([1.0, 1.0, 1.0]), torch.tensor(1)
    parts = list(h)   # one-element tensors that keep their identity
    rgp._grid((8, 9, 10), pe, parts)
    before = rgp._need(rgp.OP_GN_HVP, (8, 9, 10), pe, parts, torch.float32)
    h[0] = 2.0
    pe.fill_(2)
    assert _same(rgp._grid((8, 9, 10), pe, parts), rgp.make_grid((8, 9, 10), 2, (2.0, 1.0, 1.0)))
    after = rgp._need(rgp.OP_GN_HVP, (8, 9, 10), pe, parts, torch.float32)
    assert after == rgp.workspace_size(rgp.OP_GN_HVP, (8, 9, 10), 2, (2.0, 1.0, 1.0), torch.float32)
    assert before == rgp.workspace_size(rgp.OP_GN_HVP, (8, 9, 10), 1, (1.0, 1.0, 1.0), torch.float32)
