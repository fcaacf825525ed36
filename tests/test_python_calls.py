"""What the Python layer does around the library's calls, without a GPU."""
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
