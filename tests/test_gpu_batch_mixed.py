"""Batches whose volumes take both forms of the PCG on one level: those that fit the chip are solved
by one launch per solve, those that do not by one launch per iteration."""
import pytest
import torch

from gpu_helpers import DEV, say

pytestmark = pytest.mark.gpu

F64 = torch.float64
BIG, SMALL = ((104, 104, 100), 1), ((40, 44, 36), 0)
BIG2 = ((100, 106, 104), 2)


def _pair(shape, pe, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    I = torch.nn.functional.avg_pool3d(torch.rand((1, 1) + shape, device=DEV, generator=g), 5, 1, 2)[0, 0]
    return (I * 20.0).to(F64).contiguous(), (torch.roll(I, 1, pe) * 20.0).to(F64).contiguous()


@pytest.mark.parametrize("specs", [[BIG, SMALL, BIG2], [SMALL, BIG], [BIG, BIG2]])
def test_volumes_beyond_the_chip_in_a_batch(specs):
    """Fields bitwise those of each pair alone, in the plan and without a graph."""
    from paper_2403_10706_amd import rgp
    gn, its = 2, 4
    opts = rgp.Options(levels=2, gn_iters=gn, pcg_iters=its, pcg_rtol=0.0)
    pairs = [_pair(sh, pe, 60 + i) for i, (sh, pe) in enumerate(specs)]
    pes = [pe for _, pe in specs]
    alone = [rgp.correct(P, M, pe, opts=opts, real_dtype=F64)["b"] for (P, M), pe in zip(pairs, pes)]
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        bp = rgp.BatchPlan([p for p, _ in pairs], [m for _, m in pairs], pes, opts, real_dtype=F64,
                           stream=s)
        bp.launch(s)
        s.synchronize()
        for i, b in enumerate(alone):
            assert torch.equal(bp.b[i], b), i
            bp.b[i].fill_(3.0)
        rgp.timing_start()
        bp.run_eager(s)
        s.synchronize()
    kernels = [k["kernel"] for k in rgp.timing_stop()]
    say(f"[batch mixed] {specs}: {kernels.count('pcg_step')} steps, {kernels.count('pcg_solve')} solves")
    for i, b in enumerate(alone):
        assert torch.equal(bp.b[i], b), i
    # the finest level's big volumes: one launch per iteration and one for the last update, each step;
    # without a small one beside them they share it
    big = sum(sp is not SMALL for sp in specs)
    assert kernels.count("pcg_step") == gn * (its + 1) * (big if SMALL in specs else 1)
    assert kernels.count("pcg_solve") > 0
