"""The form of one launch per PCG iteration against the oracle.  Calls on an ordinary stream take the
resident form wherever a volume fits the chip; on a stream that lacks one compute unit they do not,
so the parity tests run here a second time on such a stream."""
import ctypes

import pytest
import torch

from tests import test_gpu_parity as parity
from tests.gpu_helpers import DEV, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def narrow():
    """A stream with all compute units but one."""
    from paper_2403_10706_amd import rgp
    rgp.load()
    torch.zeros(1, device=DEV)
    hip = ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))
    handle = ctypes.c_void_p()
    mask = (ctypes.c_uint32 * 8)(*([0x7fffffff] + [0xffffffff] * 7))
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(handle), 8, mask) == 0
    yield torch.cuda.ExternalStream(handle.value)
    torch.cuda.synchronize()   # (the stream lives as long as the process: workspaces are kept by handle)


def _kernels(rgp, call):
    rgp.timing_start()
    call()
    torch.cuda.synchronize()
    return {k["kernel"] for k in rgp.timing_stop()}


@pytest.mark.parametrize("real", ["f64", "f32"])
@pytest.mark.parametrize("test,args", [
    *[("test_pcg_parity", s) for s in parity.SHAPES[:5]],
    ("test_correct_single_level_c1", ()),
    ("test_correct_with_ot_blur", ()),
    ("test_correct_line_search_backtracks", ()),
    ("test_correct_line_search_failure", (3000.0, 3)),
    ("test_correct_barrier_violating_b_init", ()),
])
def test_stepped_form_against_the_oracle(narrow, test, args, real):
    rgp = parity._rgp()
    say(f"[stepped] {test} {args} {real}")

    def call():
        with torch.cuda.stream(narrow):
            if test == "test_correct_line_search_failure":
                parity.test_correct_line_search_failure(real, *args)
            else:
                getattr(parity, test)(*args, real)

    got = _kernels(rgp, call)
    assert "pcg_step" in got and "pcg_solve" not in got


def test_stepped_plan_and_batch_match_the_eager_call(narrow):
    """A plan replayed on the narrow stream, a batch with and without a graph, and a correction that
    the caller captures on any stream give the bits of the eager correction there."""
    rgp = parity._rgp()
    specs = [((37, 29, 23), 0), ((21, 45, 67), 1), ((19, 26, 41), 2)]
    opts = rgp.Options(levels=2, gn_iters=3, pcg_iters=6, pcg_rtol=0.0)
    dt, pairs = torch.float32, []
    for i, (shape, pe) in enumerate(specs):
        p = parity._pair(shape, pe, seed=40 + i, scale=30.0)
        pairs.append((parity.to_dev(p.I_plus, dt), parity.to_dev(p.I_minus, dt), pe))
    torch.cuda.synchronize()
    with torch.cuda.stream(narrow):
        eager = [rgp.correct(P, M, pe, opts=opts)["b"] for P, M, pe in pairs]
        bp = rgp.BatchPlan([p[0] for p in pairs], [p[1] for p in pairs], [p[2] for p in pairs], opts,
                           stream=narrow)
        bp.launch(narrow)
        narrow.synchronize()
        for b, ref in zip(bp.b, eager):
            assert torch.equal(b, ref)
            b.fill_(3.0)
        bp.run_eager(narrow)
        narrow.synchronize()
        for b, ref in zip(bp.b, eager):
            assert torch.equal(b, ref)
    P, M, pe = pairs[0]
    b, T = torch.empty_like(eager[0]), (torch.empty_like(P), torch.empty_like(M))
    need = rgp.workspace_size(rgp.OP_CORRECT, tuple(P.shape), pe, (1, 1, 1), dt, opts.to_c())
    ws = torch.zeros(need, dtype=torch.uint8, device=DEV)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    plan = rgp.Plan(P, M, pe, opts, b, T[0], T[1], ws, stream=s)
    plan.launch(narrow)
    torch.cuda.synchronize()
    assert torch.equal(b, eager[0])
    graph, b2, T2 = torch.cuda.CUDAGraph(), torch.empty_like(b), (torch.empty_like(P), torch.empty_like(M))
    with torch.cuda.graph(graph):
        rgp.correct_into(P, M, pe, opts, b2, T2[0], T2[1], ws, stream=torch.cuda.current_stream())
    for _ in range(3):
        b2.fill_(3.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(b2, eager[0])
    plan.launch(s)   # on a whole stream: the resident form, equal to rounding
    torch.cuda.synchronize()
    assert torch.equal(b, rgp.correct(P, M, pe, opts=opts)["b"])
    assert float((b - eager[0]).abs().max()) <= 1e-3   # as in test_overlapping_solves_agree
    plan.close()
