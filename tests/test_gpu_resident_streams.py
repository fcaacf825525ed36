"""Which form of the PCG a call takes depends on the call alone: solves and corrections that overlap
on several streams and threads give the bits of one that runs by itself, and a stream that lacks some
of the device's compute units takes the form of one launch per iteration."""
import ctypes
import threading

import pytest
import torch

from gpu_helpers import DEV, say
from test_gpu_resident import F32, F64, _system

pytestmark = pytest.mark.gpu


def _workspace(rgp, shape, pe, dt):
    return torch.zeros(rgp.workspace_size(rgp.OP_PCG_SOLVE, shape, pe, (1, 1, 1), dt),
                       dtype=torch.uint8, device=DEV)


def _hip():
    """The HIP runtime that this process has loaded."""
    return ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))


class _Handle:
    """A stream known by its handle."""

    def __init__(self, handle):
        self.cuda_stream = handle


@pytest.mark.parametrize("shape,pe,dt,streams", [
    ((97, 113, 75), 2, F32, 2),    # 225 workgroups: one after the other
    ((40, 37, 30), 0, F64, 3),     # 63: beside each other
    ((12, 14, 10), 1, F32, 40),    # more streams than the library keeps entries for
])
def test_overlapping_solves_are_bitwise_equal(shape, pe, dt, streams):
    from paper_2403_10706_amd import rgp
    say(f"[resident streams] {shape} {dt} on {streams} streams")
    d, o, r = _system(rgp, shape, pe, dt)
    ref, it, _ = rgp.pcg_solve(d, o, r, shape, pe, maxit=40, rtol=0.0)
    ss = [torch.cuda.Stream() for _ in range(streams)]
    ws = [_workspace(rgp, shape, pe, dt) for _ in ss]
    xs = [[torch.full_like(r, 7.0) for _ in range(3)] for _ in ss]
    torch.cuda.synchronize()
    rgp.timing_start()
    for k in range(3):
        for s, w, x in zip(ss, ws, xs):
            rgp.pcg_solve_into(d, o, r, x[k], shape, pe, 40, w, stream=s)
    torch.cuda.synchronize()
    assert [k["kernel"] for k in rgp.timing_stop()] == ["pcg_solve"] * (3 * streams)
    for x in xs:
        for y in x:
            assert torch.equal(y, ref)


def test_threads_on_their_own_default_streams():
    """hipStreamPerThread is one handle for a stream of each thread (which ends with its thread: each
    waits for its own work)."""
    from paper_2403_10706_amd import rgp
    shape, pe = (97, 113, 75), 1
    d, o, r = _system(rgp, shape, pe, F32)
    ref, _, _ = rgp.pcg_solve(d, o, r, shape, pe, maxit=40, rtol=0.0)
    ws = [_workspace(rgp, shape, pe, F32) for _ in range(4)]
    xs = [[torch.full_like(r, 7.0) for _ in range(4)] for _ in ws]
    torch.cuda.synchronize()
    errors, hip = [], _hip()

    def work(w, x):
        try:
            torch.cuda.set_device(0)
            for y in x:
                rgp.pcg_solve_into(d, o, r, y, shape, pe, 40, w, stream=_Handle(2))
            assert hip.hipStreamSynchronize(ctypes.c_void_p(2)) == 0
        except Exception as e:   # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=a) for a in zip(ws, xs)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not errors, errors
    for x in xs:
        for y in x:
            assert torch.equal(y, ref)


def test_overlapping_plans_are_bitwise_equal():
    from paper_2403_10706_amd import rgp
    shape, pe = (72, 84, 56), 1
    opts = rgp.Options(levels=2, gn_iters=3, pcg_iters=12, pcg_rtol=0.0)
    g = torch.Generator(device=DEV).manual_seed(5)
    I = torch.nn.functional.avg_pool3d(torch.rand((1, 1) + shape, device=DEV, generator=g), 5, 1, 2)[0, 0]
    P, M = I * 20.0, torch.roll(I, 1, pe) * 20.0
    alone = rgp.correct(P, M, pe, opts=opts)["b"]
    need = rgp.workspace_size(rgp.OP_CORRECT, shape, pe, (1, 1, 1), F32, opts.to_c())
    plans, keep = [], []
    for _ in range(3):
        s = torch.cuda.Stream()
        b = torch.empty(rgp.field_shape(shape, pe), dtype=F32, device=DEV)
        T = torch.empty_like(P), torch.empty_like(M)
        ws = torch.zeros(need, dtype=torch.uint8, device=DEV)
        torch.cuda.synchronize()
        plans.append((rgp.Plan(P, M, pe, opts, b, T[0], T[1], ws, stream=s), s, b))
        keep.append((T, ws))
    for _ in range(4):
        for p, s, b in plans:
            with torch.cuda.stream(s):
                b.zero_()
            p.launch(s)
    torch.cuda.synchronize()
    for p, _, b in plans:
        assert torch.equal(b, alone)
        p.close()


def test_stream_without_all_compute_units_is_stepped():
    from paper_2403_10706_amd import rgp
    hip = _hip()
    handle = ctypes.c_void_p()
    mask = (ctypes.c_uint32 * 8)(*[0xffff] * 8)
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(handle), 8, mask) == 0
    shape, pe = (40, 44, 36), 1
    d, o, r = _system(rgp, shape, pe, F32)
    x, ws = torch.empty_like(r), _workspace(rgp, shape, pe, F32)
    torch.cuda.synchronize()
    rgp.timing_start()
    rgp.pcg_solve_into(d, o, r, x, shape, pe, 5, ws, stream=_Handle(handle.value))
    torch.cuda.synchronize()
    assert {k["kernel"] for k in rgp.timing_stop()} == {"pcg_step"}
    ref, _, _ = rgp.pcg_solve(d, o, r, shape, pe, maxit=5, rtol=0.0)
    eps = 2.0 ** -23   # as in test_resident_matches_stepped
    assert float((x - ref).abs().max() / ref.abs().max()) <= 20 * 5 * eps
    assert hip.hipStreamDestroy(handle) == 0
