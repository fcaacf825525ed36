"""The one-launch (resident) form of the PCG against the stepped form on the same inputs, at the
edges of its tiles and of every kernel variant, and its use by solves that overlap on two streams.

A call captured by the caller takes the stepped form, an eager one on an idle device the resident
form.  Per node both do the same arithmetic; only the order of the FP64 block sums differs, so the
coefficients agree to about 1e-13 relative and, rounded to FP32, to at most one unit in the last
place."""
import pytest
import torch

from gpu_helpers import DEV, say

pytestmark = pytest.mark.gpu

F32, F64 = torch.float32, torch.float64


def _system(rgp, shape, pe, dt, seed=3):
    """A diagonally dominant system (condition number about 20) and a right-hand side."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    rand = lambda: torch.rand(rgp.field_shape(shape, pe), dtype=F64, device=DEV, generator=g)  # noqa: E731
    return (2000 + 500 * rand()).to(dt), (-300 - 50 * rand()).to(dt), (rand() - 0.5).to(dt)


def _stepped(rgp, d, o, r, shape, pe, maxit, rtol):
    ws = torch.zeros(rgp.workspace_size(rgp.OP_PCG_SOLVE, shape, pe, (1, 1, 1), r.dtype),
                     dtype=torch.uint8, device=DEV)
    x = torch.empty_like(r)
    it = torch.zeros(1, dtype=torch.int32, device=DEV)
    rel = torch.zeros(1, dtype=F64, device=DEV)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rgp.pcg_solve_into(d, o, r, x, shape, pe, maxit, ws, rtol=rtol, iters=it, relres=rel,
                           stream=torch.cuda.current_stream())
    graph.replay()
    torch.cuda.synchronize()
    return x, it, rel


@pytest.mark.parametrize("shape,pe,dt,maxit,rtol", [
    ((2, 2, 1), 0, F32, 3, 0.0),            # one unit, one node per row
    ((7, 5, 6), 2, F64, 4, 0.0),
    ((33, 9, 255), 2, F32, 6, 0.0),         # 256 nodes per row: the widest rows it takes
    ((5, 41, 100), 1, F32, 6, 0.0),         # last tile with fewer rows, last unit with fewer planes
    ((3, 300, 250), 1, F32, 5, 0.0),
    ((97, 113, 75), 2, F32, 10, 0.1),       # units of 4 planes; stops early
    ((130, 131, 61), 0, F32, 5, 0.0),       # units of up to 8 planes
    ((144, 168, 111), 1, F32, 5, 0.0),      # up to 12
    ((150, 190, 117), 2, F32, 5, 0.0),      # up to 16
    ((200, 200, 132), 0, F32, 4, 0.0),      # three positions per thread
    ((199, 201, 131), 1, F32, 4, 0.0),
    ((200, 170, 131), 2, F32, 4, 0.0),
    ((40, 37, 30), 0, F64, 6, 0.0),         # FP64 units of 2, 4 and 8 planes
    ((70, 71, 50), 1, F64, 6, 0.0),
    ((90, 90, 89), 2, F64, 6, 0.0),
])
def test_resident_matches_stepped(shape, pe, dt, maxit, rtol):
    from paper_2403_10706_amd import rgp
    say(f"[resident] {shape} pe {pe} {dt}")
    d, o, r = _system(rgp, shape, pe, dt)
    x0, i0, rel0 = _stepped(rgp, d, o, r, shape, pe, maxit, rtol)
    rgp.timing_start()
    x1, i1, rel1 = rgp.pcg_solve(d, o, r, shape, pe, maxit=maxit, rtol=rtol)
    torch.cuda.synchronize()
    assert [k["kernel"] for k in rgp.timing_stop()] == ["pcg_solve"]
    err = float((x1 - x0).abs().max() / x0.abs().max())
    say(f"[resident] max|x - x_stepped| / max|x| = {err:.2e}, {int(i1)} iterations")
    assert int(i0) == int(i1)
    eps = 2.0 ** -23 if dt == F32 else 1e-13
    assert err <= 20 * maxit * eps, err
    assert abs(float(rel1) - float(rel0)) <= 20 * maxit * eps * (float(rel0) + eps)
    x2, _, _ = rgp.pcg_solve(d, o, r, shape, pe, maxit=maxit, rtol=rtol)
    assert torch.equal(x1, x2)


def test_resident_zero_rhs():
    from paper_2403_10706_amd import rgp
    shape, pe = (24, 30, 20), 1
    d, o, r = _system(rgp, shape, pe, F32)
    x, it, rel = rgp.pcg_solve(d, o, torch.zeros_like(r), shape, pe, maxit=5, rtol=0.0)
    assert int(it) == 0 and float(rel) == 0.0 and not bool(x.any())


def test_overlapping_solves_agree():
    """Plans replayed without waiting on two streams: whichever form each replay takes, the fields
    are those of a plan that runs alone, up to the order of the block sums."""
    from paper_2403_10706_amd import rgp
    shape, pe = (40, 44, 36), 1
    opts = rgp.Options(levels=2, gn_iters=4, pcg_iters=8, pcg_rtol=0.0)
    g = torch.Generator(device=DEV).manual_seed(5)
    I = torch.nn.functional.avg_pool3d(torch.rand((1, 1) + shape, device=DEV, generator=g), 5, 1, 2)[0, 0]
    pairs = [(I * k, torch.roll(I, 1, pe) * k) for k in (20.0, 30.0)]
    alone = [rgp.correct(P, M, pe, opts=opts)["b"] for P, M in pairs]
    need = rgp.workspace_size(rgp.OP_CORRECT, shape, pe, (1, 1, 1), F32, opts.to_c())
    plans, fields, keep = [], [], []
    for P, M in pairs:
        s = torch.cuda.Stream()
        b = torch.empty(rgp.field_shape(shape, pe), dtype=F32, device=DEV)
        T = torch.empty_like(P), torch.empty_like(M)
        ws = torch.zeros(need, dtype=torch.uint8, device=DEV)
        torch.cuda.synchronize()
        plans.append((rgp.Plan(P, M, pe, opts, b, T[0], T[1], ws, stream=s), s))
        fields.append(b)
        keep.append((T, ws))
    for _ in range(4):
        for p, s in plans:
            p.launch(s)
    torch.cuda.synchronize()
    for b, ref in zip(fields, alone):
        assert float((b - ref).abs().max()) <= 1e-3
    for p, _ in plans:
        p.close()
