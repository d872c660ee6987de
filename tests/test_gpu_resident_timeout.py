"""A solve on the chip whose workgroups do not answer each other in time (the
test hook allows an exchange no look, or one or two) must end on the tile
passes with their answer: bit for bit that of a context that never iterates on
the chip, whether from zero or capped, and within the solve's tolerance from a
warm start.  A grid of one workgroup exchanges nothing and stays."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TANK = (0, 0, 0, 0, 0, 1)
P = 2


def _make(F, shape, bc, kind):
    nx, ny, nz = shape
    case = F.make_two_phase(nx, ny, nz, surface_seed=31, velocity_seed=32, wedge=F.Wedge(), bc=bc)
    if kind == "densities":
        case.rho = case.rho * (1.0 + 0.3 * np.random.default_rng(5).random(case.rho.shape))
    return case


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _solver(case, precision, **kw):
    from paper_1410_1942_amd.solver import Solver
    return Solver(_t(case.rho), _t(case.mask), case.bc, case.h, precision=precision, **kw)


@pytest.mark.parametrize("shape,bc", [((97, 66, 45), (1, 0, 0, 1, 0, 1)), ((36, 50, 20), (P, P, 0, 0, 0, 0))],
                         ids=str)
@pytest.mark.parametrize("kind", ["classes", "densities"])
@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "ir"])
@pytest.mark.parametrize("polls", [0, 1, 2])
def test_timeout(orc, F, shape, bc, kind, precision, polls):
    import torch
    print(f"case resident timeout {shape} bc={bc} {kind} prec={precision} polls={polls}", flush=True)
    case = _make(F, shape, bc, kind)
    rhs = _t(case.rhs)
    ref = orc.pcg(case.rho, case.mask, case.bc, case.h, case.rhs, tol=1e-12)
    scale = np.abs(ref.p).max()

    def close(p, tol):
        q = p.cpu().numpy()
        assert orc.relres(case.rho, case.mask, case.bc, case.h, case.rhs, q) <= tol
        assert np.abs(q - ref.p).max() <= 1e-6 * scale

    # the caller's own launch shape keeps a solve off the chip
    s, tiles = _solver(case, precision), _solver(case, precision, grid_blocks=256)
    try:
        want, sw = tiles.solve(rhs, tol=1e-8)
        s.set_resident_limits(polls=polls)
        got, sg = s.solve(rhs, tol=1e-8)
        assert sg["status"] == 0, sg
        close(got, 1e-8)
        if polls == 0:
            assert sg["iters"] == sw["iters"] and torch.equal(got, want)
        s.set_resident_limits()
        again, sa = s.solve(rhs, tol=1e-8)      # the context stays with the passes
        if polls == 0:
            assert sa["iters"] == sw["iters"] and torch.equal(again, want)
        close(again, 1e-8)
    finally:
        s.close()
        tiles.close()
    for k in (1, 40):
        s, tiles = _solver(case, precision), _solver(case, precision, grid_blocks=256)
        s.set_resident_limits(polls=polls)
        got, sg = s.solve(rhs, tol=1e-30, maxit=k, raise_on_error=False)
        want, sw = tiles.solve(rhs, tol=1e-30, maxit=k, raise_on_error=False)
        s.close()
        tiles.close()
        assert (sg["status"], sg["iters"]) == (sw["status"], sw["iters"]) == (1, k)
        assert np.abs((got - want).cpu().numpy()).max() <= 1e-6 * np.abs(want.cpu().numpy()).max()
    s = _solver(case, precision)
    s.set_resident_limits(polls=polls)
    got, sg = s.solve(rhs, p=_t(ref.p), tol=1e-8, warm=True)
    s.close()
    assert sg["status"] == 0 and sg["iters"] <= 5, sg
    close(got, 1e-8)


def test_device_held_by_another_stream(F):
    """A kernel on another stream holds a compute unit for a second; the bricks of
    this grid need all of them."""
    import torch
    print("case resident, device held", flush=True)
    case = _make(F, (320, 128, 96), TANK, "classes")
    rhs = _t(case.rhs)
    mine, other = torch.cuda.Stream(), torch.cuda.Stream()
    tiles = _solver(case, 0, grid_blocks=512)
    want = tiles.solve(rhs)[0].clone()
    tiles.close()
    s = _solver(case, 0, stream=mine)
    assert s.resident_form()[0] == 256
    s.set_resident_limits(polls=1 << 21)     # the default, not counted against later contexts
    torch.cuda.synchronize()
    with torch.cuda.stream(other):
        torch.cuda._sleep(2_400_000_000)     # about a second
    p, st = s.solve(rhs, tol=1e-8)
    torch.cuda.synchronize()
    s.close()
    assert st["status"] == 0
    assert float((p - want).abs().max()) <= 1e-6 * float(want.abs().max())


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "ir"])
def test_one_workgroup_exchanges_nothing(F, precision):
    import torch
    print(f"case resident timeout, one workgroup prec={precision}", flush=True)
    case = _make(F, (7, 5, 6), TANK, "classes")
    rhs = _t(case.rhs)
    s = _solver(case, precision)
    want, sw = s.solve(rhs, tol=1e-8)
    s.set_resident_limits(polls=0)
    got, sg = s.solve(rhs, tol=1e-8)
    s.close()
    assert sg["iters"] == sw["iters"] and torch.equal(got, want)
