"""Solves that fit on the chip (the resident iteration, the default of small
and mid grids coded by density class), through the C ABI, against the oracle.

The iteration is the textbook one, so the bar is the oracle's: the converged
answer, the iteration count and the k-th iterate of a capped solve.  The
shapes sit at the edges of its bricks (whole rows, a share of the rows and
planes each): a single brick, one row or plane a brick, ragged last bricks
along y and z, rows of one cell, rows longer than a workgroup, every wall
kind, and periodic axes with one brick and with several.  Tolerances are
those of the other tile forms' tests.
"""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TANK = (0, 0, 0, 0, 0, 1)
P = 2
FLAT_TILES = 16
WARM = 1


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available()
    return torch, torch.device("cuda:0")


def _to(torch, dev, a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


def _solve(torch_dev, case, tol=1e-8, maxit=1000000, p0=None, **kw):
    torch, dev = torch_dev
    from paper_1410_1942_amd.solver import Solver
    s = Solver(_to(torch, dev, case.rho), _to(torch, dev, case.mask), case.bc, case.h, **kw)
    p = None if p0 is None else _to(torch, dev, p0)
    p, st = s.solve(_to(torch, dev, case.rhs), p=p, tol=tol, maxit=maxit,
                    raise_on_error=False, warm=p0 is not None)
    torch.cuda.synchronize()
    s.close()
    return p.cpu().numpy(), st


def _case(F, shape, bc, wedge=True):
    nx, ny, nz = shape
    return F.make_two_phase(nx, ny, nz, surface_seed=41, velocity_seed=42,
                            wedge=F.Wedge() if wedge else None, bc=bc)


CASES = [
    ((7, 5, 6), TANK, False),                   # one brick
    ((1, 1, 64), TANK, False),                  # a single column
    ((2, 9, 8), (P, P, 0, 0, 0, 1), False),     # periodic x of two cells
    ((33, 31, 29), TANK, True),                 # odd everywhere
    ((64, 1, 40), TANK, False),                 # a single row
    ((48, 40, 1), (1, 0, 0, 1, 0, 1), False),   # a single plane
    ((600, 6, 9), TANK, True),                  # rows longer than a workgroup
    ((40, 12, 10), (P, P, P, P, 0, 1), True),   # both axes periodic
    ((24, 2, 9), (0, 1, P, P, 1, 0), False),    # periodic y of two rows
    ((36, 50, 20), (P, P, 0, 0, 0, 0), True),   # singular
    ((30, 26, 22), (P, P, P, P, 0, 0), False),  # singular, periodic both ways
    ((20, 24, 28), (1, 1, 1, 1, 1, 1), True),   # p = 0 everywhere
    ((97, 66, 45), (1, 0, 0, 1, 0, 1), True),   # several bricks along y and z, ragged both
    ((128, 72, 50), TANK, True),                # eight planes a brick, ragged
]


@pytest.mark.parametrize("shape,bc,wedge", CASES, ids=lambda v: str(v))
@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "ir"])
def test_resident_parity(orc, F, torch_dev, shape, bc, wedge, precision):
    case = _case(F, shape, bc, wedge)
    _say(f"case resident {shape} bc={bc} wedge={wedge} precision={precision}")
    tol = 1e-8
    p, st = _solve(torch_dev, case, tol=tol, precision=precision)
    assert st["status"] == 0, st
    rr = orc.relres(case.rho, case.mask, case.bc, case.h, case.rhs, p)
    assert rr <= tol, (rr, st)
    ref = orc.pcg(case.rho, case.mask, case.bc, case.h, case.rhs, tol=1e-12)
    scale = np.abs(ref.p).max()
    assert np.abs(p - ref.p).max() <= 1e-6 * scale
    assert np.all(p[case.mask.astype(bool)] == 0.0)
    if precision == 0:
        o8 = orc.pcg(case.rho, case.mask, case.bc, case.h, case.rhs, tol=tol)
        assert abs(st["iters"] - o8.iters) <= max(2, 0.02 * o8.iters), (st, o8.iters)
    # the tiles of a launch per pass solve the same system
    pf, stf = _solve(torch_dev, case, tol=tol, precision=precision, flags=FLAT_TILES)
    assert stf["status"] == 0
    assert np.abs(p - pf).max() <= 1e-6 * scale


@pytest.mark.parametrize("shape,bc", [((33, 31, 29), TANK), ((97, 66, 45), (1, 0, 0, 1, 0, 1)),
                                      ((40, 12, 10), (P, P, P, P, 0, 1))], ids=lambda v: str(v))
@pytest.mark.parametrize("k", [1, 2, 33, 100])
def test_resident_capped_iterate(orc, F, torch_dev, shape, bc, k):
    """Capped at k iterations (within the first launch, at its end, in a later
    one) the answer is the oracle's k-th iterate."""
    case = _case(F, shape, bc)
    _say(f"case resident capped {shape} k={k}")
    ref = orc.pcg(case.rho, case.mask, case.bc, case.h, case.rhs, tol=1e-30, maxit=k)
    scale = np.abs(ref.p).max()
    p, st = _solve(torch_dev, case, tol=1e-30, maxit=k)
    assert st["status"] == 1 and st["iters"] == k, st
    assert np.abs(p - ref.p).max() <= 1e-10 * scale


def test_resident_launch_length_and_start(orc, F, torch_dev):
    """The answer does not depend on how many iterations a launch takes; a
    warm start and a second solve on the context agree with it."""
    torch, dev = torch_dev
    from paper_1410_1942_amd.solver import Solver
    case = _case(F, (61, 47, 39), TANK)
    p1, s1 = _solve(torch_dev, case, check_every=1)
    p2, s2 = _solve(torch_dev, case, check_every=64)
    assert s1["iters"] == s2["iters"] and np.array_equal(p1, p2)
    ref = orc.pcg(case.rho, case.mask, case.bc, case.h, case.rhs, tol=1e-12)
    scale = np.abs(ref.p).max()
    pw, sw = _solve(torch_dev, case, p0=ref.p)
    assert sw["status"] == 0 and sw["iters"] <= 2
    assert np.abs(pw - ref.p).max() <= 1e-6 * scale
    s = Solver(_to(torch, dev, case.rho), _to(torch, dev, case.mask), case.bc, case.h)
    rhs = _to(torch, dev, case.rhs)
    a, _ = s.solve(rhs)
    b, _ = s.solve(rhs)
    s.close()
    assert torch.equal(a, b) and np.array_equal(a.cpu().numpy(), p1)
