"""The cut-cell tile passes (GPU) on grids that would iterate on the chip by
default: consecutive tiles asked for, keys by density class and per-cell
densities, one, two and four cells a thread, one tile and several with a
remainder a column, every wall kind and periodic wraps.  A capped FP64 solve is
the oracle's k-th iterate (1e-10 of its largest value); a converged one has the
oracle's residual below the tolerance and its answer (1e-6 at 1e-8)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TANK = (0, 0, 0, 0, 0, 1)
P = 2

CASES = [
    ((33, 20, 17), TANK),                    # odd rows: one cell a thread
    ((35, 18, 24), (P, P, 0, 0, 0, 1)),      # odd and periodic
    ((34, 21, 3), (1, 1, 1, 1, 1, 1)),       # pairs in both precisions
    ((34, 12, 11), (P, P, P, P, 1, 0)),      # pairs, periodic both ways
    ((36, 20, 17), (P, P, P, P, 0, 1)),      # pairs and quads, periodic both ways
    ((36, 23, 40), (1, 0, 0, 1, 0, 1)),      # pairs and quads, several tiles a column
    ((30, 22, 18), (P, P, 0, 0, 0, 0)),      # singular
    ((40, 34, 30), TANK),
]


def _make(F, shape, bc):
    nx, ny, nz = shape
    return F.make_two_phase(nx, ny, nz, surface_seed=7, velocity_seed=8, wedge=F.Wedge(), bc=bc,
                            fractions=True)


def _solve(case, precision, coded, **kw):
    import torch
    from paper_1410_1942_amd import _lib as L
    from paper_1410_1942_amd.solver import Solver
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    s = Solver(t(case.rho), t(case.mask), case.bc, case.h, precision=precision,
               flags=L.FRACTIONS | L.FLAT_TILES | (0 if coded else L.NO_DENSITY_CLASSES))
    try:
        s.set_fractions(*(t(a) for a in case.frac))
        p, st = s.solve(t(case.rhs), raise_on_error=False, **kw)
        return p.cpu().numpy(), st
    finally:
        s.close()


@pytest.mark.parametrize("shape,bc", CASES, ids=str)
@pytest.mark.parametrize("coded", [True, False], ids=["classes", "densities"])
def test_capped_iterate(orc, F, shape, bc, coded):
    print(f"case cut tile passes capped {shape} bc={bc} coded={coded}", flush=True)
    case = _make(F, shape, bc)
    for k in (1, 2, 3, 33):     # x catches up every third iteration
        ref = orc.pcg(case.rho, case.mask, case.bc, case.h, case.rhs, tol=1e-30, maxit=k,
                      frac=case.frac)
        p, st = _solve(case, 0, coded, tol=1e-30, maxit=k)
        assert ref.iters == k and st["iters"] == k, (ref.iters, st)
        assert np.abs(p - ref.p).max() <= 1e-10 * np.abs(ref.p).max()


@pytest.mark.parametrize("shape,bc", CASES, ids=str)
@pytest.mark.parametrize("coded", [True, False], ids=["classes", "densities"])
@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "ir"])
def test_converged(orc, F, shape, bc, coded, precision):
    print(f"case cut tile passes {shape} bc={bc} coded={coded} prec={precision}", flush=True)
    case = _make(F, shape, bc)
    p, st = _solve(case, precision, coded, tol=1e-8)
    assert st["status"] == 0, st
    rr = orc.relres(case.rho, case.mask, case.bc, case.h, case.rhs, p, frac=case.frac)
    assert rr <= 1e-8, rr
    assert abs(st["rel_res_true"] - rr) <= 1e-3 * rr + 1e-15
    ref = orc.pcg(case.rho, case.mask, case.bc, case.h, case.rhs, tol=1e-12, frac=case.frac)
    assert np.abs(p - ref.p).max() <= 1e-6 * np.abs(ref.p).max()
    assert np.all(p[case.mask.astype(bool)] == 0.0)
