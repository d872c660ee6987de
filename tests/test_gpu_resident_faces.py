"""Solves on the chip with face coefficients of their own (GPU): densities
that are not coded by class, and cut cells.  Shapes sit at the edges of the
bricks (one brick, ragged last bricks along y and z, rows of one cell and
longer than a workgroup, the most cells a thread of each precision) under
every wall kind and periodic axes.  The iteration is the textbook one, so a
capped FP64 solve is the oracle's k-th iterate (1e-10 of its largest value,
the bar of the class-coded form), and a converged one has the oracle's
residual below the tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TANK = (0, 0, 0, 0, 0, 1)
P = 2

CASES = [
    ((7, 5, 6), TANK), ((1, 3, 40), (0, 0, 0, 1, 1, 0)), ((2, 9, 8), (P, P, 0, 0, 0, 1)),
    ((33, 31, 29), TANK), ((48, 40, 1), (1, 0, 0, 1, 0, 1)), ((600, 6, 9), (0, 1, 0, 0, 0, 0)),
    ((40, 12, 10), (P, P, P, P, 0, 1)), ((24, 2, 9), (0, 1, P, P, 1, 0)),
    ((20, 24, 28), (1, 1, 1, 1, 1, 1)), ((97, 66, 45), (1, 0, 0, 1, 0, 1)),
    ((128, 72, 50), (0, 1, 0, 1, 0, 1)),
]


def _make(F, shape, bc, kind):
    nx, ny, nz = shape
    case = F.make_two_phase(nx, ny, nz, surface_seed=21, velocity_seed=22, wedge=F.Wedge(), bc=bc,
                            fractions=kind == "cut")
    if kind == "densities":
        case.rho = case.rho * (1.0 + 0.3 * np.random.default_rng(4).random(case.rho.shape))
        case.frac = None
    return case


def _solve(case, precision, **kw):
    import torch
    from paper_1410_1942_amd import _lib as L
    from paper_1410_1942_amd.solver import Solver
    dev = torch.device("cuda:0")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    s = Solver(t(case.rho), t(case.mask), case.bc, case.h, precision=precision,
               flags=L.FRACTIONS if case.frac else 0)
    try:
        if case.frac:
            s.set_fractions(*(t(a) for a in case.frac))
        assert s.density_classes() == 0
        p, st = s.solve(t(case.rhs), raise_on_error=False, **kw)
        return p.cpu().numpy(), st
    finally:
        s.close()


@pytest.mark.parametrize("shape,bc", CASES, ids=str)
@pytest.mark.parametrize("kind", ["densities", "cut"])
def test_capped_iterate(orc, F, shape, bc, kind):
    print(f"case resident faces {shape} bc={bc} {kind}", flush=True)
    case = _make(F, shape, bc, kind)
    if case.frac is None and len(np.unique(case.rho[case.mask == 0])) <= 14:
        pytest.skip("few enough densities for classes")
    for k in (1, 33):
        ref = orc.pcg(case.rho, case.mask, case.bc, case.h, case.rhs, tol=1e-30, maxit=k,
                      frac=case.frac)
        p, st = _solve(case, 0, tol=1e-30, maxit=k)
        if ref.iters < k:       # the oracle ran out of residual before the cap
            continue
        assert st["iters"] == k, st
        assert np.abs(p - ref.p).max() <= 1e-10 * np.abs(ref.p).max()


@pytest.mark.parametrize("shape,bc", CASES + [((150, 141, 60), TANK)], ids=str)
@pytest.mark.parametrize("kind", ["densities", "cut"])
@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "ir"])
def test_converged(orc, F, shape, bc, kind, precision):
    print(f"case resident faces {shape} bc={bc} {kind} prec={precision}", flush=True)
    case = _make(F, shape, bc, kind)
    if case.frac is None and len(np.unique(case.rho[case.mask == 0])) <= 14:
        pytest.skip("few enough densities for classes")
    tol = 1e-9
    p, st = _solve(case, precision, tol=tol)
    assert st["status"] == 0, st
    rr = orc.relres(case.rho, case.mask, case.bc, case.h, case.rhs, p, frac=case.frac)
    assert rr <= tol, rr
    assert abs(st["rel_res_true"] - rr) <= 1e-3 * rr + 1e-15
    assert np.all(p[case.mask.astype(bool)] == 0.0)
