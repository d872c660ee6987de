"""Periodic and singular problems on the tile passes (GPU): small grids iterate
on the chip by default, so each tile form is asked for (a form that a grid does
not allow falls back to consecutive cells), with classes and per-cell
densities, both precisions.  The bar is that of the default form's test."""
import numpy as np
import pytest

from tests.test_gpu_periodic import CASES

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,bc,wedge", CASES, ids=str)
@pytest.mark.parametrize("form", ["FLAT_TILES", "PLANE_TILES", "NARROW_TILES"])
@pytest.mark.parametrize("coded", [True, False], ids=["classes", "densities"])
@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "ir"])
def test_periodic_tiles(orc, F, shape, bc, wedge, form, coded, precision):
    import torch
    from paper_1410_1942_amd import _lib as L
    from paper_1410_1942_amd.solver import Solver
    print(f"case periodic tiles {shape} bc={bc} {form} coded={coded} prec={precision}", flush=True)
    nx, ny, nz = shape
    case = F.make_two_phase(nx, ny, nz, surface_seed=71, velocity_seed=72,
                            wedge=F.Wedge() if wedge else None, bc=bc)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    tol = 1e-8
    s = Solver(t(case.rho), t(case.mask), case.bc, case.h, precision=precision,
               flags=getattr(L, form) | (0 if coded else L.NO_DENSITY_CLASSES))
    p, st = s.solve(t(case.rhs), tol=tol, raise_on_error=False)
    s.close()
    p = p.cpu().numpy()
    assert st["status"] == 0, st
    rr = orc.relres(case.rho, case.mask, case.bc, case.h, case.rhs, p)
    assert rr <= tol, rr
    assert abs(st["rel_res_true"] - rr) <= 1e-3 * rr + 1e-15
    ref = orc.pcg(case.rho, case.mask, case.bc, case.h, case.rhs, tol=1e-12)
    scale = np.abs(ref.p).max()
    assert np.abs(p - ref.p).max() <= 1e-6 * scale
    fluid = case.mask == 0
    assert np.all(p[~fluid] == 0.0)
    if 1 not in bc:
        assert abs(p[fluid].mean()) <= 1e-12 * scale
    if precision == 0:
        o8 = orc.pcg(case.rho, case.mask, case.bc, case.h, case.rhs, tol=tol)
        assert abs(st["iters"] - o8.iters) <= max(2, 0.02 * o8.iters), (st, o8.iters)
