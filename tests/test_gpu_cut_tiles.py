"""The cut-cell passes (GPU): keys by density class and per-cell densities,
one, two and four cells a thread, one tile and several with a remainder a
column, and tile heights that leave one tile a CU (160 x 140 x 97: FP64 5
chunks of 20 planes instead of 7 of 16).  The reference recomputes the
residual of what is returned, in FP64 with its own operator: it must be below
the solve's tolerance (its own rounding is 1e-16 of the source), and clearing
the fractions must bring back the bits of the solve before they were set."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

P = 2


@pytest.mark.parametrize("shape,bc", [((33, 20, 17), (0, 0, 0, 0, 0, 1)),
                                      ((34, 21, 3), (1, 1, 1, 1, 1, 1)),
                                      ((36, 20, 17), (P, P, P, P, 0, 1)),
                                      ((160, 140, 97), (0, 1, 0, 1, 0, 1))], ids=str)
@pytest.mark.parametrize("coded", [True, False], ids=["classes", "densities"])
@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "ir"])
def test_cut_cell_passes(orc, F, shape, bc, coded, precision):
    import torch
    from paper_1410_1942_amd import _lib as L
    from paper_1410_1942_amd.solver import Solver
    dev = torch.device("cuda:0")
    print(f"case cut tiles {shape} bc={bc} coded={coded} prec={precision}", flush=True)
    nx, ny, nz = shape
    case = F.make_two_phase(nx, ny, nz, surface_seed=7, velocity_seed=8, wedge=F.Wedge(), bc=bc,
                            fractions=True)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    tol, rhs = 1e-9, t(case.rhs)
    s = Solver(t(case.rho), t(case.mask), case.bc, case.h, precision=precision,
               flags=L.FRACTIONS | (0 if coded else L.NO_DENSITY_CLASSES))
    try:
        before, _ = s.solve(rhs, tol=tol)
        s.set_fractions(*(t(a) for a in case.frac))
        p, st = s.solve(rhs, tol=tol)
        s.set_fractions()
        after, _ = s.solve(rhs, tol=tol)
    finally:
        s.close()
    rr = orc.relres(case.rho, case.mask, case.bc, case.h, case.rhs, p.cpu().numpy(),
                    frac=case.frac)
    assert rr <= tol, rr
    assert abs(st["rel_res_true"] - rr) <= 1e-3 * rr + 1e-15
    assert torch.equal(before, after)
