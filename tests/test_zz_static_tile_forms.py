"""The allocation-free entry point on the tile passes (GPU): grids small enough
for its fixed array iterate on the chip by default, so each tile form is asked
for.  Calls in a row, each on a smaller grid than the one before and each equal
to the workspace path's result bit for bit (the same kernels in the same
order), and below the tolerance by the oracle's residual."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "ir"])
@pytest.mark.parametrize("warm", [False, True], ids=["cold", "warm"])
def test_static_tile_forms(orc, F, precision, warm):
    import torch
    from paper_1410_1942_amd import _lib as L
    from paper_1410_1942_amd.solver import Solver, solve_static
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    wide = 128 if precision == 0 else 256      # one tile across
    forms = [((200, 24, 30), L.PLANE_TILES, (wide, 4, 1)),
             ((wide, 2560 // wide, 17), L.PLANE_TILES | L.TWO_SWEEPS, (wide, 4, 2)),
             ((37, 29, 23), L.NARROW_TILES, (64, 4, 1)),
             ((36, 25, 23), L.FLAT_TILES, (0, 0, 2)),
             ((wide, 1024 // wide, 9), L.PLANE_TILES | L.NO_DENSITY_CLASSES, (wide, 4, 1)),
             ((21, 20, 19), L.FLAT_TILES, (0, 0, 2))]
    for shape, flags, form in forms:
        print(f"case static tile form {shape} flags={flags} prec={precision} warm={warm}", flush=True)
        case = F.make_two_phase(*shape, surface_seed=51, velocity_seed=52, wedge=F.Wedge())
        rho, mask, rhs = t(case.rho), t(case.mask), t(case.rhs)
        ref = orc.pcg(case.rho, case.mask, case.bc, case.h, case.rhs, tol=1e-12)
        start = t(1.25 * ref.p) if warm else torch.full_like(rhs, np.nan)
        p_s, st_s = solve_static(rho, mask, case.bc, case.h, rhs, p=start.clone(), tol=1e-8,
                                 precision=precision, flags=flags | (L.WARM_START if warm else 0))
        s = Solver(rho, mask, case.bc, case.h, precision=precision, flags=flags)
        try:
            assert s.tile_form_ex() == form
            p_w, st_w = s.solve(rhs, p=start.clone(), tol=1e-8, warm=warm)
        finally:
            s.close()
        assert st_s["status"] == 0 and st_s["iters"] == st_w["iters"], (st_s, st_w)
        assert torch.equal(p_s, p_w)
        p = p_s.cpu().numpy()
        assert orc.relres(case.rho, case.mask, case.bc, case.h, case.rhs, p) <= 1e-8
        assert np.abs(p - ref.p).max() <= 1e-6 * np.abs(ref.p).max()
