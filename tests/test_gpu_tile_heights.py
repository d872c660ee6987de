"""Tile heights chosen for an even load (GPU): every tile form, with room for
more tiles than the least workspace holds and without, on grids whose tiles
leave remainders in every direction.  The reference's residual of what is
returned must be below the tolerance, and the two cuts, which differ only in
the order of their sums, must take the same number of iterations (one more or
less) to answers within the solve's tolerance of each other (1e-6 of the
largest pressure at 1e-9)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(130, 90, 97), (97, 105, 110), (512, 300, 7)], ids=str)
@pytest.mark.parametrize("form", ["FLAT_TILES", "PLANE_TILES", "NARROW_TILES"])
@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "ir"])
def test_cuts(orc, F, monkeypatch, shape, form, precision):
    import torch
    from paper_1410_1942_amd import _lib as L
    from paper_1410_1942_amd import solver
    dev = torch.device("cuda:0")
    print(f"case tile heights {shape} {form} prec={precision}", flush=True)
    case = F.make_two_phase(*shape, surface_seed=3, velocity_seed=4, wedge=F.Wedge())
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    got = []
    for spare in (solver._SPARE_BYTES, 0):
        monkeypatch.setattr(solver, "_SPARE_BYTES", spare)
        s = solver.Solver(t(case.rho), t(case.mask), case.bc, case.h, precision=precision,
                          flags=getattr(L, form))
        try:
            p, st = s.solve(t(case.rhs), tol=1e-9)
        finally:
            s.close()
        p = p.cpu().numpy()
        assert orc.relres(case.rho, case.mask, case.bc, case.h, case.rhs, p) <= 1e-9
        got.append((p, st["iters"]))
    (a, ia), (b, ib) = got
    assert np.abs(a - b).max() <= 1e-6 * np.abs(a).max()
    if precision == 0:
        assert abs(ia - ib) <= 1
