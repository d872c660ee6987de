"""What a context says of its next solve (GPU): whether it iterates on the chip,
by grid, flags, coefficients, fractions and timing; and that the tile form asked
for is the one that runs then (its own answer, bit for bit, with the launches
timed and not)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1], ids=["fp64", "ir"])
def test_resident_form(F, precision):
    import torch
    from paper_1410_1942_amd import _lib as L
    from paper_1410_1942_amd.solver import Solver
    print(f"case resident form prec={precision}", flush=True)
    case = F.make_two_phase(33, 31, 29, surface_seed=41, velocity_seed=42, wedge=F.Wedge(),
                            fractions=True)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    rhs = t(case.rhs)

    def make(flags=0, **kw):
        return Solver(t(case.rho), t(case.mask), case.bc, case.h, precision=precision, flags=flags, **kw)

    for flags, kw, on in ((0, {}, True), (L.NO_DENSITY_CLASSES, {}, True), (L.FLAT_TILES, {}, False),
                          (L.PLANE_TILES, {}, False), (L.NARROW_TILES, {}, False),
                          (L.TWO_SWEEPS, {}, False), (0, {"tz": 8}, False),
                          (0, {"grid_blocks": 256}, False), (L.FRACTIONS, {}, False)):
        s = make(flags, **kw)
        g, c = s.resident_form()
        assert (g > 1 and c >= 1) if on else (g, c) == (0, 0), (flags, kw, g, c)
        if flags == L.FRACTIONS:
            s.set_fractions(*(t(a) for a in case.frac))
            assert s.resident_form()[0] > 1
            s.set_fractions()
            assert s.resident_form() == (0, 0)
        s.close()
    s, tiles = make(), make(grid_blocks=256)
    s.set_timing(True)
    assert s.resident_form() == (0, 0)
    got, want = s.solve(rhs)[0].clone(), tiles.solve(rhs)[0]
    assert torch.equal(got, want) and s.last_timing()[2] > 0
    s.set_timing(False)
    assert s.resident_form()[0] > 1
    s.close()
    tiles.close()
    rho = torch.ones((200, 200, 200), dtype=torch.float64, device="cuda:0")   # 8 million cells
    s = Solver(rho, None, (0, 0, 0, 0, 0, 1), 0.01, precision=precision)
    assert s.resident_form() == (0, 0)
    s.close()
