"""Solves on the chip whose sums come near the smallest numbers of FP64
(densities of 1e-9, sources down to 1e-150).  Powers of two scale every
quantity of the iteration exactly until it leaves the normal range, so the
solve has to take the iterations of the unscaled one, give or take two for the
bits that numbers below that range have lost, to a residual below the
tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["classes", "densities", "cut"])
@pytest.mark.parametrize("shape", [(7, 5, 6), (24, 20, 16)], ids=str)
def test_scaled_source(F, kind, shape):
    import torch
    from paper_1410_1942_amd import _lib as L
    from paper_1410_1942_amd.solver import Solver
    dev = torch.device("cuda:0")
    case = F.make_two_phase(*shape, surface_seed=1, velocity_seed=2, wedge=F.Wedge(),
                            fractions=kind == "cut")
    if kind == "densities":
        case.rho = case.rho * (1.0 + 0.3 * np.random.default_rng(4).random(case.rho.shape))
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    want = None
    for m, k in ((0, 0), (-40, -480), (-40, -490), (-40, -495), (-40, -500), (-40, -505), (40, 440)):
        print(f"case resident range {shape} {kind} rho 2^{m} rhs 2^{k}", flush=True)
        s = Solver(t(case.rho * 2.0 ** m), t(case.mask), case.bc, case.h,
                   flags=L.FRACTIONS if kind == "cut" else 0)
        if kind == "cut":
            s.set_fractions(*(t(a) for a in case.frac))
        p, st = s.solve(t(case.rhs * 2.0 ** k), tol=1e-4, raise_on_error=False)
        s.close()
        want = want or st["iters"]
        assert st["status"] == 0 and st["rel_res_true"] <= 1e-4, st
        assert abs(st["iters"] - want) <= 2, (st, want)
