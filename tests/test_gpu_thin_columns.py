"""Source, projection and divergence on grids of few columns, where the columns
of many chunks of planes share a workgroup, and at the edges of that form (15
and 16 columns, one below and above a whole tile, 1023 to 1025), against the
reference, face by face.  Tolerances are those of the other tests of these
kernels: the operations are the reference's, so a rounding or two of the
largest value."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 4099), (3, 2, 1001), (5, 5, 300), (15, 1, 77), (16, 1, 77),
                                   (51, 5, 9), (16, 16, 33), (257, 1, 21), (341, 3, 9),
                                   (32, 32, 10), (41, 25, 6), (37, 27, 1), (64, 64, 2)], ids=str)
@pytest.mark.parametrize("coded", [True, False], ids=["classes", "densities"])
def test_thin_columns(orc, shape, coded):
    import torch
    from paper_1410_1942_amd import _lib as L
    from paper_1410_1942_amd.solver import Solver
    print(f"case thin columns {shape} coded={coded}", flush=True)
    dev = torch.device("cuda:0")
    nx, ny, nz = shape
    rng = np.random.default_rng(nx + 7 * ny + 31 * nz)
    bc, h, dt = (1, 0, 0, 1, 0, 1), 0.25, 1e-3
    rho = np.where(rng.random((nz, ny, nx)) < 0.5, 1000.0, 1.2)
    mask = (rng.random(rho.shape) < 0.2).astype(np.uint8)
    faces = lambda: [rng.uniform(-1, 1, s) for s in ((nz, ny, nx + 1), (nz, ny + 1, nx), (nz + 1, ny, nx))]
    a, b, p = faces(), faces(), rng.uniform(-1, 1, rho.shape)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev)
    s = Solver(t(rho), t(mask), bc, h,
               flags=L.SKIP_CONNECTIVITY_CHECK | (0 if coded else L.NO_DENSITY_CLASSES))
    try:
        both = [x + y for x, y in zip(a, b)]
        for add, vel in ((None, a), ([t(y) for y in b], both)):
            got = s.rhs(dt, *(t(x) for x in a), add=add).cpu().numpy()
            want = orc.source(*vel, h, dt, mask)
            assert np.abs(got - want).max() <= 1e-15 * np.abs(want).max()
            out = [torch.empty_like(t(x)) for x in a]
            s.project(t(p), dt, *(t(x) for x in a), add=add, weight=0.5, out=out)
            ref = [0.5 * x for x in orc.project(rho, mask, bc, h, dt, p, *vel)]
            scale = max(np.abs(x).max() for x in ref)
            for x, y in zip(out, ref):
                assert np.abs(x.cpu().numpy() - y).max() <= 1e-13 * scale
        l2, mx = s.divergence(*(t(x) for x in a))
    finally:
        s.close()
    div = orc.divergence(*a, h)[mask == 0]
    assert abs(l2 - np.linalg.norm(div)) <= 1e-12 * np.linalg.norm(div)
    assert abs(mx - np.abs(div).max()) <= 1e-12 * np.abs(div).max()
