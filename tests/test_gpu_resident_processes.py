"""Two programs on one device (GPU), each solving on a grid whose workgroups fill
most of it.  The runtime lets only one of them launch all of its workgroups at
once.  Every solve of both must end with the answer (1e-6 of the largest
pressure from the tile passes' at 1e-8), on the chip or off it."""
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _child():
    sys.path.insert(0, ROOT)
    import torch
    from paper_1410_1942_amd import fields as F
    from paper_1410_1942_amd.solver import Solver
    case = F.make_two_phase(128, 100, 96, surface_seed=1, velocity_seed=2, wedge=F.Wedge())
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    rho, mask, rhs = t(case.rho), t(case.mask), t(case.rhs)
    tiles = Solver(rho, mask, case.bc, case.h, grid_blocks=512)
    want = tiles.solve(rhs)[0].clone()
    scale = float(want.abs().max())
    for _ in range(3):
        s = Solver(rho, mask, case.bc, case.h)
        for _ in range(8):
            p, st = s.solve(rhs)
            assert st["status"] == 0, st
            assert float((p - want).abs().max()) <= 1e-6 * scale
        print("on the chip" if s.resident_form()[0] else "off the chip", flush=True)
        s.close()
    tiles.close()
    print("done", flush=True)


def test_two_processes():
    print("case two processes", flush=True)
    ps = [subprocess.Popen([sys.executable, "-u", os.path.abspath(__file__)], stdout=subprocess.PIPE,
                           stderr=subprocess.STDOUT, text=True) for _ in range(2)]
    out = [p.communicate(timeout=100)[0] for p in ps]
    for p, o in zip(ps, out):
        print(o, flush=True)
        assert p.returncode == 0 and "done" in o, o


if __name__ == "__main__":
    _child()
