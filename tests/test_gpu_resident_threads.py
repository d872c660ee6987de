"""Solves on the chip from several threads at once, each with its own context
(or batch) and stream: grids of one kernel shape whose workgroups take
different shares of LDS, and of different shapes, in both precisions.  Every
answer must be, bit for bit, the one of the same solve alone."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TANK = (0, 0, 0, 0, 0, 1)
# rows and bricks of different lengths: LDS of 10 .. 100 KB in neighbouring shapes
SHAPES = [(97, 66, 45), (33, 31, 29), (200, 24, 30), (64, 64, 64)]


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def test_contexts_on_threads(F):
    import torch
    from paper_1410_1942_amd import _lib as L
    from paper_1410_1942_amd.solver import Batch, Solver
    cases = [F.make_two_phase(*s, surface_seed=61, velocity_seed=62, wedge=F.Wedge(), bc=TANK)
             for s in SHAPES]
    dev = [tuple(_t(a) for a in (c.rho, c.mask, c.rhs)) for c in cases]
    torch.cuda.synchronize()

    def single(i, precision, stream):
        rho, mask, rhs = dev[i]
        s = Solver(rho, mask, cases[i].bc, cases[i].h, precision=precision, stream=stream)
        p = torch.zeros_like(rhs)
        torch.cuda.synchronize()
        out = []
        for _ in range(3):
            s.solve(rhs, p=p, tol=1e-8)
            out.append(p.cpu())
        s.close()
        return out

    def batch(i, precision, stream):
        b = Batch(64 << 20, 4, precision=precision, stream=stream)
        ps, slots = [torch.zeros_like(d[2]) for d in dev], []
        torch.cuda.synchronize()
        for c, d, p in zip(cases, dev, ps):
            code, slot = b.admit(d[0], d[1], c.bc, c.h, d[2], p, tol=1e-8)
            assert code == L.OK
            slots.append(slot)
        while b.step(1):
            pass
        for slot in slots:
            assert b.poll(slot)[0] == L.OK
            b.release(slot)
        out = [p.cpu() for p in ps]
        b.close()
        return out

    jobs = [(single, i, prec) for i in range(len(cases)) for prec in (0, 1)] + [(batch, 0, 1)]
    print("case resident alone", flush=True)
    alone = [f(i, prec, torch.cuda.Stream()) for f, i, prec in jobs]
    print("case resident on threads", flush=True)
    got, errors = [None] * len(jobs), []

    def work(k):
        f, i, prec = jobs[k]
        try:
            got[k] = f(i, prec, torch.cuda.Stream())
        except Exception as e:          # reported by the test's own thread
            errors.append((jobs[k], e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for job, a, b in zip(jobs, alone, got):
        for x, y in zip(a, b):
            assert torch.equal(x, y), job
