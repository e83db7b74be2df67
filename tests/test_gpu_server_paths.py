"""Chunks of several steps run as one sequence, on each launch path of the server's members:
batches of two and three whose members join and leave between chunks, with output points
inside and at the end of chunks, give the plain solver's fields and invariants bit for bit.
"""
import math

import numpy as np
import pytest

from paper_2210_06232_amd import inputs

pytestmark = pytest.mark.gpu

BOX = (0.0, 2 * math.pi, 0.0, 4 * math.pi, 0.0, 3 * math.pi)
# in place through the (x, z) plane pass (one workgroup a plane, and several planes a
# workgroup), through the (y, z) plane pass, through the separate passes; and the separate
# passes with a work buffer (states of 64 MiB or more)
SHAPES = [(32, 24, 32), (128, 12, 96), (12, 16, 16), (8, 32, 48), (48, 256, 128)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_batched_chunks_equal_the_solver_bitwise(shape, prec):
    from paper_2210_06232_amd import eifp as m
    H, E = inputs.random_fields(shape, BOX, workload=61, p=2.0)
    H2, E2 = H[:, ::-1].copy(), E[:, ::-1].copy()
    # (fields, eps, tau, steps, cadence); a long first solve keeps the batch busy
    reqs = [((H, E), 1.1, 0.05, 3000, 1500), ((H2, E2), 1.7, 0.03, 11, 0), ((H, E), 1.4, 0.02, 24, 5),
            ((H2, E2), 1.2, 0.04, 33, 33), ((H, E), 1.9, 0.06, 5, 1)]
    with m.Server(4 << 30, 3) as sv:
        ids = [sv.submit(F[0], F[1], BOX, 1.0, eps, tau, n, cad, prec, i, m.EIFP_REQ_KEEP_RESULT)
               for i, (F, eps, tau, n, cad) in enumerate(reqs)]
        sv.drain(60000)
        evs = []
        while True:
            got = sv.poll(4096, 0)
            if not got:
                break
            evs += got
        st = sv.stats()
        assert st["completed"] == len(reqs) and st["failed"] == 0 and st["peak_running"] >= 2
        res = [sv.fields(i, shape) for i in ids]
    for i, (F, eps, tau, n, cad) in enumerate(reqs):
        mine = {e["step"]: e["inv"] for e in evs if e["tag"] == i}
        assert sorted(mine) == sorted(set(range(cad, n, cad) if cad else ()) | {n})
        with m.Solver(F[0], F[1], BOX, 1.0, eps, prec) as s:
            at = 0
            for step in sorted(mine):
                s.step(tau, step - at)
                at = step
                inv = s.invariants()
                assert {k: v for k, v in mine[step].items() if k != "t"} == {k: v for k, v in inv.items() if k != "t"}
            Hs, Es = s.fields()
        assert res[i][2] == n
        np.testing.assert_array_equal(res[i][0], Hs)
        np.testing.assert_array_equal(res[i][1], Es)
