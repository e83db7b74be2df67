"""Batch tables of the server, run without a GPU: they are sized for the members the budget
has room for, so that a large batch limit does not shut out requests that fit.
"""
import math
import os

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2210_06232_amd", "libeifp.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libeifp.so not built")

CUBE = (0.0, 2 * math.pi, 0.0, 2 * math.pi, 0.0, 2 * math.pi)


@pytest.mark.parametrize("flags", [0, 4], ids=["stepped", "anchored"])
@pytest.mark.parametrize("shape,prec", [((128, 16, 128), "fp32"), ((96, 64, 96), "fp64"), ((16, 16, 16), "fp64")])
def test_requests_that_fit_twice_are_taken_at_any_batch_limit(shape, prec, flags):
    from paper_2210_06232_amd import eifp as m
    z = np.zeros((3, shape[2], shape[1], shape[0]))
    budget = 2 * m.eifp_server_footprint(*shape, prec, flags)
    for max_batch in (1, 1024):
        with m.Server(budget, max_batch, m.EIFP_SERVER_DRY_RUN) as sv:
            for i in range(5):
                sv.submit(z, z, CUBE, tau=0.1, nsteps=3, prec=prec, tag=i, flags=flags)
            sv.drain(20000)
            st = sv.stats()
        assert st["completed"] == 5 and st["failed"] == 0
        assert st["peak_bytes"] <= budget
