"""Large field arrays cross the host in pieces on several threads: every value of a
submitted field is checked, the first NaN or infinity reported by its flat index, and a
served solve's fields come back whole, the same as the plain solver's.
"""
import math

import numpy as np
import pytest

from paper_2210_06232_amd import inputs

SHAPE = (64, 64, 96)  # 3 * 64 * 64 * 96 = 1179648 values an array: 9 MB, several threads
N3 = 3 * SHAPE[0] * SHAPE[1] * SHAPE[2]
DOMAIN = (0.0, 2 * math.pi, 0.0, 2 * math.pi, 0.0, 3 * math.pi)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("at", [(0, 0), (0, 4095), (0, 4096), (1, 294911), (1, 294912), (1, N3 - 1), (0, N3 - 1)],
                         ids=lambda a: f"{a[0]}-{a[1]}")
def test_submit_reports_the_first_nonfinite_value(at, prec):
    from paper_2210_06232_amd import eifp
    nx, ny, nz = SHAPE
    f = [np.ones((3, nz, ny, nx)), np.ones((3, nz, ny, nx))]
    part, q = at
    f[part].reshape(-1)[q] = math.nan
    if part == 0 and q + 5000 < N3:
        f[0].reshape(-1)[q + 5000] = math.inf  # a later one is not the one reported
    with eifp.Server(10 ** 9, 4, eifp.EIFP_SERVER_DRY_RUN) as sv:
        with pytest.raises(eifp.EifpError) as ei:
            sv.submit(f[0], f[1], DOMAIN, nsteps=1, prec=prec)
        assert ei.value.status == eifp.EIFP_ERR_NONFINITE
        assert str(ei.value).endswith(f"flat index {part * N3 + q}")
        f[part].reshape(-1)[q] = 1e308  # large but finite
        if part == 0 and q + 5000 < N3:
            f[0].reshape(-1)[q + 5000] = -5e-324
        if prec == "fp64":
            sv.submit(f[0], f[1], DOMAIN, nsteps=1, prec=prec)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(32, 32, 32), (96, 96, 128), (128, 128, 192)], ids=lambda s: "x".join(map(str, s)))
def test_served_fields_equal_the_solvers(shape, prec):
    # below the staged copies, one piece, and several pieces with a ragged last one
    from paper_2210_06232_amd import eifp
    H, E = inputs.white_noise_fields(shape, seed=77)
    with eifp.Solver(H, E, DOMAIN, 1.0, 1.5, prec) as s:
        s.step(0.1, 3)
        want = s.fields()
    with eifp.Server(8 * 10 ** 9, 4) as sv:
        for _ in range(2):
            i = sv.submit(H, E, DOMAIN, 1.0, 1.5, 0.1, 3, 0, prec, 0, eifp.EIFP_REQ_KEEP_RESULT)
            sv.drain(60000)
            got = sv.fields(i, shape)
            np.testing.assert_array_equal(got[0], want[0])
            np.testing.assert_array_equal(got[1], want[1])
            sv.release(i)
