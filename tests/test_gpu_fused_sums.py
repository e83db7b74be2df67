"""The sums of the fused pass's mode loop that a wrong sign of b_y or a mishandled Nyquist
mode shows in first, at every length of the one-component form: the per-axis extended
invariants of the initial fields (the forward half), and the divergence norms before and
after a step and after a jump, for white noise, where none of them is zero.

Gates as in the extended invariants' and the (y, z) plane pass's tests: 1e-12 (FP64) and 1e-5
(FP32) of each sum's own size; the divergence norms 1e-11 and 1e-5 of theirs.
"""
import math

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2210_06232_amd import inputs
from tests.test_gpu_invariants_ext import compare

pytestmark = pytest.mark.gpu

DOMAIN = (0.0, 2 * math.pi, -1.0, 4 * math.pi - 1.0, 0.5, 2.5)
# (nx, ny, nz): every length of the form (8 to 256), beside the (x, z) plane pass and the
# separate passes (Nx = 12, Nz = 6), columns that do not fill a tile; two whole tiles at 256;
# and a length of each other form (384, 512)
SHAPES = [(24, 8, 32), (24, 12, 16), (24, 16, 16), (24, 24, 8), (24, 32, 8), (48, 48, 8), (12, 64, 8), (12, 96, 6),
          (24, 128, 8), (12, 192, 6), (16, 256, 8), (8, 384, 4), (8, 512, 4)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_per_axis_sums_and_divergence_norms_match_oracle(shape, prec):
    from paper_2210_06232_amd import eifp as m
    H, E = (f.astype(np.float32).astype(np.float64) for f in inputs.white_noise_fields(shape, seed=300 + sum(shape)))
    mu, eps, tau = 1.3, 0.8, 0.17
    want = orc.invariants(H, E, DOMAIN, mu, eps)
    Ho, Eo, _ = orc.step(H, E, DOMAIN, mu, eps, tau, 1)
    after = orc.invariants(Ho, Eo, DOMAIN, mu, eps)
    got = []
    with m.Solver(H, E, DOMAIN, mu, eps, prec) as s:
        ext, first = s.invariants_ext(), s.invariants()
        s.step(tau, 1)
        got.append(s.invariants())
    with m.Solver(H, E, DOMAIN, mu, eps, prec) as s:
        s.jump(tau, 1)
        got.append(s.invariants())
    tol = 1e-12 if prec == "fp64" else 1e-5
    compare(ext, want, tol)
    tol = 1e-11 if prec == "fp64" else 1e-5
    for g, w in ((first, want), (got[0], after), (got[1], after)):
        assert abs(g["div_h_l2"] - w["divH_l2"]) <= tol * w["divH_l2"]
        assert abs(g["div_e_l2"] - w["divE_l2"]) <= tol * w["divE_l2"]
