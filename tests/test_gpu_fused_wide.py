"""The fused y pass with one component per wave (few tiles, or FP64 at lengths 64 to 256),
beside the other forms.

Gates, as for every pass: one step against one oracle step (Def. 2.3 / Alg. 2) at 1e-12
(FP64) and 2e-6 (FP32, from FP32-rounded input), in the energy norm and element by
element, and the invariants of the new state; the same for a jump (the form's inverse
half alone), and the extended invariants of the initial fields (its forward half).
"""
import math

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2210_06232_amd import inputs
from tests.helpers import elementwise_rel_error, energy_rel_error

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 2e-6}
DOMAIN = (0.0, 2 * math.pi, -1.0, 4 * math.pi - 1.0, 0.5, 2.5)
# (nx, ny, nz): every pencil length of the form; columns that do not fill a tile (M = 2, 3,
# 12, 24 against tiles of 4 to 64); one tile only; several tiles a workgroup (FP64 128,
# 192 and 256 with more tiles than CUs); tile counts on both sides of the limits (32 x 32 x 512
# has 512 tiles, 256 x 32 x 96 768; in FP32 96^3 has 576 and 128 x 96 x 96 768)
SHAPES = [(48, 8, 128), (6, 12, 96), (96, 16, 64), (24, 24, 48), (32, 32, 512), (256, 32, 96), (4, 48, 64),
          (64, 64, 32), (96, 96, 96), (128, 96, 96), (128, 128, 48), (48, 192, 48), (96, 192, 96), (24, 256, 16),
          (48, 256, 64), (16, 512, 8)]


def eifp():
    from paper_2210_06232_amd import eifp as m
    m.load()
    return m


def rounded32(F):
    return np.ascontiguousarray(np.asarray(F, dtype=np.float32).astype(np.float64))


def check_fields(Hg, Eg, Ho, Eo, mu, eps, prec, what):
    en = energy_rel_error(Hg, Eg, Ho, Eo, mu, eps)
    el = elementwise_rel_error(Hg, Eg, Ho, Eo, mu, eps)
    print(f"{what} {prec}: energy-norm {en:.3e}, element-wise {el:.3e}", flush=True)
    assert en <= TOL[prec] and el <= TOL[prec]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_wide_fused_step_and_jump_match_oracle(shape, prec):
    m = eifp()
    H, E = inputs.white_noise_fields(shape, seed=900 + sum(shape))  # full spectrum, Nyquist included
    H, E = rounded32(H), rounded32(E)
    mu, eps, tau = 1.3, 0.8, 0.17
    Ho, Eo, _ = orc.step(H, E, DOMAIN, mu, eps, tau, 1)
    want = orc.invariants(Ho, Eo, DOMAIN, mu, eps)
    tol = 1e-12 if prec == "fp64" else 1e-6
    e_ref = math.sqrt(want["E1"] * want["E2"])
    with m.Solver(H, E, DOMAIN, mu, eps, prec) as s:
        ext = s.invariants_ext()
        s.step(tau, 1)
        check_fields(*s.fields(), Ho, Eo, mu, eps, prec, f"{shape} step")
        got = [s.invariants()]
    with m.Solver(H, E, DOMAIN, mu, eps, prec) as s:
        s.jump(tau, 1)
        check_fields(*s.fields(), Ho, Eo, mu, eps, prec, f"{shape} jump")
        got.append(s.invariants())
    for g in got:
        assert abs(g["energy"] - want["E1"]) <= tol * want["E1"]
        assert abs(g["helicity"] - want["H1"]) <= tol * e_ref
        for k, c in enumerate("xyz"):
            assert abs(g["momentum"][k] - want[f"M1_{c}"]) <= tol * e_ref
    # E2 and E3 are conserved, so those of the initial fields are those of the new state
    assert abs(ext["E2"] - want["E2"]) <= 10 * tol * want["E2"]
