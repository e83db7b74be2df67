"""The (x, z) plane pass: grids whose (x, z) plane of one component fits in LDS run the z
inverse, x inverse, next x forward and next z forward between two fused passes as one
kernel, and the first and last of them in pairs.

Gates, as for the separate passes: two steps (one plane pass of each kind) against two
oracle steps (Def. 2.3 / Alg. 2) at 1e-12 (FP64) and 2e-6 (FP32, from FP32-rounded
input), in the energy norm and element by element, with the invariants of the new state;
and the same bits from one call of n steps, n calls of one step, and the steps applied in
place to a caller's buffer.
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
# (nx, ny, nz): the smallest plane; columns and rows that do not fill a wave's group
# (M = 12 and 24 against 16 or 32 columns a wave, Nz = 8 and 12 against 64 or 32 rows); the
# longest columns and rows beside short ones; the largest planes, one workgroup a CU, with
# fewer planes than CUs and with more (several planes a workgroup, FP64); planes of FP32
# at the two-workgroups-a-CU limit and just beyond it (separate passes)
XZ_SHAPES = [(16, 96, 8), (24, 64, 12), (48, 32, 32), (48, 96, 8), (16, 4, 512), (512, 6, 16), (192, 8, 96),
             (128, 32, 128), (128, 48, 128), (96, 48, 192), (192, 16, 64), (128, 8, 192),
             # the smallest grid of the pass, and its neighbours that take the (y, z) plane
             (16, 4, 8), (12, 4, 8), (16, 4, 6), (256, 8, 6)]


def eifp():
    from paper_2210_06232_amd import eifp as m
    m.load()
    return m


def rounded32(F):
    return np.ascontiguousarray(np.asarray(F, dtype=np.float32).astype(np.float64))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", XZ_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_xz_plane_steps_match_oracle(shape, prec):
    m = eifp()
    H, E = inputs.white_noise_fields(shape, seed=700 + sum(shape))  # full spectrum, Nyquist included
    H, E = rounded32(H), rounded32(E)
    mu, eps, tau = 1.3, 0.8, 0.17
    Ho, Eo, _ = orc.step(H, E, DOMAIN, mu, eps, tau, 2)
    with m.Solver(H, E, DOMAIN, mu, eps, prec) as s:
        s.step(tau, 2)
        Hg, Eg = s.fields()
        got = s.invariants()
    en = energy_rel_error(Hg, Eg, Ho, Eo, mu, eps)
    el = elementwise_rel_error(Hg, Eg, Ho, Eo, mu, eps)
    print(f"{shape} {prec}: energy-norm {en:.3e}, element-wise {el:.3e}", flush=True)
    assert en <= TOL[prec] and el <= TOL[prec]
    want = orc.invariants(Ho, Eo, DOMAIN, mu, eps)
    tol = 1e-12 if prec == "fp64" else 1e-6
    e_ref = math.sqrt(want["E1"] * want["E2"])
    assert abs(got["energy"] - want["E1"]) <= tol * want["E1"]
    assert abs(got["helicity"] - want["H1"]) <= tol * e_ref
    for k, c in enumerate("xyz"):
        assert abs(got["momentum"][k] - want[f"M1_{c}"]) <= tol * e_ref


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(24, 64, 12), (64, 32, 48), (128, 48, 128)], ids=lambda s: "x".join(map(str, s)))
def test_xz_plane_call_patterns_give_the_same_bits(shape, prec):
    import torch
    m = eifp()
    H, E = inputs.random_fields(shape, DOMAIN, workload=9, p=2.0)
    out = []
    for calls in ((4,), (1,) * 4, (3, 1)):
        with m.Solver(H, E, DOMAIN, 1.1, 0.9, prec) as s:
            for n in calls:
                s.step(0.13, n)
            out.append((s.fields(), s.invariants()))
    for (Hg, Eg), inv in out[1:]:
        np.testing.assert_array_equal(Hg, out[0][0][0])
        np.testing.assert_array_equal(Eg, out[0][0][1])
        assert {k: v for k, v in inv.items() if k != "t"} == {k: v for k, v in out[0][1].items() if k != "t"}
    word = torch.float64 if prec == "fp64" else torch.float32
    f = torch.from_numpy(np.concatenate([H, E])).to("cuda", word).contiguous()
    inv = torch.zeros(8, device="cuda", dtype=torch.float64)
    m.eifp_step_noalloc(f.data_ptr(), shape, DOMAIN, 1.1, 0.9, prec, 0.13, 4, inv.data_ptr(),
                        torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = f.double().cpu().numpy()
    np.testing.assert_array_equal(got[:3], out[0][0][0])
    np.testing.assert_array_equal(got[3:], out[0][0][1])
    assert inv[0].item() == out[0][1]["energy"]
