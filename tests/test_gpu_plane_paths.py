"""The (y, z) plane pass on grids that take it (Nx below 16 or Nz below 8): one step against
the oracle, with the invariants its one-wave finalize writes; the same bits from one call of
n steps, n calls of one step and the steps applied in place; and the invariants a plane step
reports against those the separate forward passes compute for the same state.

Gates as in the plane pass's other tests: 1e-12 (FP64) and 2e-6 (FP32, from FP32-rounded
input) for the fields, 1e-12 and 1e-6 for the invariants; between the two evaluations of
one state's invariants 1e-13 (FP64) and 1e-6 (FP32), relative to the energy scale.
"""
import math

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2210_06232_amd import inputs
from tests.helpers import elementwise_rel_error, energy_rel_error

pytestmark = pytest.mark.gpu

DOMAIN = (0.0, 2 * math.pi, -1.0, 4 * math.pi - 1.0, 0.5, 2.5)
# (nx, ny, nz): every pencil length along y and z; from the smallest to the largest plane (576
# points); columns M = 2 to 256, the wide ones with more workgroups than the fused pass has
# partial records
SHAPES = [(4, 4, 4), (12, 8, 16), (8, 24, 24), (12, 16, 8), (6, 32, 16), (6, 16, 32), (32, 16, 6), (24, 24, 4),
          (64, 12, 6), (256, 8, 6), (512, 6, 4), (128, 32, 6)]


def eifp():
    from paper_2210_06232_amd import eifp as m
    m.load()
    return m


def rounded32(F):
    return np.ascontiguousarray(np.asarray(F, dtype=np.float32).astype(np.float64))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_step_matches_oracle(shape, prec):
    m = eifp()
    H, E = (rounded32(f) for f in inputs.white_noise_fields(shape, seed=600 + sum(shape)))
    mu, eps, tau = 1.3, 0.8, 0.17
    Ho, Eo, _ = orc.step(H, E, DOMAIN, mu, eps, tau, 1)
    with m.Solver(H, E, DOMAIN, mu, eps, prec) as s:
        s.step(tau, 1)
        Hg, Eg = s.fields()
        got = s.invariants()
    tol = 1e-12 if prec == "fp64" else 2e-6
    assert energy_rel_error(Hg, Eg, Ho, Eo, mu, eps) <= tol
    assert elementwise_rel_error(Hg, Eg, Ho, Eo, mu, eps) <= tol
    want = orc.invariants(Ho, Eo, DOMAIN, mu, eps)
    tol = 1e-12 if prec == "fp64" else 1e-6
    e_ref = math.sqrt(want["E1"] * want["E2"])
    assert abs(got["energy"] - want["E1"]) <= tol * want["E1"]
    assert abs(got["helicity"] - want["H1"]) <= tol * e_ref
    for k, c in enumerate("xyz"):
        assert abs(got["momentum"][k] - want[f"M1_{c}"]) <= tol * e_ref
    dscale = max(1.0, want["divH_l2"], want["divE_l2"])
    assert abs(got["div_h_l2"] - want["divH_l2"]) <= tol * dscale * 10
    assert abs(got["div_e_l2"] - want["divE_l2"]) <= tol * dscale * 10


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(8, 24, 24), (12, 16, 8), (32, 16, 6), (256, 8, 6)],
                         ids=lambda s: "x".join(map(str, s)))
def test_call_patterns_give_the_same_bits(shape, prec):
    import torch
    m = eifp()
    H, E = inputs.random_fields(shape, DOMAIN, workload=51, p=2.0)
    out = []
    for calls in ((6,), (1,) * 6, (4, 2)):
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
    m.eifp_step_noalloc(f.data_ptr(), shape, DOMAIN, 1.1, 0.9, prec, 0.13, 6, inv.data_ptr(),
                        torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = f.double().cpu().numpy()
    np.testing.assert_array_equal(got[:3], out[0][0][0])
    np.testing.assert_array_equal(got[3:], out[0][0][1])
    v, w = inv.cpu().numpy(), out[0][1]
    assert list(v[:7]) == [w["energy"], w["helicity"], *w["momentum"], w["div_h_l2"], w["div_e_l2"]]


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-13), ("fp32", 1e-6)])
@pytest.mark.parametrize("shape", [(8, 24, 24), (12, 16, 8), (32, 16, 6), (256, 8, 6)],
                         ids=lambda s: "x".join(map(str, s)))
def test_step_invariants_agree_with_the_separate_evaluation(shape, prec, tol):
    m = eifp()
    H, E = inputs.random_fields(shape, DOMAIN, workload=52, p=2.0)
    with m.Solver(H, E, DOMAIN, 1.0, 2.0, prec) as s:
        s.step(0.1, 3)
        inv_step = s.invariants()
        Hg, Eg = s.fields()
    with m.Solver(Hg, Eg, DOMAIN, 1.0, 2.0, prec) as s:
        inv_fresh = s.invariants()
    for k in ("energy", "helicity"):
        scale = max(abs(inv_fresh[k]), (1e-3 if prec == "fp64" else 1.0) * abs(inv_fresh["energy"]))
        assert abs(inv_step[k] - inv_fresh[k]) <= tol * scale, (k, inv_step[k], inv_fresh[k])
