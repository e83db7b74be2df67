"""Calls on a stream that is capturing a graph: a change of tau, of a jump's time span or
a first anchor is refused and leaves no trace; a step with the tau already set, and the
allocation-free step, are recorded and give the eager calls' bits at every replay, with
eager work between the replays.
"""
import math

import numpy as np
import pytest

from paper_2210_06232_amd import inputs

pytestmark = pytest.mark.gpu

DOMAIN = (0.0, 2 * math.pi, -1.0, 4 * math.pi - 1.0, 0.5, 2.5)
T1, T2 = 0.125, 0.25  # exact in binary, so sums of them are too


def eifp():
    from paper_2210_06232_amd import eifp as m
    m.load()
    return m


def same(a, b):
    for x, y in zip(a.fields(), b.fields()):
        np.testing.assert_array_equal(x, y)
    ia, ib = a.invariants(), b.invariants()
    assert ia["energy"] == ib["energy"] and ia["helicity"] == ib["helicity"]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_a_capturing_stream_refuses_descriptor_changes(prec):
    import torch
    m = eifp()
    H, E = inputs.random_fields((24, 16, 32), DOMAIN, workload=41, p=2.0)
    stream = torch.cuda.Stream()
    with m.Solver(H, E, DOMAIN, 1.1, 0.9, prec, stream.cuda_stream) as s, \
            m.Solver(H, E, DOMAIN, 1.1, 0.9, prec) as r:
        s.step(T1, 2)
        s.sync()
        before = s.device_bytes()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream, capture_error_mode="relaxed"):
            s.step(T1, 1)
            for call in (lambda: s.step(T2, 1), lambda: s.jump(T1, 1), s.anchor):
                with pytest.raises(m.EifpError) as ei:
                    call()
                assert ei.value.status == m.EIFP_ERR_DEVICE
        assert s.device_bytes() == before
        s.step(T2, 1)  # not recorded, and not taken for written: the eager step writes it
        r.step(T1, 2).step(T2, 1)
        same(s, r)
        for n in (1, 3):
            s.step(T1, n)
            with torch.cuda.stream(stream):
                g.replay()
            s.sync()
            r.step(T1, n).step(T1, 1)
            same(s, r)
        # a jump from here: the anchor the capture refused is made now
        s.jump(T1, 3)
        r.jump(T1, 3)
        same(s, r)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(128, 6, 96), (16, 12, 8), (8, 24, 24), (256, 24, 64)],
                         ids=lambda s: "x".join(map(str, s)))
def test_noalloc_steps_replay_the_eager_bits(shape, prec):
    # (x, z) planes several to a workgroup and one each, the (y, z) plane, and (FP32) the
    # separate passes
    import torch
    m = eifp()
    word = torch.float64 if prec == "fp64" else torch.float32
    H, E = inputs.random_fields(shape, DOMAIN, workload=42, p=2.0)
    start = torch.from_numpy(np.concatenate([H, E])).to("cuda", word).contiguous()
    a, b = start.clone(), start.clone()
    ia, ib = (torch.zeros(8, device="cuda", dtype=torch.float64) for _ in range(2))
    stream = torch.cuda.Stream()

    def step(f, inv, st):
        m.eifp_step_noalloc(f.data_ptr(), shape, DOMAIN, 1.1, 0.9, prec, T1, 3, inv.data_ptr(), st.cuda_stream)

    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        step(a, ia, stream)
    for _ in range(3):
        with torch.cuda.stream(stream):
            g.replay()
        torch.cuda.synchronize()
        step(b, ib, torch.cuda.current_stream())  # eager work between the replays
        torch.cuda.synchronize()
        assert torch.equal(a, b)
        assert torch.equal(ia[:7], ib[:7])
