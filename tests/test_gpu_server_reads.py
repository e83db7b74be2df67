"""Field reads of a running server from several threads: results of different requests are
copied side by side (a short read does not wait for a long one), while a third request
steps on, and every copy holds its own request's fields.
"""
import math
import statistics
import threading
import time

import numpy as np
import pytest

from paper_2210_06232_amd import inputs

pytestmark = pytest.mark.gpu

DOMAIN = (0.0, 2 * math.pi, 0.0, 2 * math.pi, 0.0, 3 * math.pi)
LARGE, SMALL, OTHER = (192, 192, 192), (64, 64, 96), (32, 32, 32)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_reads_of_two_results_do_not_wait_for_each_other(prec):
    from paper_2210_06232_amd import eifp as m
    rng = np.random.default_rng(8)
    fields = {s: [rng.standard_normal((3, s[2], s[1], s[0])).astype(np.float32).astype(np.float64) for _ in range(2)]
              for s in (LARGE, SMALL)}
    want = {}
    for s, (H, E) in fields.items():
        with m.Solver(H, E, DOMAIN, 1.0, 1.5, prec) as solver:
            solver.step(0.1, 2)
            want[s] = solver.fields()
    took = {LARGE: [], SMALL: []}
    wrong = []
    with m.Server(8 * 10 ** 9, 4) as sv:
        ids = {s: sv.submit(H, E, DOMAIN, 1.0, 1.5, 0.1, 2, 0, prec, 0, m.EIFP_REQ_KEEP_RESULT)
               for s, (H, E) in fields.items()}
        sv.drain(60000)
        H, E = inputs.random_fields(OTHER, DOMAIN, workload=3, p=2.0)
        going = sv.submit(H, E, DOMAIN, 1.0, 1.5, 0.1, 10 ** 9, 100, prec, 1, 0)  # steps until cancelled

        def read(s):
            t0 = time.perf_counter()
            Hs, Es, step = sv.fields(ids[s], s)
            took[s].append(time.perf_counter() - t0)
            return Hs, Es, step

        def check(s, got):
            if got[2] != 2 or not all(np.array_equal(a, b) for a, b in zip(got, want[s])):
                wrong.append(s)

        reading = threading.Event()

        def read_large():
            reading.set()
            for _ in range(20):  # back to back
                got = read(LARGE)
            reading.clear()
            check(LARGE, got)

        check(SMALL, read(SMALL))
        took[SMALL].clear()
        th = threading.Thread(target=read_large)
        th.start()
        assert reading.wait(10)
        while reading.is_set():
            check(SMALL, read(SMALL))
        th.join()
        before = sv.stats()["chunks"]
        t0 = time.time()
        while sv.stats()["chunks"] == before and time.time() - t0 < 10:
            time.sleep(0.01)
        assert sv.stats()["chunks"] > before  # the third request goes on
        sv.cancel(going)
        sv.drain(60000)
    small, large = (1e3 * statistics.median(took[s]) for s in (SMALL, LARGE))
    print(f"{prec}: median read {small:.2f} ms of 9 MB x 2, {large:.2f} ms of {len(took[LARGE])} reads of 170 MB x 2")
    assert not wrong
    # one after the other, a short read takes at least the long one's copy of an array
    assert small < 0.5 * large
