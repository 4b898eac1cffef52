"""GPU: a server with small grids that run on chip beside grids of the batch.

* Neither kind waits for the other's streaming budget: with one batched solve
  filling it, on-chip requests behind a second, waiting one are all done before
  that one is admitted.
* Every result is bitwise the single solve's, with other on-chip solves of the
  device on another thread meanwhile, whose results are too.
"""
import threading

import numpy as np
import pytest

from paper_1709_01126_amd import pot3d as P

from test_gpu_parity import GRIDS
from test_gpu_serving import alone, requests

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SMALL = GRIDS[4]                                            # 2.5 MB of FP64 vectors, on chip
FLAT = (2, 300, 600, "stretched", "uniform", "uniform")     # 11.5 MB, more columns than an on-chip launch takes


@pytest.mark.parametrize("precision", [P.FP64, P.FP32_REFINED], ids=["fp64", "fp32_refined"])
def test_small_requests_run_beside_a_batched_one(precision):
    reqs = requests([FLAT, SMALL, FLAT] + [SMALL] * 5, tol=1e-9)
    ref = alone(reqs, precision)
    with P.Server(precision=precision, max_slots=8) as sv:
        sv.set_cache_budget(12e6 if precision == P.FP64 else 6e6)
        ids = [sv.submit(rf, tf, pf, br, tol, maxit) for _, rf, tf, pf, br, tol, maxit in reqs]
        for _ in range(100_000):
            if sv.step()[2] == len(ids):
                break
        out = [sv.take(rid) for rid in ids]
    t_admit = [o[1]["t_admit"] for o in out]
    t_done = [o[1]["t_done"] for o in out]
    assert t_admit[2] >= t_done[0]                    # one batched solve at a time
    assert max(t_done[q] for q in (1, 3, 4, 5, 6, 7)) < t_admit[2]
    for (phi_a, st_a, it_a, _), (phi_s, info) in zip(ref, out):
        assert info["status"] == st_a == P.OK and info["iters"] == it_a and np.array_equal(phi_s, phi_a)


def test_server_and_single_solves_on_two_threads():
    reqs = requests([FLAT, SMALL, SMALL, SMALL], tol=1e-9)
    ref = alone(reqs, P.FP64)
    _, rf, tf, pf, br, tol, maxit = reqs[1]
    got, stop = [], threading.Event()

    def singles():
        with P.Solver(rf, tf, pf) as s:
            while not stop.is_set():
                got.append(s.solve(br, tol, maxit))

    th = threading.Thread(target=singles)
    with P.Server(max_slots=8) as sv:
        ids = [sv.submit(f0, f1, f2, b, t, m) for _, f0, f1, f2, b, t, m in reqs]
        th.start()
        try:
            for _ in range(100_000):
                if sv.step()[2] == len(ids) and len(got) >= 2:
                    break
        finally:
            stop.set()
            th.join()
        out = [sv.take(rid) for rid in ids]
    for (phi_a, st_a, it_a, _), (phi_s, info) in zip(ref, out):
        assert info["status"] == st_a == P.OK and info["iters"] == it_a and np.array_equal(phi_s, phi_a)
    for phi, st, it, _ in got:
        assert st == P.OK and it == ref[1][2] and np.array_equal(phi, ref[1][0])
