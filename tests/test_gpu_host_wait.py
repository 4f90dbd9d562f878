"""A solve waits for the device on the calling thread: a long wait leaves the core to others."""
import time

import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def test_long_waits_sleep():
    from paper_2306_03574_amd.abac import Plan, fill_normal
    print("[case] host wait 511x511x1024 fp32", flush=True)
    p = Plan(511, 511, 1024, alpha=1e-3, prec="fp32", device=DEV)
    f = fill_normal(p.empty(), 3)
    u = p.empty()
    p.solve(f, u)
    wall, cpu = time.perf_counter(), time.thread_time()
    _, iters, _, status = p.solve(f, u)
    wall, cpu = time.perf_counter() - wall, time.thread_time() - cpu
    print(f"{iters[0]} iterations, {wall * 1e3:.1f} ms, {cpu * 1e3:.1f} ms on the core")
    assert status == [0]
    # an iteration takes over 4 ms; 1 ms of it the thread looks, then it sleeps most of the time
    assert wall / iters[0] > 3e-3
    assert cpu < 0.6 * wall
