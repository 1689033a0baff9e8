"""FP64 hub_cg_solve from several threads: the launches of solves that stay on the
chip follow each other, and nobody waits longer than for those before it."""
import threading

import numpy as np
import pytest

from paper_1007_3432_amd import hub, inputs
from tests import hubtest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hubtest.ensure_built()


class Problem:
    def __init__(self, shape, max_iter, tol=1e-10):
        import torch
        self.lat = hub.lattice(*shape)
        sigma, phi = inputs.sigma_eta(*shape, seed=12)
        self.sigma, self.phi = hubtest.to_dev(sigma), hubtest.to_dev(phi)
        self.x = hubtest.empty(self.lat.volume, hub.F64)
        self.opts = hub.cg_opts(hub.F64, tol=tol, max_iter=max_iter)
        self.stream = torch.cuda.Stream()

    def solve(self):
        import torch
        with torch.cuda.stream(self.stream):
            return hub.hub_cg_solve(self.lat, self.sigma, self.phi, self.x, self.opts,
                                    raise_on_noconv=False)


def test_short_solve_beside_a_long_one():
    """A thread that solves without a pause, eight or more launches a solve:
    another thread's solves of one launch each wait for one or two of those
    launches, not for the solve they belong to."""
    import torch
    hubtest.log_case("cg threads: short beside long")
    long, short = Problem((1, 4096, 128), 200000), Problem((3, 5, 20), 300)
    assert long.solve()["iters"] > 8000
    alone = short.solve()
    x = short.x.cpu().numpy()
    torch.cuda.synchronize()
    count, stop = [0], threading.Event()

    def work():
        while not stop.is_set():
            long.solve()
            count[0] += 1

    t = threading.Thread(target=work)
    t.start()
    try:
        while count[0] == 0:
            stop.wait(0.01)
        before = count[0]
        for _ in range(8):
            st = short.solve()
        meanwhile = count[0] - before
    finally:
        stop.set()
        t.join()
    assert st["iters"] == alone["iters"] and np.array_equal(x, short.x.cpu().numpy())
    assert meanwhile <= 4, f"{meanwhile} long solves ended during 8 short ones"


def test_solve_beside_a_busy_stream():
    """A thread whose stream has long work queued before its solve keeps no other
    thread's solve waiting for that work."""
    import torch
    hubtest.log_case("cg threads: busy stream")
    late, other = Problem((3, 8, 80), 500), Problem((3, 8, 80), 500)
    late.solve(), other.solve()
    load = torch.ones(1 << 27, device="cuda:0")
    torch.cuda.synchronize()
    queued = threading.Event()
    ready = torch.cuda.Event()

    def work():
        with torch.cuda.stream(late.stream):
            for _ in range(2000):  # about 0.3 s
                load.mul_(1.0)
            ready.record()
        queued.set()
        late.solve()

    t = threading.Thread(target=work)
    t.start()
    try:
        queued.wait()
        threading.Event().wait(0.02)  # the other thread is in its solve
        other.solve()
        pending = not ready.query()
    finally:
        t.join()
    assert pending, "the solve ended only after the other stream's work"
    assert np.array_equal(late.x.cpu().numpy(), other.x.cpu().numpy())


def test_products_beside_a_solve():
    """A kernel of another stream that finds no room beside a resident solve waits
    for a launch of 300 iterations, 1.8 ms on this lattice (1000 iterations: 5.9)."""
    import time

    import torch
    hubtest.log_case("cg threads: products beside a solve")
    solve = Problem((3, 16, 128), 3000, tol=1e-14)
    lat = hub.lattice(3, 16, 32)
    x = torch.randn(lat.volume, dtype=torch.float64, device="cuda:0")
    links, z = torch.empty_like(x), torch.empty_like(x)
    hub.hub_links_from_sigma(lat, x, links, hub.F64)
    solve.solve()
    torch.cuda.synchronize()
    ended = threading.Event()

    def work():
        for _ in range(6):
            solve.solve()
        ended.set()

    waits = []
    stream = torch.cuda.Stream()
    t = threading.Thread(target=work)
    t.start()
    try:
        with torch.cuda.stream(stream):
            while not ended.is_set():
                t0 = time.perf_counter()
                hub.hub_apply_MtM(lat, links, hub.F64, hub.F64, x, z)
                stream.synchronize()
                waits.append(time.perf_counter() - t0)
    finally:
        t.join()
    held = sorted(w for w in waits if w > 4e-4)
    assert not held or held[len(held) // 2] <= 3.6e-3, f"{held[len(held) // 2] * 1e3:.1f} ms"
