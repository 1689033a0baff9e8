"""FP64 hub_cg_solve at the edges of its kernels: one, two and four sites per
lane of one workgroup, full and with a remainder, in each number of dimensions,
and the resident solver's cuts.  Checked as in test_gpu_cg.py: the oracle's true residual, the
distance to the oracle's solution (two solutions with residual <= tol differ
by at most 2 cond(Q) tol; twice that for the Lanczos estimate of cond(Q)), and
the iteration count."""
import threading

import numpy as np
import pytest

import oracle
from paper_1007_3432_amd import hub, inputs
from tests import dense, hubtest

pytestmark = pytest.mark.gpu

TOL = 1e-10


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hubtest.ensure_built()
    oracle.set_threads(16)


def check(shape, cheb=None):
    olat, lat = oracle.Lattice(*shape), hub.lattice(*shape)
    hubtest.log_case(f"cg sizes {shape}")
    sigma, eta = inputs.sigma_eta(*shape, seed=11)
    A = oracle.links(olat, sigma)
    phi = oracle.apply_Mt(olat, A, eta)
    x_o, res, (al, be) = oracle.cg(olat, A, phi, tol=TOL, record=True)
    assert res.converged
    x_d = hubtest.empty(lat.volume, hub.F64)
    args = (lat, hubtest.to_dev(sigma), hubtest.to_dev(phi), x_d, hub.cg_opts(hub.F64))
    st = hub.hub_pcg_solve(*args, cheb) if cheb else hub.hub_cg_solve(*args)
    x = x_d.cpu().numpy()
    assert st["status"] == "HUB_OK"
    r = np.linalg.norm(phi - oracle.apply_MtM(olat, A, x)) / np.linalg.norm(phi)
    assert r <= 1.1 * TOL
    assert hubtest.rel_err(x, x_o) <= 4 * dense.lanczos_condition(al, be) * TOL
    if cheb:
        res = oracle.pcg(olat, A, phi, cheb.n, cheb.eps, tol=TOL)[1]
        assert abs(st["iters"] - res.iters) <= max(2, 0.05 * res.iters)
    else:
        assert abs(st["iters"] - res.iters) <= 0.03 * res.iters + 3


@pytest.mark.parametrize("shape", [
    (1, 16, 32), (1, 27, 19), (1, 32, 32), (1, 205, 5), (1, 64, 32), (2, 8, 8), (2, 5, 21),
    (2, 2, 129), (2, 32, 2), (2, 18, 6), (3, 8, 2), (3, 2, 66), (3, 4, 32), (3, 3, 75)],
    ids=lambda s: "d%d_%dx%d" % s)
def test_one_workgroup(shape):
    assert shape[1] ** shape[0] * shape[2] <= 2048
    check(shape)


# The resident solver: z whole and cut, tiles of unequal size, one slice and
# several per block, inner planes that leave lanes idle, every level.
@pytest.mark.parametrize("shape", [
    (1, 37, 60), (1, 257, 33), (1, 5000, 7), (1, 3, 900), (1, 2048, 200), (2, 33, 20), (2, 5, 100),
    (2, 512, 2), (2, 300, 3), (2, 47, 47), (3, 5, 20), (3, 9, 17), (3, 2, 300), (3, 16, 12),
    (3, 20, 6), (3, 22, 3), (3, 12, 50)],
    ids=lambda s: "d%d_%dx%d" % s)
def test_resident(shape):
    assert shape[1] ** shape[0] * shape[2] > 2048
    check(shape)


# One factor and several; lattices below what plain CG keeps in one workgroup.
@pytest.mark.parametrize("n", [1, 4])
@pytest.mark.parametrize("shape", [
    (1, 2, 2), (1, 16, 9), (1, 300, 37), (1, 700, 90), (2, 3, 4), (2, 21, 40), (2, 47, 11), (3, 2, 2),
    (3, 6, 21), (3, 9, 17), (3, 16, 12), (3, 20, 3)], ids=lambda s: "d%d_%dx%d" % s)
def test_resident_preconditioned(shape, n):
    check(shape, hub.cheb_opts(n, 0.01))


def test_resident_wait_given_up(monkeypatch):
    """With a single read allowed, blocks give up the first wait for each
    other: the solve ends and is done by the multi-kernel solver."""
    monkeypatch.setenv("HUB_CG_RESIDENT_READS", "1")
    check((1, 256, 32))
    check((1, 256, 32), hub.cheb_opts(3, 0.01))


def test_resident_threads():
    """Two threads that solve at the same time get what each gets alone."""
    import torch
    probs, alone, both = [], [], [None, None]
    for shape in ((3, 8, 24), (1, 300, 40)):
        lat = hub.lattice(*shape)
        sigma, phi = inputs.sigma_eta(*shape, seed=12)
        probs.append((lat, hubtest.to_dev(sigma), hubtest.to_dev(phi)))

    def solve(k, stream):
        lat, sigma, phi = probs[k]
        x = hubtest.empty(lat.volume, hub.F64)
        with torch.cuda.stream(stream):
            for _ in range(3):
                hub.hub_cg_solve(lat, sigma, phi, x, hub.cg_opts(hub.F64))
        return x.cpu().numpy()

    streams = [torch.cuda.Stream() for _ in probs]
    alone = [solve(k, streams[k]) for k in range(2)]
    torch.cuda.synchronize()
    threads = [threading.Thread(target=lambda k=k: both.__setitem__(k, solve(k, streams[k]))) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for a, b in zip(alone, both):
        assert b is not None and np.array_equal(a, b)
