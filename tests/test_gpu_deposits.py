"""Mixed CG where a sweep takes over the sums of the phase B before it: at the
edges of the deposit counts (2048 sites each) that choose how, with solves that
end inside a chunk of iterations, at its end, and by max_iter.

The persistent serving engine adds every deposit in a pass of its own, in the
same order, so alone, batched and persistent must agree bit for bit."""
import pytest

from paper_1007_3432_amd import hub, inputs
from tests import hubtest
from tests.test_gpu_serve import _wait_all
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hubtest.ensure_built()
    oracle.set_threads(16)


# 1, 15.6, 256, 256.5, 512 and 512.5 deposits in d = 1; 256 and 272 with the
# nx = 32 tile, 513 with the nx = 16 tile.
@pytest.mark.parametrize("shape", [(1, 32, 64), (1, 250, 128), (1, 1024, 512), (1, 1024, 513),
                                   (1, 1024, 1024), (1, 1024, 1025), (3, 32, 16), (3, 32, 17),
                                   (3, 16, 257)], ids=str)
@pytest.mark.parametrize("link", [hub.F32, hub.F16], ids=["f32", "f16"])
def test_engines_agree(shape, link):
    hubtest.log_case(f"deposits {shape} link={link}")
    lat = hub.lattice(*shape)
    olat = oracle.Lattice(*shape)
    sigma, eta = inputs.sigma_eta(*shape, seed=5)
    phi = oracle.apply_Mt(olat, oracle.links(olat, sigma), eta)
    for tol, max_iter in ((1e-2, 1000), (1e-12, 5), (1e-12, 13)):
        opts = hub.cg_opts(hub.F32, link, tol=tol, max_iter=max_iter, reliable_every=5)
        x_d = hubtest.empty(lat.volume, hub.F64)
        st = hub.hub_cg_solve(lat, hubtest.to_dev(sigma), hubtest.to_dev(phi), x_d, opts,
                              raise_on_noconv=False)
        x = x_d.cpu().numpy()
        assert (st["status"] == "HUB_OK") == (tol > 1e-6)
        for engine in (0, 1):
            srv = hub.Server(hbm_budget_bytes=8 << 30, max_inflight=4, cg=opts, engine=engine)
            try:
                # the same solve twice, so that solves share a launch
                ts = [srv.submit(c, lat, sigma, phi) for c in (0, 1)]
                for xs, ss in _wait_all(srv, ts, {t: lat.volume for t in ts}).values():
                    assert (xs == x).all()
                    assert all(ss[k] == st[k] for k in ("iters", "reliable_updates", "status",
                                                        "true_rel_resid"))
            finally:
                srv.close()
