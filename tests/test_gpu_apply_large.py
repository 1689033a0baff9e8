"""FP64 M, M^T and force on lattices whose two inputs exceed the Infinity Cache
(just over 2^24 sites), where the input read once at each site is loaded past the
caches: against the oracle, with the tolerance of the smaller lattices (1e-13 of
the norm: a dozen operations a site)."""
import pytest

import oracle
from paper_1007_3432_amd import hub, inputs
from tests import hubtest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hubtest.ensure_built()
    oracle.set_threads(16)


@pytest.mark.parametrize("shape", [(1, 4098, 4096), (2, 410, 100), (3, 64, 65)],
                         ids=lambda s: "d%d_%dx%d" % s)
def test_inputs_larger_than_the_cache(shape):
    olat, lat = oracle.Lattice(*shape), hub.lattice(*shape)
    assert 16 * lat.volume > 256 << 20
    hubtest.log_case(f"apply large {shape}")
    sigma, x = inputs.sigma_eta(*shape, seed=17)
    A = oracle.links(olat, sigma)
    sigma_d, x_d, A_d = hubtest.to_dev(sigma), hubtest.to_dev(x), hubtest.to_dev(A)
    y_d = hubtest.empty(lat.volume, hub.F64)
    for transpose, ref in ((0, oracle.apply_M), (1, oracle.apply_Mt)):
        hub.hub_apply_M(lat, A_d, hub.F64, hub.F64, x_d, y_d, transpose)
        assert hubtest.rel_err(y_d.cpu().numpy(), ref(olat, A, x)) <= 1e-13
    hub.hub_hmc_force(lat, sigma_d, x_d, y_d)
    assert hubtest.rel_err(y_d.cpu().numpy(), oracle.force(olat, sigma, x)) <= 1e-13
