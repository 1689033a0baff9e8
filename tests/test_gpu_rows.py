"""The row tiles of the fused sweep (d = 2, and d = 3 with nx not a tile's):
hub_apply_MtM in every precision, and a mixed and a preconditioned solve whose
sweeps run on them, against the oracle.  Shapes: whole slices and cut ones,
tiles of unequal height, one-row tiles, a last chunk of one slice, each level,
and rows too long for a tile (two passes).  Tolerances as in
test_gpu_apply.py and test_gpu_cg.py."""
import numpy as np
import pytest

import oracle
from paper_1007_3432_amd import hub, inputs
from tests import dense, hubtest

pytestmark = pytest.mark.gpu

SHAPES = [(2, 2, 2), (2, 3, 9), (2, 7, 3), (2, 22, 5), (2, 23, 4), (2, 33, 35), (2, 64, 200), (2, 130, 3),
          (2, 300, 4), (2, 511, 3), (2, 600, 2), (2, 1100, 2), (3, 2, 2), (3, 2, 40), (3, 3, 5), (3, 9, 5),
          (3, 10, 37), (3, 21, 7), (3, 31, 3), (3, 48, 2), (3, 90, 2)]


@pytest.fixture(scope="module", autouse=True)
def _lib():
    hubtest.ensure_built()
    oracle.set_threads(16)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "d%d_%dx%d" % s)
def test_mtm_rows(shape):
    import torch
    olat = oracle.Lattice(*shape, mu=0.07)
    lat = hub.lattice(*shape, olat.t_hop, olat.dtau, olat.U, olat.mu)
    hubtest.log_case(f"mtm rows {shape}")
    V = lat.volume
    sigma, _ = inputs.sigma_eta(*shape, seed=21)
    x = inputs.random_vector(V, 22)
    A = oracle.links(olat, sigma)
    s16 = np.sin(np.roll(sigma.reshape(shape[2], -1), 1, axis=0)).astype(np.float16).astype(np.float64)
    A16 = np.exp(olat.dtau * olat.mu) * (1 + oracle.hs_coupling(olat.dtau, olat.U) * s16)
    A16[1:] *= -1
    for vec, link, ref, tol in ((hub.F64, hub.F64, A, 1e-13), (hub.F32, hub.F32, A, 2e-6),
                                (hub.F32, hub.F16, A16.reshape(-1), 2e-6)):
        links = hubtest.empty(V, link)
        hub.hub_links_from_sigma(lat, hubtest.to_dev(sigma), links, link)
        xv = hubtest.to_dev(x, hub._torch_dtype(vec))
        z = torch.full((V + 256,), float("nan"), dtype=xv.dtype, device=xv.device)
        hub.hub_apply_MtM(lat, links, link, vec, xv, z[:V])
        want = oracle.apply_MtM(olat, ref, xv.double().cpu().numpy())
        assert hubtest.rel_err(z[:V].double().cpu().numpy(), want) <= tol
        assert bool(torch.isnan(z[V:]).all())  # nothing written past the end


@pytest.mark.parametrize("shape", [(2, 33, 20), (3, 11, 6)], ids=lambda s: "d%d_%dx%d" % s)
@pytest.mark.parametrize("how", ["f32", "f16", "pcg"])
def test_solve_rows(shape, how):
    olat, lat = oracle.Lattice(*shape), hub.lattice(*shape)
    hubtest.log_case(f"solve rows {shape} {how}")
    sigma, eta = inputs.sigma_eta(*shape, seed=23)
    A = oracle.links(olat, sigma)
    phi = oracle.apply_Mt(olat, A, eta)
    x_o, res, (al, be) = oracle.cg(olat, A, phi, tol=1e-10, record=True)
    x_d = hubtest.empty(lat.volume, hub.F64)
    args = (lat, hubtest.to_dev(sigma), hubtest.to_dev(phi), x_d)
    if how == "pcg":
        hub.hub_pcg_solve(*args, hub.cg_opts(hub.F64), hub.cheb_opts(6, 0.003))
    else:
        hub.hub_cg_solve(*args, hub.cg_opts(hub.F32, hub.F32 if how == "f32" else hub.F16))
    x = x_d.cpu().numpy()
    r = np.linalg.norm(phi - oracle.apply_MtM(olat, A, x)) / np.linalg.norm(phi)
    assert r <= 1.1e-10
    assert hubtest.rel_err(x, x_o) <= 4 * dense.lanczos_condition(al, be) * 1e-10


def test_current_stream():
    """Calls without a stream go to the stream that is current in torch."""
    import torch
    assert hub._stream(None) == torch.cuda.current_stream().cuda_stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert hub._stream(None) == s.cuda_stream
        assert hub._stream(None) == hub._current_stream_slow()
    assert hub._stream(s) == s.cuda_stream and hub._stream(7) == 7


# The unrolled march of the d = 3 tiles (nx = 32, 64): a last chunk that starts
# early and repeats slices, and the fewest slices that take it.
@pytest.mark.parametrize("shape", [(3, 32, 125), (3, 32, 131), (3, 64, 17)], ids=lambda s: "d%d_%dx%d" % s)
def test_mtm_unrolled(shape):
    test_mtm_rows(shape)


@pytest.mark.parametrize("nt", [2, 23, 24, 31, 243])
def test_nx32_tile_by_slices(nt):
    """nx = 32 on either side of the number of slices that chooses its tile,
    and where the larger tile's march is unrolled."""
    test_mtm_rows((3, 32, nt))
