"""Row tiles or two passes (csrc/sweep.h): on the CPU the choice on both sides of
each line, where it is the faster of the two as measured on MI355X; on the GPU the
products and factors there, against the oracle."""
import os
import subprocess

import numpy as np
import pytest

from paper_1007_3432_amd import build, hub, inputs
from tests import hubtest

HERE = os.path.dirname(os.path.abspath(__file__))
CHOICE = {
    (3, 63, 17, "b64"): "rows", (3, 67, 7, "b64"): "two", (3, 67, 17, "b64"): "two",
    (3, 72, 3, "b64"): "rows", (3, 72, 7, "b64"): "two", (3, 72, 17, "b32"): "two",
    (3, 76, 7, "b32"): "rows", (2, 260, 17, "b64"): "rows",
    (3, 22, 40, "s64"): "two", (3, 40, 7, "s64"): "two", (3, 40, 17, "s64"): "rows",
    (3, 72, 7, "s64"): "two", (3, 80, 3, "s64"): "two", (2, 260, 17, "s64"): "two",
    (2, 256, 17, "s64"): "rows", (3, 54, 40, "s64"): "rows", (3, 20, 96, "s64"): "rows",
    (3, 72, 3, "s32"): "rows", (3, 72, 7, "s32"): "two", (3, 20, 96, "s32"): "rows",
    (3, 4, 400, "f"): "rows", (3, 4, 525, "f"): "two", (3, 40, 3, "f"): "two",
    (3, 44, 3, "f"): "two", (3, 29, 40, "f"): "two", (3, 29, 100, "f"): "rows",
    (2, 260, 17, "f"): "two", (2, 300, 17, "f"): "rows", (2, 33, 60, "f"): "rows"}


def test_choice(tmp_path):
    exe = str(tmp_path / "rows_pay")
    cmd = [build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-function",
           "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
           os.path.join(HERE, "native", "rows_pay.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        pytest.fail("hipcc failed:\n" + r.stderr[-2000:])
    env = {k: v for k, v in os.environ.items() if not k.startswith("HUB_")}
    out = subprocess.run([exe] + [str(v) for key in CHOICE for v in key], capture_output=True,
                         text=True, timeout=120, env=env)
    assert out.returncode == 0, out.stderr
    assert dict(zip(CHOICE, out.stdout.split())) == CHOICE


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(3, 63, 3), (3, 67, 7), (3, 44, 3), (3, 4, 525), (2, 260, 17)],
                         ids=lambda s: "d%d_%dx%d" % s)
def test_products(shape):
    """Tolerances as in test_gpu_apply.py and test_gpu_cheb.py."""
    import oracle
    import torch
    hubtest.ensure_built()
    oracle.set_threads(16)
    hubtest.log_case(f"rows or two passes {shape}")
    olat, lat = oracle.Lattice(*shape), hub.lattice(*shape)
    sigma, x = inputs.sigma_eta(*shape, seed=23)
    A = oracle.links(olat, sigma)
    ref = oracle.apply_MtM(olat, A, x)
    for vec, dtype, tol in ((hub.F64, torch.float64, 1e-13), (hub.F32, torch.float32, 2e-6)):
        z = hubtest.empty(lat.volume, vec)
        hub.hub_apply_MtM(lat, hubtest.to_dev(A, dtype), vec, vec, hubtest.to_dev(x, dtype), z)
        assert hubtest.rel_err(z.cpu().numpy().astype(np.float64), ref) <= tol
    A_d, x_d, cheb = hubtest.to_dev(A), hubtest.to_dev(x), hub.cheb_opts(3, 0.01)
    z, z2 = hubtest.empty(lat.volume, hub.F64), hubtest.empty(lat.volume, hub.F64)
    hub.hub_apply_cheb(lat, A_d, x_d, z, cheb)
    hub.hub_apply_cheb_noalloc(lat, A_d, x_d, z2, cheb)
    assert torch.equal(z, z2)
    assert hubtest.rel_err(z.cpu().numpy(), oracle.cheb_apply(olat, A, x, 3, 0.01)) <= 1e-9
