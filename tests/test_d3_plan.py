"""The tile of the bare d = 3 product by the number of slices (csrc/sweep.h): on
the CPU the plan on both sides of each line, where it is the faster of the two as
measured on MI355X; on the GPU the product there, against the oracle."""
import os
import subprocess

import numpy as np
import pytest

from paper_1007_3432_amd import build, hub, inputs
from tests import hubtest

HERE = os.path.dirname(os.path.abspath(__file__))
LOW, TALL = "32x8x4@512", "32x8x8@512"
PLANS = {(32, 8, 64): LOW, (32, 24, 64): LOW, (32, 25, 64): TALL, (32, 256, 64): TALL,
         (32, 257, 64): LOW, (32, 384, 64): LOW, (32, 512, 64): LOW, (32, 640, 64): LOW,
         (32, 641, 64): TALL, (32, 768, 64): TALL, (32, 769, 64): LOW,
         (32, 24, 32): LOW, (32, 25, 32): TALL, (32, 257, 32): TALL,
         (64, 16, 32): "64x4x4@512", (64, 17, 32): "64x4x4@256", (64, 25, 32): "64x4x4@256",
         (64, 26, 32): "64x4x4@512", (64, 17, 64): "64x4x4@512"}


def test_tile_by_slices(tmp_path):
    exe = str(tmp_path / "d3_plan")
    cmd = [build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-function",
           "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
           os.path.join(HERE, "native", "d3_plan.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        pytest.fail("hipcc failed:\n" + r.stderr[-2000:])
    env = {k: v for k, v in os.environ.items() if not k.startswith("HUB_")}
    out = subprocess.run([exe] + [str(v) for key in PLANS for v in key], capture_output=True,
                         text=True, timeout=120, env=env)
    assert out.returncode == 0, out.stderr
    got = dict(zip(PLANS, out.stdout.split()))
    assert got == PLANS


@pytest.mark.gpu
@pytest.mark.parametrize("shape,vec,tol", [
    ((3, 32, 24), hub.F64, 1e-13), ((3, 32, 25), hub.F64, 1e-13), ((3, 32, 257), hub.F64, 1e-13),
    ((3, 32, 641), hub.F64, 1e-13), ((3, 64, 17), hub.F32, 2e-6), ((3, 64, 26), hub.F32, 2e-6)],
    ids=["32x24", "32x25", "32x257", "32x641", "64x17", "64x26"])
def test_product_by_slices(shape, vec, tol):
    """Tolerances as in test_gpu_apply.py."""
    import oracle
    import torch
    hubtest.ensure_built()
    oracle.set_threads(16)
    hubtest.log_case(f"mtm {shape} vec {vec}")
    olat, lat = oracle.Lattice(*shape), hub.lattice(*shape)
    sigma, x = inputs.sigma_eta(*shape, seed=19)
    A = oracle.links(olat, sigma)
    dtype = torch.float64 if vec == hub.F64 else torch.float32
    z_d = hubtest.empty(lat.volume, vec)
    hub.hub_apply_MtM(lat, hubtest.to_dev(A, dtype), vec, vec, hubtest.to_dev(x, dtype), z_d)
    z, ref = z_d.cpu().numpy().astype(np.float64), oracle.apply_MtM(olat, A, x)
    assert hubtest.rel_err(z, ref) <= tol
    assert np.max(np.abs(z - ref)) <= 4 * tol * np.max(np.abs(ref))
