"""The plan of the row tiles depends on the lattice alone: environment variables
of other programs, with names as short as RB or RL, neither change it nor end the
process (csrc/sweep.h compiled for the host, no GPU needed)."""
import os
import subprocess

import pytest

from paper_1007_3432_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rows") / "rows_plan")
    cmd = [build.HIPCC, "-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-function",
           "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
           os.path.join(HERE, "native", "rows_plan.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        pytest.fail("hipcc failed:\n" + r.stderr[-2000:])

    def run(**env):
        base = {k: v for k, v in os.environ.items()
                if k not in ("RB", "RL") and not k.startswith("HUB_")}
        return subprocess.run([exe], capture_output=True, text=True, timeout=120, env=base | env)
    return run


@pytest.mark.parametrize("env", [dict(RB="0"), dict(RB="on"), dict(RB="64"), dict(RL="3"), dict(RL="99")],
                         ids=lambda e: "_".join(f"{k}={v}" for k, v in e.items()))
def test_plan_ignores_foreign_variables(plans, env):
    ref, got = plans(), plans(**env)
    assert ref.returncode == 0 and len(ref.stdout.splitlines()) == 14
    assert got.returncode == 0, f"ended with {got.returncode}"
    assert got.stdout == ref.stdout
