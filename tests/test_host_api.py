"""Scenarios of the C ABI's host side that a GPU does not bring about on
demand (a launch that fails in the middle of a run, memory that runs out): vg_api.cpp built for the
host alone, with stand-ins for the HIP calls and the kernel launchers
(host_api_harness.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def harness(tmp_path_factory):
    from paper_2406_04177_amd.build import CSRC, hipcc
    out = str(tmp_path_factory.mktemp("host_api") / "harness")
    cmd = [hipcc(), "-O1", "-std=c++17", "-x", "hip", "--offload-host-only", "--offload-arch=gfx950",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, "vg_api.cpp"),
           os.path.join(HERE, "host_api_harness.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


@pytest.mark.parametrize("scenario", ["failed_runs", "no_allocation", "short_runs"])
def test_scenario(harness, scenario):
    r = subprocess.run([harness, scenario], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout + r.stderr
