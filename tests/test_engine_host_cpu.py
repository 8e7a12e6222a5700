"""The host engine's launches, waits and results on a stand-in device (CPU
only): tests/host/engine_scenarios.cpp, one scenario a test."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def scenarios(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("engine") / "engine_scenarios")
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-std=c++17", "-O1", "-g", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_1205_0106_amd", "csrc"),
                        os.path.join(HERE, "host", "engine_scenarios.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.mark.parametrize("name", ["mixed_timeout", "order_across_streams", "claim_queues",
                                  "served_share", "segments", "tile_table", "spin_limit",
                                  "one_group_a_unit", "wide_options"])
def test_scenario(scenarios, name):
    r = subprocess.run([scenarios, name], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "passed" in r.stdout, r.stdout + r.stderr
