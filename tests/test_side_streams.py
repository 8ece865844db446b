"""The fork and join of launches on side streams (side_streams.hpp) on stand-ins of the HIP
calls: the caller's stream waits for every launch queued, also when a later one failed."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = "/opt/rocm/include"


@pytest.mark.skipif(not os.path.isdir(ROCM), reason="HIP headers not available")
def test_the_caller_waits_for_every_queued_launch(tmp_path):
    exe = str(tmp_path / "side_streams")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unused-result",
                    "-D__HIP_PLATFORM_AMD__", "-I", ROCM,
                    "-I", os.path.join(ROOT, "paper_1006_3340_amd", "csrc"),
                    os.path.join(HERE, "helpers", "side_streams_driver.cpp"), "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
