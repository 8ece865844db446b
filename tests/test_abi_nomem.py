"""No exception leaves the C ABI when the host has no memory left: lll_plan_nodes, which
reads one count per Euler step, on host code alone (tests/helpers/abi_nomem_driver.cpp)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = "/opt/rocm/bin/hipcc"
CSRC = os.path.join(ROOT, "paper_1006_3340_amd", "csrc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_plan_nodes_returns_a_status_without_host_memory(tmp_path):
    host = ["-x", "hip", "--cuda-host-only", "-O1", "-std=c++17",
            "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    objs = []
    for src, flags in ((os.path.join(CSRC, "abi.hip"), host),
                       (os.path.join(HERE, "helpers", "abi_host_stubs.cpp"), host),
                       (os.path.join(HERE, "helpers", "abi_nomem_driver.cpp"), host),
                       (os.path.join(CSRC, "noalloc.hip"),
                        ["-x", "hip", "--offload-arch=gfx950", "-O1", "-std=c++17",
                         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", *host[5:]])):
        obj = str(tmp_path / (os.path.basename(src) + ".o"))
        subprocess.run([HIPCC, *flags, "-c", src, "-o", obj], check=True, capture_output=True)
        objs.append(obj)
    exe = str(tmp_path / "abi_nomem")
    subprocess.run([HIPCC, "--offload-arch=gfx950", *objs, "-o", exe], check=True,
                   capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60,
                       env=dict(os.environ, HIP_VISIBLE_DEVICES=""))
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
