"""The build's flags across failed builds, on the host alone: the host runtime (ptraster.cpp) linked with stubs of the HIP
calls and the kernel launches (host_build_flags.cpp), one of which fails between a raised flag and its clear."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_failed_build_leaves_nothing_behind(tmp_path):
    exe = tmp_path / "host_build_flags"
    src = os.path.join(HERE, "..", "paper_2204_01287_amd", "csrc", "ptraster.cpp")
    # the launches that no build calls stay undefined
    cmd = ["g++", "-O1", "-std=c++17", "-w", "-no-pie", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
           os.path.join(HERE, "host_build_flags.cpp"), src, "-Wl,--unresolved-symbols=ignore-all", "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "host build flags ok" in r.stdout, (r.returncode, r.stdout, r.stderr)
