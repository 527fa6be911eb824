"""Which launches a call makes (one launch or three, which tile, what the tuner
times), on the CPU: the host code as it is, against the stand-ins of
tests/native with every likelihood launch noted."""
import os
import shutil
import subprocess

import pytest

from tests.test_host_sanitizers import CSRC, HIP_INCLUDE, NATIVE

pytestmark = pytest.mark.skipif(
    shutil.which("g++") is None or not os.path.isdir(os.path.join(HIP_INCLUDE, "hip")),
    reason="needs g++ and the HIP headers")


def test_routes_of_small_thin_batches(tmp_path):
    exe = str(tmp_path / "routes")
    src = [os.path.join(CSRC, f) for f in ("fgl_host.cpp", "fgl_serve.cpp", "fgl_plan.cpp")] + \
          [os.path.join(NATIVE, f) for f in ("hip_stub.cpp", "route_test.cpp")]
    p = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", HIP_INCLUDE, "-g", "-O1",
                        "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", *src, "-o", exe,
                        "-lpthread"], capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-4000:]
    env = {k: v for k, v in os.environ.items() if not k.startswith("FGL_") and k != "LD_PRELOAD"}
    p = subprocess.run([exe, str(tmp_path / "tiles.jsonl")], capture_output=True, text=True, env=env,
                       timeout=300)
    assert p.returncode == 0 and "checks failed: 0, stand-in reports: 0" in p.stdout, \
        (p.stdout[-2000:], p.stderr[-6000:])
