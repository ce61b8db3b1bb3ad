"""Plans whose level-slice partials cannot be allocated (tests/level_memory.cpp:
the built library over stand-ins for the HIP calls)."""

import os
import shutil
import subprocess

import pytest

import paper_1710_06189_amd  # noqa: F401  (builds the library if it is not there)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC) and shutil.which("hipcc") is None, reason="hipcc not installed")
def test_no_memory_for_the_partials_is_no_error(tmp_path):
    exe, lib = str(tmp_path / "level_memory"), os.path.join(ROOT, "paper_1710_06189_amd")
    subprocess.check_call([HIPCC if os.path.exists(HIPCC) else "hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17",
                           "-I" + os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "level_memory.cpp"),
                           "-rdynamic", "-L" + lib, "-lglcm", "-Wl,-rpath," + lib, "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
