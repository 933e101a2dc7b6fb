"""Which pooling calls go through LDS, and the LDS they ask for (tests/pool_tiles_check.cpp, on the host)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_pooling_tiles(tmp_path):
    exe = str(tmp_path / "pool_tiles_check")
    subprocess.check_call([HIPCC, "-x", "hip", "-O2", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                           "-w", "-I", os.path.join(ROOT, "paper_1412_4564_amd", "csrc"), "-o", exe, os.path.join(ROOT, "tests", "pool_tiles_check.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.endswith("OK\n"), r.stdout[-800:] + r.stderr[-500:]
