"""The stream-K split as the kernels read it from their arguments (no GPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_walk_and_pieces(tmp_path):
    exe = str(tmp_path / "streamk_walk_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_1412_4564_amd", "csrc"),
                           "-o", exe, os.path.join(ROOT, "tests", "streamk_walk_check.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("OK"), r.stdout[-500:] + r.stderr[-500:]
