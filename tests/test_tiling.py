"""The tiles of a packed batch (hb_plan_rules.hpp), on the host."""
import subprocess
from pathlib import Path

HERE = Path(__file__).resolve().parent


def test_tiles_of_a_packed_batch(tmp_path):
    exe = tmp_path / "tiling_check"
    r = subprocess.run(["g++", "-std=c++17", "-O1", str(HERE / "cpp" / "tiling_check.cpp"), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "tiling ok" in out.stdout
