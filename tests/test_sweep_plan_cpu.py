"""Strip segments and the choice between sweeps and tile steps, from the library's own plan header (tests/cpp/sweep_plan_check.cpp)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_segments_and_choice(tmp_path):
    exe = str(tmp_path / "sweep_plan_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-o", exe, os.path.join(HERE, "cpp", "sweep_plan_check.cpp")], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
    assert out.stdout.startswith("ok")
