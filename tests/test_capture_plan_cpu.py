"""Plain steps mixed with launches captured by the caller, over the library's own step loop (tests/cpp/capture_plan_check.cpp)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_captured_launches_find_the_state(tmp_path):
    exe = str(tmp_path / "capture_plan_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-o", exe, os.path.join(HERE, "cpp", "capture_plan_check.cpp")], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout
    assert out.stdout.startswith("ok")
