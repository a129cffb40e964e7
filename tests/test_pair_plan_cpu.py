"""The pairs of steps that the step loop fuses, from the library's own plan header (tests/cpp/pair_plan_check.cpp)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_pairs_keep_diagnostics_graphs_and_buffers(tmp_path):
    exe = str(tmp_path / "pair_plan_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-o", exe, os.path.join(HERE, "cpp", "pair_plan_check.cpp")], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout
    assert out.stdout.startswith("ok")
