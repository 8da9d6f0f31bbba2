"""The point flow's chunks share the landmarks evenly (CPU)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_flow_chunks_are_equal_shares(tmp_path):
    exe = tmp_path / "flow_plan_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=address,undefined",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1907_04839_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cpp", "flow_plan_test.cpp"), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and "flow plans ok" in out.stdout, out.stdout
