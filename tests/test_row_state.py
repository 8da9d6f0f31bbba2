"""A row workgroup reads no state that another workgroup of the same launch stores.

The wave that ends a step has more lanes than the workgroup has rows; the plans'
indexes are walked on the CPU, and the kernels have to take theirs from the same
function."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1907_04839_amd", "csrc")


def test_row_workgroups_read_their_own_state(tmp_path):
    exe = tmp_path / "row_state_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=address,undefined",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "cpp", "row_state_test.cpp"), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "row states ok" in out.stdout


def test_row_kernels_load_states_by_that_index():
    with open(os.path.join(CSRC, "shoot_kernels.hip")) as f:
        src = f.read()
    for fn in ("fwd_rows", "adj_rows"):
        body = src[src.index(f"void {fn}("):]
        body = body[:body.index("\n}\n")]
        loads = re.findall(r"load_(?:fwd|adj)_state<RKS>\(A, (.*)\);", body)
        assert len(loads) == 2 and set(loads) == {"row_state(row0, A.ig * M, lane)"}, loads
