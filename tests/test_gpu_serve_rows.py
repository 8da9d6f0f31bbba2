"""The kernels a server's configuration selects: the rule on the CPU, and the row items
at the sizes where their plan changes, against the oracle's solver (row items need a
server of few slots, in FP32 one of max_n up to 15000).

One optimiser iteration from p0 = 0 leaves a multiple of the first gradient in p0, so
its direction is compared as a gradient is; tolerances are the library's bars, 1e-12
for FP64 sums and 1e-5 for FP32 ones (1e-10 where an FP64 step length enters)."""
import os
import subprocess

import numpy as np
import pytest

from paper_1907_04839_amd import synth

from conftest import rel_err, row_err

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_configuration_gets_the_slower_kernels(tmp_path):
    exe = tmp_path / "batch_family_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1907_04839_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cpp", "batch_family_test.cpp"), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and "families ok" in out.stdout, out.stdout


# below one row group, one tile and its neighbours, the last and first size of each
# share of the j tiles (3071 | 3072, in FP64 16383 | 16384), the largest of FP32, several rounds of 18 tiles (above
# 2304 with two waves to the tiles)
CASES = [("fp32c", n, 3, "euler") for n in (1, 3, 64, 65, 257, 3071, 3072, 9300, 15000)]
CASES += [("fp64", n, 3, "euler") for n in (5, 65, 3071, 3072, 9300, 16383, 16385)]
CASES += [("fp32", 3072, 3, "euler"), ("fp32c", 3072, 2, "euler"), ("fp32c", 3072, 3, "rk4"),
          ("fp64", 3072, 2, "rk4")]


@pytest.mark.gpu
@pytest.mark.parametrize("mode,n,dim,integrator", CASES)
def test_served_rows_match_oracle(orc_mt, mode, n, dim, integrator):
    from paper_1907_04839_amd import lddmm
    pb = synth.random_problem(7500 + n, n, T=1)
    if dim == 2:
        pb = synth.planar(pb)
    with lddmm.Server(1, mode, max_slots=2, max_n=20000 if mode == "fp64" else 15000,
                      hbm_budget_bytes=128 << 20, integrator=integrator) as s:
        jid = s.submit(pb.q0, pb.target, pb.sigma, pb.lam, max_iter=1, dim=dim)
        r = s.result(jid, timeout=120)
    if integrator == "euler":
        o = orc_mt.solve(pb.q0, pb.target, pb.sigma, pb.lam, 1, orc_mt.SolveOpts(max_iter=1))
        assert r["iters"] == o["iters"] and r["fevals"] == o["fevals"]
        b, loss = o["p0"], abs(r["loss"] - o["loss"]) / o["loss"]
    else:   # the oracle's solver takes Euler steps: the gradient at p0 = 0 alone
        o = orc_mt.shoot_grad(pb.q0, np.zeros_like(pb.q0), pb.target, pb.sigma, pb.lam, 1,
                              integrator=integrator)
        b, loss = -o["grad"], 0.0
    a, b = r["p0"] / np.linalg.norm(r["p0"]), b / np.linalg.norm(b)
    direction = max(rel_err(a, b), row_err(a, b))
    print(f"[rows {mode} d{dim} {integrator} n={n}] direction={direction:.1e} loss={loss:.1e}",
          flush=True)
    assert direction <= (1e-12 if mode == "fp64" else 1e-5)
    assert loss <= (1e-10 if mode == "fp64" else 1e-5)
