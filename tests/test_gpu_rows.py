"""The row kernels (one launch per step, every j in one workgroup) at the sizes
where their launch plan or their tiles change, against the oracle.

Tolerances are the library's bars: 1e-12 for FP64 sums and 1e-5 for FP32 ones,
normwise and row by row.  Sizes: below one row group, one tile of 64 and its
neighbours, several tiles; 1 or 2 workgroups per CU and the sizes around each
change of the rows per wave (m) and of the i-groups; the last size of the row
kernels and the first one of the split kernels (3072 in FP64, 5120 in FP32)."""
import os
import subprocess

import numpy as np
import pytest

from paper_1907_04839_amd import synth

from conftest import rel_err, row_err, to_dev

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TOL = {"fp64": 1e-12, "fp32c": 1e-5, "fp32": 1e-5}
SMALL = [1, 2, 3, 5, 63, 65, 127, 129]
SIZES = {"fp64": SMALL + [511, 513, 767, 769, 1024, 1025, 1536, 1537, 2049, 3072, 3073],
         "fp32c": SMALL + [767, 769, 1024, 1025, 1281, 1537, 2049, 2560, 3073, 5120, 5121],
         "fp32": SMALL + [769, 1281, 5120, 5121]}
CASES = [(m, n) for m, v in SIZES.items() for n in v]


def test_row_plan_covers_every_row_once(tmp_path):
    exe = tmp_path / "row_plan_test"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=address,undefined",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1907_04839_amd", "csrc"),
                    os.path.join(ROOT, "tests", "cpp", "row_plan_test.cpp"), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "row plans ok" in out.stdout


def check(r, o, mode, tag):
    import torch
    torch.cuda.synchronize()
    errs = dict(loss=abs(float(r.loss) - o["loss"]) / abs(o["loss"]),
                H0=abs(float(r.H0) - o["H0"]) / o["H0"])
    for name, got in (("grad", r.grad), ("q1", r.q1), ("grad_q0", r.grad_q0)):
        got = got.cpu().numpy()
        errs[name] = max(rel_err(got, o[name]), row_err(got, o[name]))
    print(f"[{tag} {mode}] " + " ".join(f"{k}={v:.1e}" for k, v in errs.items()), flush=True)
    assert max(errs.values()) <= TOL[mode], errs


@pytest.mark.gpu
@pytest.mark.parametrize("mode,n", CASES)
def test_row_kernels_match_oracle(gpu_ctx, orc_mt, mode, n):
    pb = synth.random_problem(9000 + n, n, T=1)
    r = gpu_ctx.shoot_grad(to_dev(pb.q0), to_dev(pb.p0), to_dev(pb.target), 1, pb.sigma, pb.lam,
                           precision=mode, want_grad_q0=True)
    o = orc_mt.shoot_grad(pb.q0, pb.p0, pb.target, pb.sigma, pb.lam, 1, all_grads=True)
    check(r, o, mode, f"rows n={n}")


@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["fp64", "fp32c"])
@pytest.mark.parametrize("n", [66, 1281])
@pytest.mark.parametrize("dim,integrator,energy", [(2, "euler", "initial"), (3, "rk4", "final"),
                                                   (2, "rk4", "initial")])
def test_row_kernel_variants_match_oracle(gpu_ctx, orc_mt, mode, n, dim, integrator, energy):
    pb = synth.random_problem(9500 + n, n, T=1)
    if dim == 2:
        pb = synth.planar(pb)
    r = gpu_ctx.shoot_grad(to_dev(pb.q0), to_dev(pb.p0), to_dev(pb.target), 1, pb.sigma, pb.lam,
                           precision=mode, want_grad_q0=True, dim=dim, integrator=integrator,
                           energy=energy)
    o = orc_mt.shoot_grad(pb.q0, pb.p0, pb.target, pb.sigma, pb.lam, 1, all_grads=True,
                          energy=energy, integrator=integrator)
    check(r, o, mode, f"rows n={n} d{dim} {integrator} {energy}")
    assert dim == 3 or np.all(r.grad.cpu().numpy()[:, 2] == 0.0)
