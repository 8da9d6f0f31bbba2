"""The 64-landmark block items, which a server of many slots runs: a job's result is
the same alone and in a mix of 3D and planar jobs (bitwise), and matches the oracle
with Euler steps and Runge-Kutta stages.

The first L-BFGS iteration moves p0 along the gradient there, so from a given p0 the
displacement's direction is compared as a gradient is, normwise at the library's bars
(1e-12 for FP64 sums, 1e-5 for FP32 ones) and row by row at the row gates; subtracting p0 from the iterate costs a few ulps of |p0|
over the displacement's size, below 1e-13 here."""
import numpy as np
import pytest

from paper_1907_04839_amd import synth

from conftest import ROW_TOL, rel_err, row_err

pytestmark = pytest.mark.gpu
SLOTS, MAX_N = 64, 4096      # 64-landmark blocks in every precision
KEYS = ("loss", "H0", "mismatch", "grad_norm", "avg_dist", "max_dist", "iters", "fevals", "status")


def job(k, n, T, dim):
    pb = synth.random_problem(6000 + k, n, T=T)
    return (synth.planar(pb) if dim == 2 else pb), dim


def serve(jobs, T, mode, integrator, iters):
    from paper_1907_04839_amd import lddmm
    with lddmm.Server(T, mode, max_slots=SLOTS, max_n=MAX_N, hbm_budget_bytes=256 << 20,
                      integrator=integrator) as s:
        ids = [s.submit(pb.q0, pb.target, pb.sigma, pb.lam, max_iter=iters, dim=dim)
               for pb, dim in jobs]
        return [s.result(i, timeout=120) for i in ids]


@pytest.mark.parametrize("mode,integrator", [("fp32c", "euler"), ("fp32c", "rk4"),
                                             ("fp32", "euler"), ("fp64", "euler"), ("fp64", "rk4")])
def test_block_results_are_bitwise_the_same_alone_and_in_the_mix(mode, integrator):
    sizes = [(700, 3), (64, 2), (1500, 3), (333, 2), (65, 3), (1, 3), (900, 2), (129, 3)]
    jobs = [job(k, n, 3, dim) for k, (n, dim) in enumerate(sizes)]
    mixed = serve(jobs, 3, mode, integrator, 5)
    for jb, m in zip(jobs, mixed):
        a = serve([jb], 3, mode, integrator, 5)[0]
        np.testing.assert_array_equal(a["p0"], m["p0"])
        for k in KEYS:
            assert a[k] == m[k], k


@pytest.mark.parametrize("mode", ["fp32c", "fp32", "fp64"])
@pytest.mark.parametrize("integrator", ["euler", "rk4"])
@pytest.mark.parametrize("n,dim", [(1, 3), (64, 3), (65, 2), (1000, 3), (1000, 2), (4096, 3)])
def test_block_step_matches_oracle(orc_mt, mode, integrator, n, dim):
    from paper_1907_04839_amd import lddmm
    T = 2
    pb, _ = job(100 + n, n, T, dim)
    with lddmm.Server(T, mode, max_slots=SLOTS, max_n=MAX_N, hbm_budget_bytes=64 << 20,
                      integrator=integrator) as s:
        r = s.result(s.submit(pb.q0, pb.target, pb.sigma, pb.lam, p0=pb.p0, max_iter=1, dim=dim),
                     timeout=120)
    g = orc_mt.shoot_grad(pb.q0, pb.p0, pb.target, pb.sigma, pb.lam, T, integrator=integrator)["grad"]
    a, b = pb.p0 - r["p0"], g
    a, b = a / np.linalg.norm(a), b / np.linalg.norm(b)
    e, rows = rel_err(a, b), row_err(a, b)
    print(f"[blocks {mode} d{dim} {integrator} n={n}] direction={e:.1e} rows={rows:.1e}", flush=True)
    assert r["iters"] == 1
    assert e <= (1e-12 if mode == "fp64" else 1e-5) and rows <= ROW_TOL[mode]
