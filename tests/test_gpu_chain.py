"""The chain kernels (every step of up to 64 landmarks in one launch) against the
oracle, and their launches against each other.

Tolerances are the library's bars, 1e-12 for FP64 sums and 1e-5 for FP32 ones.
Sizes: fewer landmarks than waves, around a wave's share of eight, a full wave
and the first size of the row kernels; the checkpoint ring cuts a pass into
launches, whose results are bitwise those of one launch, and a long pass is
more than one launch of 4096 steps."""
import numpy as np
import pytest

from paper_1907_04839_amd import synth

from conftest import rel_err, row_err, to_dev

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-12, "fp32c": 1e-5, "fp32": 1e-5}


def errors(r, o):
    import torch
    torch.cuda.synchronize()
    errs = dict(loss=abs(float(r.loss) - o["loss"]) / abs(o["loss"]),
                H0=abs(float(r.H0) - o["H0"]) / o["H0"])
    for name, got in (("grad", r.grad), ("q1", r.q1), ("grad_q0", r.grad_q0)):
        got = got.cpu().numpy()
        errs[name] = max(rel_err(got, o[name]), row_err(got, o[name]))
    return errs


@pytest.mark.parametrize("mode", ["fp64", "fp32c", "fp32"])
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 63, 64, 65])
@pytest.mark.parametrize("dim,integrator,energy", [(3, "euler", "initial"), (2, "euler", "final"),
                                                   (3, "rk4", "final"), (2, "rk4", "initial")])
def test_chain_matches_oracle(gpu_ctx, orc_mt, mode, n, dim, integrator, energy):
    pb = synth.random_problem(6000 + n, n, T=2)
    if dim == 2:
        pb = synth.planar(pb)
    r = gpu_ctx.shoot_grad(to_dev(pb.q0), to_dev(pb.p0), to_dev(pb.target), 2, pb.sigma, pb.lam,
                           precision=mode, want_grad_q0=True, dim=dim, integrator=integrator,
                           energy=energy)
    o = orc_mt.shoot_grad(pb.q0, pb.p0, pb.target, pb.sigma, pb.lam, 2, all_grads=True,
                          integrator=integrator, energy=energy)
    errs = errors(r, o)
    assert max(errs.values()) <= TOL[mode], errs


@pytest.mark.parametrize("mode", ["fp64", "fp32c"])
@pytest.mark.parametrize("integrator", ["euler", "rk4"])
@pytest.mark.parametrize("every", [1, 3, 4])
def test_chain_segments_are_bitwise_the_whole(gpu_ctx, mode, integrator, every):
    import torch
    pb = synth.random_problem(6100, 37, T=7)
    args = (to_dev(pb.q0), to_dev(pb.p0), to_dev(pb.target), 7, pb.sigma, pb.lam)
    kw = dict(precision=mode, integrator=integrator, want_grad_q0=True)
    a = gpu_ctx.shoot_grad(*args, **kw)
    b = gpu_ctx.shoot_grad(*args, ckpt_every=every, **kw)
    torch.cuda.synchronize()
    for name in ("loss", "grad", "q1", "grad_q0"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name


def test_chain_of_more_than_one_launch(gpu_ctx, orc_mt):
    T = 4099
    pb = synth.random_problem(6200, 5, T=T)
    r = gpu_ctx.shoot_grad(to_dev(pb.q0), to_dev(pb.p0), to_dev(pb.target), T, pb.sigma, pb.lam,
                           precision="fp64", want_grad_q0=True)
    o = orc_mt.shoot_grad(pb.q0, pb.p0, pb.target, pb.sigma, pb.lam, T, all_grads=True)
    errs = errors(r, o)
    # rounding of T steps: the bar times sqrt(T)
    assert max(errs.values()) <= 1e-12 * np.sqrt(T), errs
