"""The point flow's launches (one or two points per lane, a wave per chunk or per
pair of chunks, a velocity spread over workgroups) give a point the same bits,
and match the oracle at the edges of the chunks and tiles.  Tolerances are the
library's bars, row by row."""
import numpy as np
import pytest

from paper_1907_04839_amd import synth

from conftest import row_err, to_dev

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-12, "fp32c": 1e-5, "fp32": 1e-5}


def pts(seed, m):
    return np.ascontiguousarray(4.0 * np.random.default_rng(seed).standard_normal((m, 3)))


@pytest.mark.parametrize("mode", ["fp64", "fp32c", "fp32"])
@pytest.mark.parametrize("n", [1, 63, 65, 127, 129, 255, 257, 511, 1023, 1025, 2049])
def test_velocity_at_chunk_edges(gpu_ctx, orc_mt, mode, n):
    import torch
    pb = synth.random_problem(3100 + n, n, T=1)
    x = pts(3200 + n, 131)
    v = gpu_ctx.velocity(to_dev(pb.q0), to_dev(pb.p0), to_dev(x), pb.sigma, precision=mode)
    torch.cuda.synchronize()
    e = row_err(v.cpu().numpy(), orc_mt.velocity(pb.q0, pb.p0, x, pb.sigma))
    assert e <= TOL[mode], e


@pytest.mark.parametrize("mode,dim,integrator", [("fp32c", 3, "euler"), ("fp32c", 2, "euler"),
                                                 ("fp32", 3, "rk4"), ("fp64", 3, "euler"),
                                                 ("fp64", 2, "rk4")])
def test_every_launch_gives_a_point_the_same_bits(gpu_ctx, orc_mt, mode, dim, integrator):
    """131072 points (two per lane in FP32, a wave per pair of chunks in FP64)
    against the first 100 and the first 40001 alone; the 100 against the oracle."""
    import torch
    pb = synth.random_problem(3300, 1100, T=2)
    x = pts(3301, 131072)
    if dim == 2:
        pb = synth.planar(pb)
        x[:, 2] = 0.0
    q, p, xd = to_dev(pb.q0), to_dev(pb.p0), to_dev(x)
    kw = dict(precision=mode, dim=dim)
    full = gpu_ctx.flow(q, p, xd, 2, pb.sigma, integrator=integrator, **kw)
    vfull = gpu_ctx.velocity(q, p, xd, pb.sigma, **kw)
    for m in (100, 40001):
        part = xd[:m].contiguous()
        got = gpu_ctx.flow(q, p, part, 2, pb.sigma, integrator=integrator, **kw)
        assert torch.equal(got, full[:m])
        assert torch.equal(gpu_ctx.velocity(q, p, part, pb.sigma, **kw), vfull[:m])
    ref = orc_mt.flow(pb.q0, pb.p0, x[:100], pb.sigma, 2, integrator=integrator)["x1"]
    assert row_err(full[:100].cpu().numpy() - x[:100], ref - x[:100]) <= TOL[mode]
