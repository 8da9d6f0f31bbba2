"""A served job of mode fp32 gets the sums of fp32c whatever the server's size: the
row items of a server of few slots and the 64-landmark blocks of one of many."""
import numpy as np
import pytest

from paper_1907_04839_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", [2, 64])
@pytest.mark.parametrize("n,dim,integrator", [(65, 3, "euler"), (1500, 3, "euler"), (130, 2, "euler"),
                                              (700, 3, "rk4"), (130, 2, "rk4")])
def test_served_fp32_is_bitwise_fp32c(slots, n, dim, integrator):
    from paper_1907_04839_amd import lddmm
    pb = synth.random_problem(8000 + n, n, T=3)
    if dim == 2:
        pb = synth.planar(pb)
    got = []
    for mode in ("fp32", "fp32c"):
        with lddmm.Server(3, mode, max_slots=slots, max_n=8000, hbm_budget_bytes=64 << 20,
                          integrator=integrator) as s:
            jid = s.submit(pb.q0, pb.target, pb.sigma, pb.lam, max_iter=4, dim=dim)
            got.append(s.result(jid, timeout=60))
    np.testing.assert_array_equal(got[0]["p0"], got[1]["p0"])
    for k in ("loss", "H0", "mismatch", "grad_norm", "iters", "fevals"):
        assert got[0][k] == got[1][k], k
