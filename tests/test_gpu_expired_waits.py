"""Bounded waits of the persistent kernels that expire in some workgroups only: a call that reports success has written all
of its outputs.  The limits are set from the host (idkm_set_spin_limit); every kernel leaves normally."""
import numpy as np
import pytest
import torch

from oracle import idkm_oracle as orc
from paper_2312_07759_amd import binding
from paper_2312_07759_amd import workloads as wl

pytestmark = pytest.mark.gpu

TOL_GRAD = 1e-3


def rel(x, ref):
    return float(np.linalg.norm(np.asarray(x, dtype=np.float64) - ref) / np.linalg.norm(ref))


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float32).cuda()


# the row, matrix-core, lane and padded families, a small team and a full device; limits from "nobody waits" to about the
# time a pass takes, so that in some launches one workgroup of the last exchange gives up and the others do not
@pytest.mark.parametrize("k,d,m", [(40, 1, 20_003), (256, 4, 5_001), (300, 2, 20_001), (16, 4, 1_025), (3, 1, 30_011), (4, 1, 300_007)])
def test_a_backward_that_reports_success_has_written_every_row(k, d, m):
    W, C0, G = wl.random_problem(m, d, k, seed=k + m, std=0.5, spread=1.5)
    C0 = (C0 + 0.01 * np.random.default_rng(k).standard_normal(C0.shape)).astype(np.float32)
    W, G = W.astype(np.float32), G.astype(np.float32)
    Wd, Cd, Gd = dev(W), dev(C0), dev(G)
    tau, dist = 0.3, wl.DIST_SQL2
    ctx = binding.Context(0)
    full = ctx.forward(Wd, Cd, tau, 0.0, 5, dist)
    Cg = full["C"].cpu().numpy()
    modes = (("jfb", binding.BWD_JFB, {}), ("implicit", binding.BWD_IMPLICIT, dict(tol=0.0, max_iter=3)))
    ref = {name: orc.backward(W, Cg, tau, dist, G, name, tol=0.0, max_iter=3)["dW"] for name, _, _ in modes}
    for limit in list(range(0, 40)) * 3:
        ctx.set_spin_limit(limit)
        for name, mode, kw in modes:
            dW = torch.full((m, d), float("nan"), device="cuda")
            ctx.backward(Gd, mode, out=dW, **kw)
            assert bool(torch.isfinite(dW).all()), (name, limit, int((~torch.isfinite(dW)).sum()))
            if limit in (0, 13):
                assert rel(dW.cpu().numpy(), ref[name]) < TOL_GRAD
        Wq = torch.full((m, d), float("nan"), device="cuda")
        f = ctx.forward(Wd, Cd, tau, 0.0, 5, dist, out={"Wq": Wq})
        assert bool(torch.isfinite(Wq).all()) and float((f["C"] - full["C"]).norm() / full["C"].norm()) < 1e-5
    ctx.close()
