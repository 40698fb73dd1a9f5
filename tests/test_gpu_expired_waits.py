"""Bounded waits of the persistent kernels that expire in some workgroups only: a call that reports success has written all
of its outputs.  The limits are set from the host (idkm_set_spin_limit); every kernel leaves normally."""
import threading

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


@pytest.mark.parametrize("k,d,m", [(16, 4, 1_025), (8, 1, 4_096), (7, 2, 2_001)])
def test_small_layers_need_nobody_to_wait_for(k, d, m):
    """Layers that one workgroup holds run as teams of eight where that is faster.  Where such a team gives up a wait the layer
    is solved by one workgroup -- under the explicit persistent path too -- and idkm_forward_noalloc, which may have nobody to
    read a result, starts with one: the same bits."""
    W, C0, G = wl.random_problem(m, d, k, seed=k + m, std=0.5, spread=1.5)
    C0 = (C0 + 0.01 * np.random.default_rng(k).standard_normal(C0.shape)).astype(np.float32)
    W, G = W.astype(np.float32), G.astype(np.float32)
    Wd, Cd, Gd = dev(W), dev(C0), dev(G)
    tau, dist = 0.15, wl.DIST_L2
    ctx = binding.Context(0)
    for path in (binding.PATH_PERSISTENT, binding.PATH_AUTO):
        ctx.set_path(path)
        ctx.set_spin_limit(0)
        f = ctx.forward(Wd, Cd, tau, 0.0, 12, dist)
        Cg = f["C"].cpu().numpy()
        assert f["info"].path == binding.PATH_PERSISTENT
        assert rel(Cg, orc.soft_kmeans(W, C0, tau, 0.0, 12, dist)["C"]) < 1e-4
        for name, mode, kw in (("jfb", binding.BWD_JFB, {}), ("implicit", binding.BWD_IMPLICIT, dict(tol=0.0, max_iter=5))):
            b = ctx.backward(Gd, mode, **kw)
            assert b["info"].path == binding.PATH_PERSISTENT
            assert rel(b["dW"].cpu().numpy(), orc.backward(W, Cg, tau, dist, G, name, tol=0.0, max_iter=5)["dW"]) < TOL_GRAD
    if k != 7:
        out = dict(C=torch.empty_like(Cd), Wq=torch.empty_like(Wd))
        info = binding.forward_noalloc(Wd, Cd, tau, 0.0, 12, dist, out)
        assert info.residual == f["info"].residual and torch.equal(out["C"], f["C"]) and torch.equal(out["Wq"], f["Wq"])
    ctx.close()


def test_small_teams_beside_other_streams():
    """Small teams, a padded codebook and a full device's solve at once, each with a context, a stream and a thread of its own."""
    shapes = [(16, 4, 1_025), (8, 1, 4_096), (4, 1, 300_007), (40, 1, 20_003)]
    tau, dist = 0.2, wl.DIST_SQL2
    probs = []
    for k, d, m in shapes:
        W, C0, G = wl.random_problem(m, d, k, seed=k + m, std=0.5, spread=1.5)
        probs.append((dev(W), dev(C0), dev(G)))

    def solve(ctx, W, C0, G):
        f = ctx.forward(W, C0, tau, 0.0, 20, dist)
        b = ctx.backward(G, binding.BWD_IMPLICIT, tol=0.0, max_iter=10)
        return f["C"], f["Wq"], b["dW"]

    want = []
    for p in probs:
        ctx = binding.Context(0)
        want.append(solve(ctx, *p))
        ctx.close()
    torch.cuda.synchronize()
    bad = []

    def work(i):
        ctx, stream = binding.Context(0), torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for _ in range(40):
                got = solve(ctx, *probs[i])
                stream.synchronize()
                for x, y in zip(got, want[i]):
                    # (a solve that gave up a wait was answered by another form: equal up to rounding)
                    if not float((x - y).norm()) <= 1e-4 * float(y.norm()):
                        bad.append((shapes[i], float((x - y).norm() / y.norm())))
        ctx.close()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(shapes))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad[:4]
