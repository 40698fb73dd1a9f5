"""Row <-> vector kernels (17 <= k <= 256 and k = 1, d = 1 and 2, persistent path): every block count and its edges, shares
that end inside a step, rows that underflow, against the float64 oracle and the stream path's lane <-> codeword kernels."""
import numpy as np
import pytest
import torch

from oracle import idkm_oracle as orc
from paper_2312_07759_amd import binding
from paper_2312_07759_amd import workloads as wl

pytestmark = pytest.mark.gpu

TOL_VAL, TOL_GRAD = 1e-4, 1e-3


def rel(x, ref):
    x, ref = np.asarray(x, dtype=np.float64), np.asarray(ref, dtype=np.float64)
    den = np.linalg.norm(ref)
    return float(np.linalg.norm(x - ref) / (den if den > 0 else 1.0))


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float32).cuda()


@pytest.fixture(scope="module")
def ctx():
    c = binding.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dist", [wl.DIST_L2, wl.DIST_SQL2])
@pytest.mark.parametrize("k,d,m", [(1, 1, 3_001), (1, 2, 70_001), (17, 1, 17), (17, 2, 513), (32, 1, 2_047), (32, 2, 4_099),
                                   (33, 1, 9_001), (64, 2, 255), (64, 1, 20_011), (65, 2, 3_001), (128, 1, 2_049),
                                   (128, 2, 300), (129, 1, 1_025), (255, 2, 5_003), (256, 1, 70_003), (256, 2, 2_304)])
def test_block_counts_and_ragged_shares(ctx, k, d, m, dist):
    W, C0, G = wl.random_problem(m, d, k, seed=3 * k + d + m, std=0.5, spread=1.5)
    C0 = C0 + 0.01 * np.random.default_rng(k).standard_normal(C0.shape)
    W[::311] += 30.0        # rows whose unshifted weights all underflow
    W, C0, G = W.astype(np.float32), C0.astype(np.float32), G.astype(np.float32)
    Wd, Cd, Gd = dev(W), dev(C0), dev(G)
    tau, iters = 0.2, 6
    ref = orc.soft_kmeans(W, C0, tau, 0.0, iters, dist)
    f = ctx.forward(Wd, Cd, tau, 0.0, iters, dist, want_A=True, want_assign=True)
    assert f["info"].path == binding.PATH_PERSISTENT and f["info"].iters == iters
    Cg = f["C"].cpu().numpy()
    assert rel(Cg, ref["C"]) < TOL_VAL
    assert rel(f["A"].cpu().numpy(), orc.attention(W, Cg, tau, dist)) < TOL_VAL
    assert rel(f["Wq"].cpu().numpy(), orc.soft_quantize(W, Cg, tau, dist)) < TOL_VAL
    assert np.array_equal(f["assign"].cpu().numpy(), orc.hard_assign_f32(W, Cg))
    bj = ctx.backward(Gd, binding.BWD_JFB)
    rj = orc.backward(W, Cg, tau, dist, G, "jfb")
    assert rel(bj["dW"].cpu().numpy(), rj["dW"]) < TOL_GRAD
    assert rel(ctx.get_cotangents(k, d)[0], rj["v"]) < TOL_GRAD
    bi = ctx.backward(Gd, binding.BWD_IMPLICIT, tol=0.0, max_iter=5, alpha=0.5)
    ri = orc.backward(W, Cg, tau, dist, G, "implicit", tol=0.0, max_iter=5, alpha=0.5)
    if not (bi["info"].converged or ri["converged"]):
        assert bi["info"].iters == ri["iters"] and bi["info"].alpha == ri["alpha"]
    assert rel(bi["dW"].cpu().numpy(), ri["dW"]) < TOL_GRAD
    ctx.set_path(binding.PATH_STREAM)
    try:
        s = ctx.forward(Wd, Cd, tau, 0.0, iters, dist, want_Wq=False)
        assert rel(Cg, s["C"].cpu().numpy()) < 1e-5
        assert rel(bj["dW"].cpu().numpy(), ctx.backward(Gd, binding.BWD_JFB)["dW"].cpu().numpy()) < 2e-4
    finally:
        ctx.set_path(binding.PATH_AUTO)
