"""The largest tiles that a persistent workgroup of the lane<->vector family keeps in LDS: the solve still runs in one launch, whatever the
kernel that serves the mode needs beside the tile, with the gradient of the stream path (which the other tests hold to the oracle)."""
import numpy as np
import pytest
import torch

from paper_2312_07759_amd import binding

pytestmark = pytest.mark.gpu

# 147456 bytes of W and dL/dWq in each of 256 workgroups
FULL = 256 * 147_456 // 8
# both sides add the same float32 terms in other orders; a gradient element is a difference of a few of them, v a sum of m terms with
# random signs (1e-6 of itself each), and a soft fixed point amplifies v about tenfold
TOL = 5e-5


def _layer(m, d, k, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    W = torch.randn((m, d), generator=gen, device="cuda") * 0.1
    C0 = W[torch.randperm(m, generator=gen, device="cuda")[:k]].clone()
    C0 += 0.01 * torch.randn((k, d), generator=gen, device="cuda")
    return W, C0, torch.randn((m, d), generator=gen, device="cuda")


@pytest.mark.parametrize("mode", ["jfb", "implicit", "gmres"])
@pytest.mark.parametrize("k,d,dist", [(5, 1, "l2"), (7, 1, "l2"), (7, 1, "sql2"), (8, 1, "l2"), (3, 4, "sql2"), (4, 4, "sql2"), (4, 1, "l2")])
def test_largest_tile_and_what_lies_just_below(k, d, dist, mode):
    mode_id = {"jfb": binding.BWD_JFB, "implicit": binding.BWD_IMPLICIT, "gmres": binding.BWD_GMRES}[mode]
    dist_id = binding.DIST_L2 if dist == "l2" else binding.DIST_SQL2
    ctx = binding.Context(0)
    try:
        for m in (FULL // d, FULL // d - 256 * 256 // d - 77):
            W, C0, G = _layer(m, d, k, seed=k + d)
            tau = (0.1 / k) * (4.0 if dist == "l2" else 0.1)
            ctx.set_path(binding.PATH_STREAM)
            ctx.forward(W, C0, tau, 0.0, 3, dist_id)
            ref = ctx.backward(G, mode_id, tol=1e-5, max_iter=20)
            # (a Krylov solve under the explicit path is offered for powers of two alone)
            ctx.set_path(binding.PATH_AUTO if k & (k - 1) else binding.PATH_PERSISTENT)
            got = ctx.backward(G, mode_id, tol=1e-5, max_iter=20)
            assert got["info"].path == binding.PATH_PERSISTENT and got["info"].converged == ref["info"].converged
            err = torch.linalg.norm((got["dW"] - ref["dW"]).double()) / torch.linalg.norm(ref["dW"].double())
            assert float(err) < TOL, (m, float(err))
    finally:
        ctx.close()
