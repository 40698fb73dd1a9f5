"""Layers read from memory in every pass: a lane's float32 sums move to float64 every 32 vectors (64 on the stream path's pass that forms the
operator), whatever the size of the layer.  References in float64 on the GPU, or the stream path (which the other tests hold to the oracle)."""
import pytest
import torch

from paper_2312_07759_amd import binding

pytestmark = pytest.mark.gpu

MODES = {"jfb": binding.BWD_JFB, "implicit": binding.BWD_IMPLICIT, "gmres": binding.BWD_GMRES, "dense": binding.BWD_DENSE}
DISTS = {"l2": binding.DIST_L2, "sql2": binding.DIST_SQL2}


def _layer(m, d, k, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    W = torch.randn((m, d), generator=gen, device="cuda") * 0.1
    if d == 1:
        C0 = (torch.arange(k, device="cuda").reshape(k, 1) + 0.5) * (0.4 / k) - 0.2
    else:
        C0 = W[:k].clone() + 0.02 * torch.randn((k, d), generator=gen, device="cuda")
    return W, C0, torch.randn((m, d), generator=gen, device="cuda")


def _tau(k, dist):
    return 0.1 / k if dist == "l2" else 2.0 * (0.1 / k) ** 2


def _solve64(W, C, tau, dist, iters):
    C = C.double()
    for _ in range(iters):
        n, s = torch.zeros(C.shape[0], dtype=torch.float64, device="cuda"), torch.zeros_like(C)
        for w in W.split(1 << 22):
            w = w.double()
            E = (w - C.t().contiguous()) ** 2
            A = torch.softmax((E.sqrt() if dist == "l2" else E) * (-1.0 / tau), dim=1)
            n += A.sum(0)
            s += (A * w).sum(0)[:, None]
        C = s / n[:, None]
    return C


@pytest.mark.parametrize("k,dist", [(8, "l2"), (4, "sql2"), (2, "l2")])
def test_error_does_not_grow_with_the_layer(k, dist):
    """60 M weights, 458 of a lane: 6e-8 is the rounding of the codebook, and twice that what runs of 32 and five evaluations leave room
    for (seen 4e-8); single runs gave 1.2e-6 and 1.2e-7 for the first two."""
    W, C0, _ = _layer(60_000_001, 1, k, seed=k)
    tau = _tau(k, dist)
    ctx = binding.Context(0)
    try:
        f = ctx.forward(W, C0, tau, 0.0, 5, DISTS[dist])
        assert f["info"].path == binding.PATH_PERSISTENT
        ref = _solve64(W, C0, tau, dist, 5)
        err = float(torch.linalg.norm(f["C"].double() - ref) / torch.linalg.norm(ref))
        assert err < 1.2e-7, err
    finally:
        ctx.close()


# vectors of the team's run (32 of each of 256 x 512 lanes; 256 x 256 from k d = 32, backward from k d = 16 on) and just beyond, then several
@pytest.mark.parametrize("k,d,dist", [(2, 1, "sql2"), (4, 1, "sql2"), (4, 1, "l2"), (8, 1, "l2"), (4, 2, "sql2"), (4, 4, "l2"), (16, 2, "sql2")])
@pytest.mark.parametrize("m", [32 * 65_536, 32 * 131_072 - 3, 32 * 131_072 + 5, 10_000_003])
def test_runs_end_together(k, d, dist, m):
    W, C0, G = _layer(m, d, k, seed=k + d)
    tau = _tau(k, dist) * d
    ctx = binding.Context(0)
    try:
        ctx.set_path(binding.PATH_STREAM)
        ref = ctx.forward(W, C0, tau, 0.0, 3, DISTS[dist])
        modes = ["jfb", "implicit", "gmres"] + (["dense"] if k * d <= 4 else [])
        grads = {x: ctx.backward(G, MODES[x], tol=1e-6, max_iter=4)["dW"].clone() for x in modes}
        ctx.set_path(binding.PATH_PERSISTENT)
        ctx.set_tile_limit(0)
        got = ctx.forward(W, C0, tau, 0.0, 3, DISTS[dist])
        assert got["info"].path == binding.PATH_PERSISTENT
        # each side within 1e-7 of the 64-bit codebook, three evaluations; gradients amplify that by at most 1 / tau times the spread
        assert float((got["C"] - ref["C"]).abs().max()) < 1e-6 * float(ref["C"].abs().max())
        for x in modes:
            b = ctx.backward(G, MODES[x], tol=1e-6, max_iter=4)
            assert b["info"].path == binding.PATH_PERSISTENT
            err = float(torch.linalg.norm((b["dW"] - grads[x]).double()) / torch.linalg.norm(grads[x].double()))
            assert err < 5e-5, (x, err)
    finally:
        ctx.close()
