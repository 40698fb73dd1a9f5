"""A layer that one workgroup solves alone: no sum crosses to another workgroup, so no total is rounded to a float32 word."""
import numpy as np
import pytest
import torch

from oracle import idkm_oracle as orc
from paper_2312_07759_amd import binding
from paper_2312_07759_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = binding.Context(0)
    yield c
    c.close()


def dev(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float32).cuda()


SHAPES = [(2, 1, wl.DIST_SQL2), (4, 1, wl.DIST_L2), (8, 1, wl.DIST_L2), (4, 2, wl.DIST_SQL2), (16, 1, wl.DIST_SQL2)]
MODES = [binding.BWD_JFB, binding.BWD_IMPLICIT, binding.BWD_GMRES, binding.BWD_DENSE]


# (the explicit Jacobian of more than four unknowns is solved on the stream path)
@pytest.mark.parametrize("k,d,dist,mode", [s + (x,) for s in SHAPES for x in MODES if x != binding.BWD_DENSE or s[0] * s[1] <= 4])
def test_totals_of_the_backward_are_float64(ctx, k, d, dist, mode):
    """v is a sum over wavefronts in float64: all of its components fit a float32 only if they were rounded to one (each does by
    chance with 2^-29 or so)."""
    W, C0, G = wl.random_problem(1_003, d, k, seed=k + d, std=0.5, spread=1.0)
    f = ctx.forward(dev(W), dev(C0), 0.2, 0.0, 4, dist)
    assert f["info"].path == binding.PATH_PERSISTENT
    b = ctx.backward(dev(G), mode, tol=1e-6, max_iter=20)
    assert b["info"].path == binding.PATH_PERSISTENT
    v, _ = ctx.get_cotangents(k, d)
    if mode != binding.BWD_DENSE:       # (there v is not kept)
        assert not np.array_equal(v, v.astype(np.float32).astype(np.float64))
    ref = orc.backward(W.astype(np.float32), f["C"].cpu().numpy(), 0.2, dist, G.astype(np.float32), "jfb")
    assert np.max(np.abs(v - ref["v"])) < 1e-5 * np.max(np.abs(ref["v"]))


def test_codebook_of_one_evaluation():
    """One evaluation of 1,000 weights under 8 codewords: what is left is the rounding of the codebook itself (2^-23 / sqrt(12) of the largest
    codeword at most, 3.4e-8, and less for the smaller ones: 1.7e-8 rms over these) and of lanes and rows of 16 (a few 1e-9).  Totals and
    masses rounded to float32, 2^-25 rms each, bring it to 2.9e-8."""
    ctx = binding.Context(0)
    err = []
    try:
        for seed in range(60):
            W, C0, _ = wl.random_problem(1_000, 1, 8, seed=seed, std=0.5, spread=1.0)
            W, C0 = W.astype(np.float32), C0.astype(np.float32)
            C = ctx.forward(dev(W), dev(C0), 0.2, 0.0, 1, wl.DIST_L2)["C"].cpu().numpy()
            ref = orc.soft_kmeans(W, C0, 0.2, 0.0, 1, wl.DIST_L2)["C"]
            err.append(((C - ref) / np.max(np.abs(ref))).ravel())
    finally:
        ctx.close()
    rms = float(np.sqrt(np.mean(np.concatenate(err) ** 2)))
    assert rms < 2.3e-8, rms
