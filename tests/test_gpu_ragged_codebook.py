"""Codebooks of 3 .. 15 codewords whose size is not a power of two: the persistent path runs them in the lane<->vector
kernels of the next power of two, with the surplus codewords' weights held at zero.  Held to the float64 oracle and to the
stream path (d = 1 and 2: the row<->vector passes, d = 4: the lane<->codeword ones) over team sizes, both energies, all backward modes and batched calls."""
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


def _problem(m, d, k, seed, shift=0.0):
    W, C0, G = wl.random_problem(m, d, k, seed=seed, std=0.5, spread=1.5)
    C0 = C0 + 0.01 * np.random.default_rng(seed + 1).standard_normal(C0.shape)
    return (W + shift).astype(np.float32), (C0 + shift).astype(np.float32), G.astype(np.float32)


# one workgroup (also fewer vectors than threads), the smallest team of eight, dies of different sizes, a full device
@pytest.mark.parametrize("dist", [wl.DIST_L2, wl.DIST_SQL2])
@pytest.mark.parametrize("k,d,m", [(3, 1, 4_096), (3, 1, 4_099), (3, 2, 300_007), (3, 4, 37), (5, 1, 9_001), (6, 2, 4_097),
                                   (7, 4, 20_011), (7, 1, 15), (9, 1, 70_001), (11, 2, 8_191), (12, 4, 30_003),
                                   (13, 1, 300_001), (15, 2, 1_000), (15, 4, 70_003)])
def test_every_padded_shape_against_the_oracle_and_the_stream_path(ctx, k, d, m, dist):
    W, C0, G = _problem(m, d, k, seed=11 * k + d + m)
    Wd, Cd, Gd = dev(W), dev(C0), dev(G)
    tau, iters = 0.15, 15
    ref = orc.soft_kmeans(W, C0, tau, 0.0, iters, dist)
    guard = torch.full((k + 1, d), 9.0, device="cuda")
    f = ctx.forward(Wd, Cd, tau, 0.0, iters, dist, want_A=True, want_assign=True, out={"C": guard[:k]})
    assert f["info"].path == binding.PATH_PERSISTENT and f["info"].iters == iters and f["info"].empty_clusters == 0
    assert torch.all(guard[k:] == 9.0)      # nothing behind the k codewords is written
    Cg = f["C"].cpu().numpy()
    assert rel(Cg, ref["C"]) < TOL_VAL
    A = orc.attention(W, Cg, tau, dist)
    assert rel(f["A"].cpu().numpy(), A) < TOL_VAL
    assert rel(f["Wq"].cpu().numpy(), orc.soft_quantize(W, Cg, tau, dist)) < TOL_VAL
    assert np.array_equal(f["assign"].cpu().numpy(), orc.hard_assign_f32(W, Cg))
    res = {}
    for name, mode, kw in (("jfb", binding.BWD_JFB, {}), ("implicit", binding.BWD_IMPLICIT, dict(tol=0.0, max_iter=8)),
                           ("gmres", binding.BWD_GMRES, dict(tol=1e-5, max_iter=200))):
        res[name] = ctx.backward(Gd, mode, **kw)
        assert res[name]["info"].path == binding.PATH_PERSISTENT
        v, g = ctx.get_cotangents(k, d)
        if name == "gmres":
            r = v + orc.vjp_F(Cg, W, tau, dist, g)[0] - g
            assert np.linalg.norm(r) < TOL_GRAD * np.linalg.norm(v)
        else:
            rb = orc.backward(W, Cg, tau, dist, G, name, tol=0.0, max_iter=8)
            assert rel(v, rb["v"]) < TOL_GRAD and rel(res[name]["dW"].cpu().numpy(), rb["dW"]) < TOL_GRAD
    with pytest.raises(binding.IdkmError):
        ctx.backward(Gd, binding.BWD_DENSE)     # offered for powers of two only
    # the general path at the same codebook
    ctx.set_path(binding.PATH_STREAM)
    try:
        s = ctx.forward(Wd, Cd, tau, 0.0, iters, dist, want_A=True, want_assign=True)
        assert s["info"].path == binding.PATH_STREAM
        Cs = s["C"].cpu().numpy()
        assert rel(Cg, Cs) < 1e-5
        assert rel(s["A"].cpu().numpy(), orc.attention(W, Cs, tau, dist)) < TOL_VAL
        assert rel(s["Wq"].cpu().numpy(), orc.soft_quantize(W, Cs, tau, dist)) < TOL_VAL
        assert np.array_equal(s["assign"].cpu().numpy(), orc.hard_assign_f32(W, Cs))
        sj = ctx.backward(Gd, binding.BWD_JFB)
        assert rel(res["jfb"]["dW"].cpu().numpy(), sj["dW"].cpu().numpy()) < 1e-4
        si = ctx.backward(Gd, binding.BWD_IMPLICIT, tol=0.0, max_iter=8)
        assert si["info"].path == binding.PATH_STREAM
        ri = orc.backward(W, Cs, tau, dist, G, "implicit", tol=0.0, max_iter=8)
        assert rel(ctx.get_cotangents(k, d)[1], ri["g"]) < TOL_GRAD and rel(si["dW"].cpu().numpy(), ri["dW"]) < TOL_GRAD
    finally:
        ctx.set_path(binding.PATH_AUTO)


@pytest.mark.parametrize("dist", [wl.DIST_L2, wl.DIST_SQL2])
@pytest.mark.parametrize("k,d", [(3, 1), (5, 2), (12, 4)])
def test_padding_does_not_shift_rows_far_from_the_origin_or_from_every_codeword(ctx, k, d, dist):
    """Layers at 100 spreads from the origin, and vectors so far out that every unshifted weight of the row underflows;
    one codeword so far away that its cluster is empty keeps its place."""
    m = 9_001
    W, C0, G = _problem(m, d, k, seed=5 * k + d, shift=100.0)
    W[::997] += 40.0
    C0[k - 1] = 5.0e3
    tau = 0.05
    ref = orc.soft_kmeans(W, C0, tau, 0.0, 5, dist)
    f = ctx.forward(dev(W), dev(C0), tau, 0.0, 5, dist)
    Cg = f["C"].cpu().numpy()
    assert f["info"].path == binding.PATH_PERSISTENT and f["info"].empty_clusters == 1
    assert np.array_equal(Cg[k - 1], C0[k - 1])
    assert rel(Cg[:k - 1] - 100.0, ref["C"][:k - 1] - 100.0) < 1e-3
    b = ctx.backward(dev(G), binding.BWD_JFB)
    assert rel(b["dW"].cpu().numpy(), orc.backward(W, Cg, tau, dist, G, "jfb")["dW"]) < TOL_GRAD


def test_batched_ragged_layers_share_launches_and_explicit_path_keeps_its_limits(ctx):
    shapes = [(70_001, 1, 3), (4_001, 1, 3), (9_000, 1, 3), (20_011, 2, 6), (5_000, 2, 5)]
    layers = [_problem(m, d, k, seed=i) for i, (m, d, k) in enumerate(shapes)]
    b = binding.Batch(len(shapes))
    fw = b.forward([(dev(W), dev(C0)) for W, C0, _ in layers], 0.1, 0.0, 12, wl.DIST_SQL2)
    assert b.launches() == 2 and all(o["info"].path == binding.PATH_PERSISTENT for o in fw)
    bw = b.backward([dev(G) for _, _, G in layers], binding.BWD_IMPLICIT, tol=0.0, max_iter=6)
    for (W, C0, G), f, r in zip(layers, fw, bw):
        Cg = f["C"].cpu().numpy()
        assert rel(Cg, orc.soft_kmeans(W, C0, 0.1, 0.0, 12, wl.DIST_SQL2)["C"]) < TOL_VAL
        rb = orc.backward(W, Cg, 0.1, wl.DIST_SQL2, G, "implicit", tol=0.0, max_iter=6)
        assert rel(r["dW"].cpu().numpy(), rb["dW"]) < TOL_GRAD
    b.close()
    W, C0, G = layers[1]
    ctx.set_path(binding.PATH_PERSISTENT)
    try:
        ctx.forward(dev(W), dev(C0), 0.1, 0.0, 5, wl.DIST_SQL2)
        with pytest.raises(binding.IdkmError):      # the Krylov solve was never offered under the explicit path here
            ctx.backward(dev(G), binding.BWD_GMRES)
    finally:
        ctx.set_path(binding.PATH_AUTO)


def test_wide_totals_do_not_meet_the_words_of_other_solves(ctx):
    """One context alternates between k = 3, 4 and 7: the same bits every time.  So too where the sequence numbers start over
    and every word of the exchange is left from a solve of other data that had the same numbers."""
    probs = {k: _problem(30_011, 1, k, seed=k) for k in (3, 4, 7)}
    d = {k: (dev(W), dev(C0), dev(G)) for k, (W, C0, G) in probs.items()}
    c = binding.Context(0)

    def solve(k, ctx):
        f = ctx.forward(d[k][0], d[k][1], 0.2, 0.0, 30, wl.DIST_SQL2)
        b = ctx.backward(d[k][2], binding.BWD_IMPLICIT, tol=0.0, max_iter=5)
        assert f["info"].path == binding.PATH_PERSISTENT
        return f["C"].clone(), b["dW"].clone()

    first = {k: solve(k, c) for k in (3, 4, 7)}
    for k in (3, 7, 4, 3, 4, 7):
        assert all(torch.equal(x, y) for x, y in zip(first[k], solve(k, c)))
    c.close()
    for k in (3, 7):
        c = binding.Context(0)
        W, C0, G = _problem(30_011, 1, k, seed=50 + k)
        c.forward(dev(W), dev(C0), 0.2, 0.0, 30, wl.DIST_SQL2)      # numbers 1 .. 31
        c.backward(dev(G), binding.BWD_IMPLICIT, tol=0.0, max_iter=5)
        c.advance_sequence(0xFFFFFFFF)                              # fewer than 31 are left: the next launch starts at 1 again
        for j in (k, 4, 7, 3):
            assert all(torch.equal(x, y) for x, y in zip(first[j], solve(j, c)))
        c.close()
