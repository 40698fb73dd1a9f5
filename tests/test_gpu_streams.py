"""Solves of several threads at once, each with its own stream and context: teams that do not fit the device together take turns, instead of
waiting for one another until the waits expire."""
import threading

import pytest
import torch

from paper_2312_07759_amd import binding

pytestmark = pytest.mark.gpu


def _layer(m, d, k, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    W = torch.randn((m, d), generator=gen, device="cuda") * 0.1
    return W, W[torch.randperm(m, generator=gen, device="cuda")[:k]].clone(), torch.randn((m, d), generator=gen, device="cuda")


def _run(workers):
    """All workers at once; the first exception of a thread is raised here."""
    errors, barrier = [], threading.Barrier(len(workers))

    def go(work):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                barrier.wait()
                work()
        except BaseException as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=go, args=(w,)) for w in workers]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    if errors:
        raise errors[0]


# teams of the whole device (one workgroup of a compute unit), of half of it, and larger than the LDS
@pytest.mark.parametrize("m,d,k,threads", [(300_000, 1, 16, 3), (300_000, 2, 8, 4), (300_000, 1, 4, 4), (2_359_296, 1, 4, 3), (10_000_000, 1, 4, 3),
                                           (100_000, 4, 256, 3), (3_000, 1, 16, 6)])
def test_every_solve_runs_in_one_launch(m, d, k, threads):
    def worker(seed):
        W, C0, G = _layer(m, d, k, seed)
        ctx = binding.Context(0)
        tau = 2.0 * (0.1 * k ** (-1.0 / d)) ** 2
        ref = ctx.forward(W, C0, tau, 0.0, 8, binding.DIST_SQL2)["C"].clone()
        dW = ctx.backward(G, binding.BWD_JFB)["dW"].clone()
        torch.cuda.synchronize()

        def work():
            for _ in range(40):
                f = ctx.forward(W, C0, tau, 0.0, 8, binding.DIST_SQL2)
                b = ctx.backward(G, binding.BWD_JFB)
                # (a wait that expired would have been answered by the stream path)
                assert f["info"].path == binding.PATH_PERSISTENT
                assert b["info"].path == (binding.PATH_PERSISTENT if m < 10_000_000 else binding.PATH_STREAM)
                assert torch.equal(f["C"], ref) and torch.equal(b["dW"], dW)
        return work

    _run([worker(s) for s in range(threads)])


def test_batches_beside_single_layers():
    def batch_worker():
        layers, G = [], []
        for i in range(8):
            W, C0, g = _layer(100_000 + 40_000 * i, 1, 4, i)
            layers.append((W, C0))
            G.append(g)
        b = binding.Batch(len(layers))
        ref = [o["C"].clone() for o in b.forward(layers, 2e-3, 0.0, 8, binding.DIST_SQL2)]
        torch.cuda.synchronize()

        def work():
            for _ in range(30):
                f = b.forward(layers, 2e-3, 0.0, 8, binding.DIST_SQL2)
                g = b.backward(G, binding.BWD_IMPLICIT, tol=1e-6, max_iter=10)
                assert all(o["info"].path == binding.PATH_PERSISTENT for o in f + g)
                assert all(torch.equal(o["C"], r) for o, r in zip(f, ref))
        return work

    def layer_worker():
        W, C0, G = _layer(300_000, 1, 16, 9)
        ctx = binding.Context(0)

        def work():
            for _ in range(60):
                assert ctx.forward(W, C0, 1e-4, 0.0, 8, binding.DIST_SQL2)["info"].path == binding.PATH_PERSISTENT
                assert ctx.backward(G, binding.BWD_JFB)["info"].path == binding.PATH_PERSISTENT
        return work

    _run([batch_worker(), batch_worker(), layer_worker()])


def test_one_stream_and_two_contexts():
    """A call that fails leaves nothing behind that later ones would wait for."""
    a, b = binding.Context(0), binding.Context(0)
    try:
        W, C0, _ = _layer(300_000, 1, 16, 1)
        bad = W.clone()
        bad[5] = float("nan")
        for _ in range(3):
            with pytest.raises(binding.IdkmError):
                a.forward(bad, C0, 1e-4, 0.0, 4, binding.DIST_SQL2)
            assert b.forward(W, C0, 1e-4, 0.0, 4, binding.DIST_SQL2)["info"].path == binding.PATH_PERSISTENT
        a.set_spin_limit(0)                     # every wait expires: answered by the stream path
        a.forward(W, C0, 1e-4, 0.0, 4, binding.DIST_SQL2)
        assert b.forward(W, C0, 1e-4, 0.0, 4, binding.DIST_SQL2)["info"].path == binding.PATH_PERSISTENT
    finally:
        a.close()
        b.close()
