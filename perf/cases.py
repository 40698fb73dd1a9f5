"""The work that users of this package have it do, as a list of timed cases.

A pass is one quantisation step of a layer (soft k-means solve, then the gradient of the layer through that solve) or of a
whole network's layers in one batched call, or the packing and unpacking of a layer's codes.  Sizes are the layers of
ResNet18, the small MNIST network and the 4096 x 4096 linear layer that the package's workloads, tests and benchmark use;
weights are Kaiming-normal stand-ins, upstream gradients N(0, 1e-4^2).

Temperatures: tau = soft (std k^(-1/d))^2 for the squared energy and soft std k^(-1/d) for the plain norm, i.e. `soft` is
the width of a row's softmax in units of the spacing of the codewords, or a fixed `tau` where a workload has its own.
"""
import math

import torch

from paper_2312_07759_amd import autograd, binding

DISTS = {"l2": binding.DIST_L2, "sql2": binding.DIST_SQL2}
MODES = {"implicit": binding.BWD_IMPLICIT, "jfb": binding.BWD_JFB, "gmres": binding.BWD_GMRES}

# Weights and fan-in of the 21 tensors of ResNet18 (first convolution, blocks, downsampling convolutions, classifier).
RESNET18 = (
    [(9_408, 147)] + [(36_864, 576)] * 4 + [(73_728, 576)] + [(147_456, 1152)] * 3 + [(8_192, 64)]
    + [(294_912, 1152)] + [(589_824, 2304)] * 3 + [(32_768, 128)]
    + [(1_179_648, 2304)] + [(2_359_296, 4608)] * 3 + [(131_072, 256)] + [(512_000, 512)]
)
STD_CONV512 = math.sqrt(2.0 / 4608.0)
STD_CONV256 = math.sqrt(2.0 / 2304.0)


def _layer(name, m, d, k, dist, std, mode, **kw):
    case = {"name": name, "kind": "layer", "m": m, "d": d, "k": k, "dist": dist, "std": std, "mode": mode,
            "soft": 2.0, "tau": 0.0, "tol": 1e-8, "max_iter": 30, "evals": 30, "btol": 1e-6, "bmax": 1000, "passes": 0,
            "assign": False}
    case.update(kw)
    return case


def listed():
    return [
        # One convolution of the 2158-parameter MNIST network, quantised through the autograd layer with the paper's
        # settings (plain norm, tau 5e-4, at most 30 clustering iterations, Jacobian-free gradient): latency is all.
        _layer("mnist_k8_autograd", 1_800, 1, 8, "l2", 0.1, "jfb", kind="autograd", tau=5e-4),
        # A 4096-weight layer at 2 bits, solved to convergence both ways: the smallest full implicit step.
        _layer("tiny_k4_implicit", 4_096, 1, 4, "sql2", 0.05, "implicit", tau=1e-3, tol=1e-6, max_iter=100, evals=37,
               passes=80),
        # A ternary classifier layer (512 x 1000, three codewords): a codebook whose size is not a power of two.
        _layer("fc_k3_implicit", 512_000, 1, 3, "sql2", math.sqrt(2.0 / 512.0), "implicit", tol=1e-7, max_iter=200, evals=35,
               passes=60),
        # 3 bits per weight, the best row of the paper's ResNet18 table, on a ragged layer; Krylov solve of the gradient.
        _layer("ragged_k8_gmres", 300_007, 1, 8, "l2", STD_CONV256, "gmres", soft=0.5, max_iter=60, evals=60, bmax=100, passes=9),
        # The headline workload: 3x3x512x512 convolution at 2 bits per weight, forward and implicit backward to convergence.
        _layer("conv512_k4_implicit", 2_359_296, 1, 4, "sql2", STD_CONV512, "implicit", tau=5e-5, tol=1e-7, max_iter=500,
               evals=37, passes=104),
        # The largest codebook of the paper's ResNet18 table (k = 16, d = 4), plain norm as in the paper, JFB, with codes.
        _layer("conv512_k16d4_jfb", 589_824, 4, 16, "l2", STD_CONV512, "jfb", tau=2e-4, assign=True),
        # Product quantisation with 8-bit codes of 4-vectors, a few passes of the averaged iteration.
        _layer("conv512_k256d4_implicit", 589_824, 4, 256, "sql2", STD_CONV512, "implicit", tau=2e-4, bmax=10, passes=10),
        # 6-bit scalar quantisation: 64 levels for single weights.
        _layer("conv256_k64_jfb", 589_824, 1, 64, "sql2", STD_CONV256, "jfb", soft=4.0),
        # One bit per weight with long vectors: 8-vectors under 8-bit codes.
        _layer("conv512_k256d8_jfb", 294_912, 8, 256, "sql2", STD_CONV512, "jfb", max_iter=20, evals=20),
        # A 4096 x 4096 linear layer, more weights than the chip's on-chip memory holds.
        _layer("linear4096_k4_implicit", 16_777_216, 1, 4, "sql2", math.sqrt(2.0 / 4096.0), "implicit", tol=1e-7,
               max_iter=30, evals=24, btol=1e-5, bmax=40, passes=40),
        # A training step's clustering of a whole ResNet18 at 2 bits: all 21 tensors in one batched call each way.
        {"name": "resnet18_k4_batch", "kind": "batch", "layers": 21, "d": 1, "k": 4, "dist": "sql2", "mode": "implicit",
         "soft": 1.84, "tol": 1e-8, "max_iter": 30, "evals": 30, "btol": 1e-6, "bmax": 300, "passes": 70},
        # The stored form: codes of a 4096 x 4096 layer at 4 bits packed, then unpacked to the quantised weights.
        {"name": "codes_k16_4096", "kind": "codes", "m": 16_777_216, "d": 1, "k": 16},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["scalar", "scalar", "vector", "vector", "large", "large", "large", "autograd", "batch", "codes"])
    dist = rng.choice(["l2", "sql2"])
    soft = math.exp(rng.uniform(0.0, math.log(4.0))) * (1.0 if dist == "sql2" else 0.125)
    std = math.sqrt(2.0 / _log(rng, 64, 4608))
    if kind == "codes":
        k, d = rng.choice([2, 3, 4, 8, 16, 32, 100, 256]), rng.choice([1, 1, 2, 4, 8])
        return {"kind": "codes", "m": _log(rng, 4_000, 16_000_000 // d), "d": d, "k": k}
    if kind == "batch":
        return {"kind": "batch", "layers": rng.randint(2, 21), "d": 1, "k": rng.choice([2, 4, 8]), "dist": dist,
                "mode": rng.choice(["implicit", "jfb"]), "soft": soft, "tol": 1e-8, "max_iter": 30, "evals": 30,
                "btol": 1e-5, "bmax": 30, "passes": 30}
    if kind == "autograd":
        k, d = rng.choice([2, 4, 8]), rng.choice([1, 2])
        case = _layer("", _log(rng, 600, 300_000), d, k, dist, std, rng.choice(["implicit", "jfb"]), kind="autograd", soft=soft)
    elif kind == "scalar":
        k = rng.choice([2, 3, 4, 5, 7, 8, 12, 16])
        case = _layer("", _log(rng, 1_000, 16_000_000 // k), 1, k, dist, std,
                      rng.choice(["implicit", "jfb", "gmres"] if k <= 4 else ["implicit", "jfb"]), soft=soft)
    elif kind == "vector":
        k, d = rng.choice([2, 3, 4, 6, 8, 12, 16]), rng.choice([2, 4])
        case = _layer("", _log(rng, 1_000, 600_000), d, k, dist, std, rng.choice(["implicit", "jfb"]), soft=soft)
    else:
        d = rng.choice([1, 2, 4, 8])
        k = rng.choice([24, 32, 48, 64] if d == 1 else [24, 32, 64, 100, 128] if d == 2 else [24, 32, 64, 100, 128, 200, 256])
        case = _layer("", _log(rng, 2_000, 150_000 if d == 8 else 300_000), d, k, dist, std, rng.choice(["implicit", "jfb"]), soft=soft,
                      max_iter=20, evals=20)
    case.pop("name")
    case["assign"] = rng.choice([False, True]) and case["kind"] == "layer"
    if case["mode"] == "implicit":
        case.update(btol=1e-5, bmax=10, passes=10)
    elif case["mode"] == "gmres":
        case.update(max_iter=60, evals=60, bmax=100, passes=case["k"] + 1)
    return case


# ------------------------------------------------------------------------------------------------ inputs

def _tau(case, std):
    if case.get("tau"):
        return case["tau"]
    spacing = std * case["k"] ** (-1.0 / case["d"])
    return case["soft"] * (spacing * spacing if case["dist"] == "sql2" else spacing)


def _inputs(m, d, k, std, seed):
    """Weights, initial codebook (quantiles of scalar weights, distinct rows of vectors) and upstream gradient."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    W = torch.randn((m, d), generator=gen, device="cuda") * std
    if d == 1:
        pos = ((torch.arange(k, dtype=torch.float64) + 0.5) / k * (m - 1)).round().long().cuda()
        C0 = torch.sort(W[:, 0]).values[pos].reshape(k, 1).contiguous()
    else:
        C0 = W[torch.randperm(m, generator=gen, device="cuda")[:k]].clone()
    G = torch.randn((m, d), generator=gen, device="cuda") * 1e-4
    return W, C0, G


def _batch_inputs(case, seed):
    out = []
    for i, (m, fan_in) in enumerate(RESNET18[:case["layers"]]):
        std = math.sqrt(2.0 / fan_in)
        out.append(_inputs(m, 1, case["k"], std, seed * 100 + i) + (_tau(case, std),))
    return out


def _code_inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    codes = torch.randint(0, case["k"], (case["m"],), generator=gen, device="cuda", dtype=torch.int32)
    C = torch.randn((case["k"], case["d"]), generator=gen, device="cuda") * 0.03
    return codes, C


def prepare(case, seed):
    if case["kind"] == "codes":
        codes, C = _code_inputs(case, seed)
        return {"case": case, "codes": codes, "C": C, "ctx": binding.Context(0)}
    if case["kind"] == "batch":
        layers = _batch_inputs(case, seed)
        return {"case": case, "layers": [(W, C0) for W, C0, _, _ in layers], "G": [G for _, _, G, _ in layers],
                "tau": [t for _, _, _, t in layers], "batch": binding.Batch(len(layers))}
    W, C0, G = _inputs(case["m"], case["d"], case["k"], case["std"], seed)
    state = {"case": case, "W": W, "C0": C0, "G": G, "tau": _tau(case, case["std"])}
    if case["kind"] == "autograd":
        state["W"] = W.requires_grad_()
        state["layer"] = autograd.SoftKMeansQuantize(state["tau"], DISTS[case["dist"]], tol=case["tol"],
                                                     max_iter=case["max_iter"], bwd_mode=MODES[case["mode"]],
                                                     bwd_tol=case["btol"], bwd_max_iter=case["bmax"])
        return state
    # a training loop keeps the context and the output buffers of a layer
    state["ctx"] = binding.Context(0)
    state["out"] = {"C": torch.empty_like(C0), "Wq": torch.empty_like(W),
                    "assign": torch.empty(case["m"], dtype=torch.int32, device="cuda")}
    state["dW"] = torch.empty_like(W)
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "codes":
        words = state["ctx"].pack_codes(state["codes"], case["k"])
        return {"words": words, "Wh": state["ctx"].unpack_quantize(words, case["m"], state["C"])}
    dist, mode = DISTS[case["dist"]], MODES[case["mode"]]
    if case["kind"] == "batch":
        f = state["batch"].forward(state["layers"], state["tau"], case["tol"], case["max_iter"], dist)
        b = state["batch"].backward(state["G"], mode, tol=case["btol"], max_iter=case["bmax"])
        return {"C": [x["C"] for x in f], "Wq": [x["Wq"] for x in f], "dW": [x["dW"] for x in b]}
    if case["kind"] == "autograd":
        state["W"].grad = None
        Wq, C = state["layer"](state["W"], state["C0"])
        Wq.backward(state["G"])
        return {"C": C, "Wq": Wq.detach(), "dW": state["W"].grad}
    f = state["ctx"].forward(state["W"], state["C0"], state["tau"], case["tol"], case["max_iter"], dist,
                             want_assign=case["assign"], out=state["out"])
    b = state["ctx"].backward(state["G"], mode, tol=case["btol"], max_iter=case["bmax"], out=state["dW"])
    res = {"C": f["C"], "Wq": f["Wq"], "dW": b["dW"]}
    if case["assign"]:
        res["assign"] = f["assign"]
    return res


# ------------------------------------------------------------------------------------------------ work and tolerances

def work(case):
    """Operations of one evaluation per (weight vector, codeword): difference and square (3 d), scale, exponential, row sum,
    sums n_j and s_j (2 d + 2).  A backward pass repeats the E-step and adds two inner products and a sum of d terms.
    Bytes: weights and upstream gradient read once, quantised weights and gradient written once."""
    if case["kind"] == "codes":
        bits = max(1, (case["k"] - 1).bit_length())
        return {"bytes": case["m"] * (4 + 2 * bits / 8 + 4 * case["d"]), "flops": case["m"] * bits}
    d, k = case["d"], case["k"]
    m = sum(n for n, _ in RESNET18[:case["layers"]]) if case["kind"] == "batch" else case["m"]
    evals, passes = case["evals"] + 1, (case["passes"] if case["mode"] != "jfb" else 0) + 2
    return {"bytes": m * (16 * d + (4 if case.get("assign") else 0)),
            "flops": m * k * (evals * (5 * d + 5) + passes * (9 * d + 6))}


def tolerance(case):
    """About four times the differences from the 64-bit reference seen over the listed and sixty drawn cases.  The
    gradient of scalar weights under many codewords is the worst conditioned output: its rows carry (w - c) / tau at a
    codebook that 32-bit sums fix to about 1e-6.  With the plain norm a row whose weight lies on a codeword may change
    sign, so single values may be off.  Codes of weights midway between two codewords may differ."""
    if case["kind"] == "codes":
        return "exact"
    rel = 1e-3 if case["d"] == 1 and case["k"] > 16 else 2e-4
    return {"rel": rel, "max": 0.5 if case["dist"] == "l2" else 40 * rel, "differ": 1e-4}


# ------------------------------------------------------------------------------------------------ 64-bit reference

CHUNK = 1 << 24


def _chunks(m, k):
    step = max(1, CHUNK // k)
    return [(i, min(m, i + step)) for i in range(0, m, step)]


def _attention(W, C, tau, dist):
    """(rows of the softmax, energies) in 64 bits."""
    E = torch.zeros((W.shape[0], C.shape[0]), dtype=torch.float64, device=W.device)
    for r in range(W.shape[1]):
        E += (W[:, r, None] - C[None, :, r]) ** 2
    if dist == "l2":
        E = E.sqrt()
    return torch.softmax(E * (-1.0 / tau), dim=1), E


def _mstep(W, C, tau, dist):
    n = torch.zeros(C.shape[0], dtype=torch.float64, device=W.device)
    s = torch.zeros_like(C)
    for i, j in _chunks(*[W.shape[0], C.shape[0]]):
        A, _ = _attention(W[i:j], C, tau, dist)
        n += A.sum(0)
        s += A.t().contiguous() @ W[i:j]
    ok = n > 0
    return torch.where(ok[:, None], s / torch.where(ok, n, torch.ones_like(n))[:, None], C), n


def _delta_sum(th, W, C, E, dist, over_rows):
    """Sum over rows (or over codewords) of th_ij d e_ij / d w_i."""
    out = torch.empty_like(C) if over_rows else torch.empty_like(W)
    for r in range(W.shape[1]):
        t = W[:, r, None] - C[None, :, r]
        dl = 2.0 * t if dist == "sql2" else torch.where(E > 0, t / torch.where(E > 0, E, torch.ones_like(E)), torch.zeros_like(t))
        out[:, r] = (th * dl).sum(0 if over_rows else 1)
    return out


def _solve(W, C0, G, tau, case):
    dist = case["dist"]
    W, C, G = W.double(), C0.double(), G.double()
    for _ in range(case["max_iter"]):
        Cp, _ = _mstep(W, C, tau, dist)
        res = float((Cp - C).norm())
        C = Cp
        if res < case["tol"]:
            break
    F, n = _mstep(W, C, tau, dist)
    chunks = _chunks(W.shape[0], C.shape[0])
    Wq, v = torch.empty_like(W), torch.zeros_like(C)
    for i, j in chunks:
        A, E = _attention(W[i:j], C, tau, dist)
        Wq[i:j] = A @ C
        p = G[i:j] @ C.t().contiguous()
        rho = A * (p - (A * p).sum(1, keepdim=True))
        v += A.t().contiguous() @ G[i:j] + _delta_sum(rho, W[i:j], C, E, dist, True) / tau

    def h_of(g):
        return torch.where(n[:, None] > 0, g / torch.where(n > 0, n, torch.ones_like(n))[:, None], torch.zeros_like(g))

    def gamma(A, h, w):
        b = w @ h.t().contiguous() - (h * F).sum(1)[None, :]
        return A * (b - (A * b).sum(1, keepdim=True))

    def jct(g):
        out, h = torch.zeros_like(C), h_of(g)
        for i, j in chunks:
            A, E = _attention(W[i:j], C, tau, dist)
            out += _delta_sum(gamma(A, h, W[i:j]), W[i:j], C, E, dist, True) / tau
        return out

    g = v
    if case["mode"] == "gmres":
        kd = v.numel()
        eye = torch.eye(kd, dtype=torch.float64, device=W.device)
        J = torch.stack([jct(eye[i].reshape(v.shape)).reshape(-1) for i in range(kd)], 1)
        g = torch.linalg.solve((eye - J).cpu(), v.reshape(-1).cpu()).reshape(v.shape).to(W.device)
    elif case["mode"] == "implicit":
        # undamped first; a step norm that grows five times in a row starts over with half the step
        alpha, vnorm = 1.0, float(v.norm())
        for attempt in range(7):
            g, prev, grow, ok = v, math.inf, 0, True
            for _ in range(case["bmax"]):
                gn = alpha * (v + jct(g)) + (1.0 - alpha) * g
                step = float((gn - g).norm())
                g = gn
                if not step > case["btol"] * vnorm:
                    break
                grow = grow + 1 if step > prev else 0
                if grow >= 5:
                    ok = False
                    break
                prev = step
            if ok:
                break
            alpha *= 0.5
    dW, h = torch.empty_like(W), h_of(g)
    for i, j in chunks:
        A, E = _attention(W[i:j], C, tau, dist)
        p = G[i:j] @ C.t().contiguous()
        th = A * (p - (A * p).sum(1, keepdim=True)) + gamma(A, h, W[i:j])
        dW[i:j] = A @ h - _delta_sum(th, W[i:j], C, E, dist, False) / tau
    return C, Wq, dW


def exact(case, seed):
    if case["kind"] == "codes":
        codes, C = _code_inputs(case, seed)
        return {"words": None, "Wh": C.double()[codes.long()]}
    if case["kind"] == "batch":
        parts = [_solve(W, C0, G, tau, case) for W, C0, G, tau in _batch_inputs(case, seed)]
        return {"C": [p[0] for p in parts], "Wq": [p[1] for p in parts], "dW": [p[2] for p in parts]}
    W, C0, G = _inputs(case["m"], case["d"], case["k"], case["std"], seed)
    C, Wq, dW = _solve(W, C0, G, _tau(case, case["std"]), case)
    res = {"C": C, "Wq": Wq, "dW": dW}
    if case.get("assign"):
        res["assign"] = None
    return res
