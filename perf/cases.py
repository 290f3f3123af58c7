"""Performance cases: the work a program has this library do, through the
Python entry points, over the sizes it is used at.

The four linears of a DiT block (qkv, proj, fc1, fc2) at three block shapes,
single linears at the small and ragged ends, the fp6-stored and 8-bit
settings, the 28-block stack as one graph, the weight quantizer, the OBS
calibration pass and the CLPS clip search.  Inputs follow the library's
synthetic laws: Gaussian activations with a few outlier channels (and, for
law L2, a lognormal scale per token), weights N(0, 1 / K), biases 0.1 N(0, 1).

A linear's run() is what a serving loop calls per layer: the activations are
rotated and quantized, then multiplied with weights quantized once.
"""
import math

import torch

import paper_2509_24416_amd as clq
from paper_2509_24416_amd.stack import DiTStack

# name -> (act quantizer, weight quantizer, linear)
SETTINGS = {
    "w4a4": (clq.clq_rotate_quant_act, clq.clq_quantize_weights, clq.clq_w4a4_linear),
    "f6": (clq.clq_rotate_quant_act_f6, clq.clq_quantize_weights_f6, clq.clq_w4a4_linear_f6),
    "w4a8": (clq.clq_rotate_quant_act8, clq.clq_quantize_weights, clq.clq_a8_linear),
    "w8a8": (clq.clq_rotate_quant_act8, clq.clq_quantize_weights8, clq.clq_a8_linear),
}
QMAX = {"w4a4": (7, 7), "f6": (7, 7), "w4a8": (127, 7), "w8a8": (127, 127)}   # (activations, weights)
GAMMA = 0.01


def listed():
    return [
        # one 256-token linear (a 256-pixel image's tokens): launches and
        # latency count, the arithmetic hardly does
        dict(name="linear_m256", kind="linear", setting="w4a4", M=256, K=1152, N=1152, block=64, perm=False,
             bias=True, law="L1"),
        # token and channel counts that fill no tile, inputs gathered by an
        # OBS swap vector, the smallest Hadamard block
        dict(name="linear_ragged_swap", kind="linear", setting="w4a4", M=777, K=1152, N=1000, block=32, perm=True,
             bias=True, law="L1"),
        # the block linears of a 1024-pixel image transformer, 4096 tokens x
        # guidance batch 2
        dict(name="pixart_block", kind="block", setting="w4a4", M=8192, hidden=1152, mlp=4608, block=64, law="L1"),
        # a width-3072 image transformer: 4096 image + 512 text tokens
        dict(name="flux_block", kind="block", setting="w4a4", M=4608, hidden=3072, mlp=12288, block=128, law="L2"),
        # a video transformer: 16 x 30 x 45 latent patches x guidance batch 2
        dict(name="video_block", kind="block", setting="w4a4", M=43200, hidden=1152, mlp=4608, block=64, law="L1"),
        # the same 4-bit codes stored as fp6, at a 2048-pixel image's 16384 tokens
        dict(name="block_f6", kind="block", setting="f6", M=16384, hidden=1152, mlp=4608, block=64, law="L1"),
        # the two 8-bit-activation settings on the image transformer's block
        dict(name="pixart_block_w4a8", kind="block", setting="w4a8", M=8192, hidden=1152, mlp=4608, block=64,
             law="L1"),
        dict(name="pixart_block_w8a8", kind="block", setting="w8a8", M=8192, hidden=1152, mlp=4608, block=64,
             law="L1"),
        # a whole denoising step's linears at 1024 tokens (a 512-pixel image):
        # 28 blocks replayed as one graph
        dict(name="stack_m1024", kind="stack", codes="int4", blocks=28, M=1024, hidden=1152, mlp=4608, block=64),
        # offline: the weights of a width-3072 block's fc1
        dict(name="quantize_fc1", kind="quantize", setting="w4a4", N=12288, K=3072, block=128, perm=False),
        # offline: channel scores of a calibration batch and the swap they give
        dict(name="obs_absmax", kind="obs", metric="absmax", B=32, N=4096, D=1152),
        # offline: the clip search of one qkv layer on 4096 calibration tokens
        dict(name="clps_qkv", kind="clps", M=4096, K=1152, N=3456, block=64, grid=20, perm=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi, block):
    step = max(64, block)
    return max(step, _log_int(rng, lo, hi) // step * step)


def draw(rng):
    kind = rng.choices(["linear", "block", "stack", "quantize", "obs", "clps"], [10, 5, 1, 2, 2, 2])[0]
    block = rng.choice([32, 64, 64, 128])
    setting = rng.choices(list(SETTINGS), [5, 2, 2, 2])[0]
    if kind == "linear":
        K = max(128, _width(rng, 128, 12288, block))
        N = _log_int(rng, 32, 12288)
        if rng.random() < 0.7:
            N = max(16, N // 16 * 16)
        M = _log_int(rng, 1, 43200)
        while 2.0 * M * N * K > 4e11 or M * (K + N) > 6e8:   # within the largest block's work
            M = max(1, M // 2 + 1)
        return dict(kind=kind, setting=setting, M=M, K=K, N=N, block=block, perm=rng.random() < 0.3,
                    bias=rng.random() < 0.8, law=rng.choice(["L1", "L2"]))
    if kind == "block":
        hidden = _width(rng, 384, 3072, block)
        mlp = 4 * hidden
        M = _log_int(rng, 64, 43200)
        while 24.0 * M * hidden * hidden > 1.3e12:
            M = M // 2 + 1
        return dict(kind=kind, setting=setting, M=M, hidden=hidden, mlp=mlp, block=block,
                    law=rng.choice(["L1", "L2"]))
    if kind == "stack":
        return dict(kind=kind, codes=rng.choice(["int4", "int4", "f6"]), blocks=rng.randint(2, 28),
                    M=_log_int(rng, 64, 2048), hidden=1152, mlp=4608, block=block)
    if kind == "quantize":
        return dict(kind=kind, setting=setting, N=_log_int(rng, 64, 12288),
                    K=max(128, _width(rng, 384, 12288, block)), block=block, perm=rng.random() < 0.5)
    if kind == "obs":
        D = 8 * _log_int(rng, 16, 576)
        N = _log_int(rng, 64, 16384)
        B = rng.randint(1, 32)
        while B * N * D > 1.6e8:
            N = N // 2 + 1
        return dict(kind=kind, metric=rng.choice(["absmax", "absmax", "range", "par", "topk_mean", "percentile"]),
                    B=B, N=N, D=D)
    return dict(kind=kind, M=_log_int(rng, 64, 4096), K=_width(rng, 384, 3072, block),
                N=_log_int(rng, 64, 4608), block=block, grid=rng.randint(2, 20), perm=rng.random() < 0.3)


# ---- inputs ---------------------------------------------------------------------

def _layers(case):
    """[(K, N)] of a block's linears."""
    h, f = case["hidden"], case["mlp"]
    return [(h, 3 * h), (h, h), (h, f), (f, h)]


def _outliers(g, K, law):
    """The per-channel factors of an activation law, fp32 [K]."""
    frac, lo, hi = (0.01, 20.0, 100.0) if law == "L1" else (0.005, 50.0, 200.0)
    n = int(round(frac * K))
    fac = torch.ones(K, device="cuda")
    if n:
        ch = torch.randperm(K, generator=g, device="cuda")[:n]
        u = torch.rand(n, generator=g, device="cuda")
        fac[ch] = torch.exp(math.log(lo) + u * math.log(hi / lo))
    return fac


def _acts(g, M, K, law):
    x = torch.randn((M, K), generator=g, device="cuda") * _outliers(g, K, law)
    if law == "L2":
        x *= torch.exp(0.5 * torch.randn((M, 1), generator=g, device="cuda"))
    return x.half()


def _weight(g, N, K):
    return (torch.randn((N, K), generator=g, device="cuda") / math.sqrt(K)).half()


def _bias(g, N):
    return (0.1 * torch.randn(N, generator=g, device="cuda")).half()


def _swap(g, K):
    return torch.randperm(K, generator=g, device="cuda").int()


def _inputs(case, seed):
    """The unquantized tensors of a case."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    kind = case["kind"]
    if kind == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        return [dict(X=_acts(g, M, K, case["law"]), W=_weight(g, N, K), b=_bias(g, N) if case["bias"] else None,
                     perm=_swap(g, K) if case["perm"] else None)]
    if kind == "block":
        return [dict(X=_acts(g, case["M"], K, case["law"]), W=_weight(g, N, K), b=_bias(g, N), perm=None)
                for K, N in _layers(case)]
    if kind == "stack":
        blocks = [{n: (_weight(g, N, K), _bias(g, N)) for n, (K, N) in zip(("qkv", "proj", "fc1", "fc2"), _layers(case))}
                  for _ in range(case["blocks"])]
        return blocks, _acts(g, case["M"], case["hidden"], "L1")
    if kind == "quantize":
        return dict(W=_weight(g, case["N"], case["K"]), perm=_swap(g, case["K"]) if case["perm"] else None)
    if kind == "obs":
        fac = _outliers(g, case["D"], "L1")
        return torch.stack([(torch.randn((case["N"], case["D"]), generator=g, device="cuda") * fac).half()
                            for _ in range(case["B"])])
    X, W = _acts(g, case["M"], case["K"], "L1"), _weight(g, case["N"], case["K"])
    return dict(X=X, W=W, Y0=X.float() @ W.float().t(), perm=_swap(g, case["K"]) if case["perm"] else None)


def prepare(case, seed):
    inp = _inputs(case, seed)
    kind = case["kind"]
    state = dict(case=case)
    if kind in ("linear", "block"):
        quant = SETTINGS[case["setting"]][1]
        state["layers"] = [(l["X"], quant(l["W"], case["block"], perm=l["perm"]), l["b"], l["perm"]) for l in inp]
    elif kind == "stack":
        weights, x = inp
        stack = DiTStack(weights, case["M"], block=case["block"], codes="fp6" if case["codes"] == "f6" else "int4")
        stack.forward(x)
        stack.capture()
        state.update(stack=stack, x=x)
    elif kind == "quantize":
        state.update(inp)
    elif kind == "obs":
        state["X"] = inp
    else:
        state.update(inp, workspace=torch.empty(clq.clq_clps_workspace_bytes(case["M"], case["N"], case["K"]),
                                                dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    return state


# ---- one pass ---------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("linear", "block"):
        act, _, linear = SETTINGS[case["setting"]]
        out = []
        for X, qw, b, perm in state["layers"]:
            Xq, xs = act(X, case["block"], perm=perm)
            out.append(linear(Xq, xs, qw, b))
        return out
    if kind == "stack":
        return state["stack"].replay(state["x"])
    if kind == "quantize":
        qw = SETTINGS[case["setting"]][1](state["W"], case["block"], perm=state["perm"])
        return qw.wq, qw.w_scale
    if kind == "obs":
        scores = clq.clq_obs_channel_scores(state["X"], case["metric"])
        return scores, clq.clq_obs_permutation(scores)
    return clq.clq_clps_search(state["X"], state["W"], state["Y0"], case["block"], perm=state["perm"], gamma=GAMMA,
                               grid=case["grid"], workspace=state["workspace"])


# ---- what a pass cannot do without ------------------------------------------------

_WEIGHT_BYTES = {"w4a4": 0.5, "f6": 0.75, "w4a8": 0.5, "w8a8": 1.0}


def _linear_work(M, K, N, wb):
    return 2.0 * M * K + wb * N * K + 6.0 * N + 2.0 * M * N, 2.0 * M * N * K


def work(case):
    kind = case["kind"]
    if kind == "linear":
        b, f = _linear_work(case["M"], case["K"], case["N"], _WEIGHT_BYTES[case["setting"]])
    elif kind == "block":
        ws = [_linear_work(case["M"], K, N, _WEIGHT_BYTES[case["setting"]]) for K, N in _layers(case)]
        b, f = sum(w[0] for w in ws), sum(w[1] for w in ws)
    elif kind == "stack":   # the weights, the input and the output; activations between layers could stay on chip
        wb = 0.75 if case["codes"] == "f6" else 0.5
        per = sum(K * N for K, N in _layers(case))
        b = case["blocks"] * per * wb + 4.0 * case["M"] * case["hidden"]
        f = 2.0 * case["blocks"] * case["M"] * per
    elif kind == "quantize":
        N, K = case["N"], case["K"]
        b, f = N * K * (2.0 + _WEIGHT_BYTES[case["setting"]]) + 4.0 * N, N * K * (math.log2(case["block"]) + 2.0)
    elif kind == "obs":
        n = float(case["B"] * case["N"] * case["D"])
        b, f = 2.0 * n + 8.0 * case["D"], n
    else:
        M, K, N, G = case["M"], case["K"], case["N"], case["grid"]
        b, f = 2.0 * M * K + 2.0 * N * K + 4.0 * M * N, 2.0 * M * N * K * G
    return {"bytes": b, "flops": f}


def tolerance(case):
    kind = case["kind"]
    if kind in ("linear", "block"):
        # the integer sums are exact and the fp16 outputs carry one rounding
        # (2.1e-4 measured against 64 bits); codes next to a rounding boundary
        # that fall the other way in 64 bits raise that to 1.1e-3
        return {"rel": 4e-3}
    if kind == "stack":
        # every layer's codes follow from the previous layer's fp16 bits, and a
        # code that flips changes all later layers: two runs agree to the bit
        # or not at all.  The library gives the same fp16 bits on every
        # schedule and code storage.
        return "exact"
    if kind == "quantize":
        # codes next to a rounding boundary may fall either way when the
        # rotation's fp32 sums are taken in another order
        return {"rel": 1e-6, "differ": 1e-5}
    if kind == "obs":
        # 32-bit means and maxima (2e-9 measured against 64 bits for abs-max)
        return {"rel": 1e-6, "differ": 0.0}
    # errors of up to 5.4e-6 against 64 bits: a few codes next to a boundary
    return {"rel": 2e-5, "differ": 0.0}


# ---- the same results in 64 bits ------------------------------------------------------

def _hadamard(b):
    h = torch.ones((1, 1), dtype=torch.float64, device="cuda")
    while h.shape[0] < b:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)], 0)
    return h


def _rotate(X, block, perm):
    x = X if perm is None else X.index_select(1, perm.long())
    return (x.double().reshape(-1, block) @ _hadamard(block)).reshape(X.shape)


def _codes(xr, qmax, alpha=1.0):
    """(codes, scale per row) of rotated rows."""
    a = alpha * xr.abs().amax(1, keepdim=True)
    s = a / qmax
    q = torch.where(a > 0, torch.round(xr / torch.where(a > 0, s, 1.0)), 0.0)
    return q.clamp(-qmax, qmax), s


def _exact_clps(case, seed):
    l = _inputs(case, seed)
    K, G, b = case["K"], case["grid"], case["block"]
    wr = _rotate(l["W"], b, l["perm"])
    qx, xs = _codes(_rotate(l["X"], b, l["perm"]), 7)
    mag = wr.abs().sort(1).values
    top = mag[:, -1]
    ratio = torch.where(top > 0, mag[:, K - 1 - int(GAMMA * (K - 1))] / torch.where(top > 0, top, 1.0), 1.0)
    lo = min(1.0, ratio.min().item())
    alphas = [1.0 - (1.0 - lo) * (G - 1 - i) / (G - 1) for i in range(G)]
    errors = []
    for al in alphas:
        qw, ws = _codes(wr, 7, al)
        errors.append(((l["Y0"].double() - (qx @ qw.t()) * xs * (ws / b).t()) ** 2).sum().item())
    return (torch.tensor(alphas, dtype=torch.float64), torch.tensor(errors, dtype=torch.float64),
            torch.tensor([min(range(G), key=lambda i: errors[i])], dtype=torch.int32))


def exact(case, seed):
    kind = case["kind"]
    if kind in ("linear", "block"):
        xmax, wmax = QMAX[case["setting"]]
        out = []
        for l in _inputs(case, seed):
            qx, xs = _codes(_rotate(l["X"], case["block"], l["perm"]), xmax)
            qw, ws = _codes(_rotate(l["W"], case["block"], l["perm"]), wmax)
            y = (qx @ qw.t()) * xs * (ws / case["block"]).t()
            out.append(y if l["b"] is None else y + l["b"].double())
        return out
    if kind == "stack":
        return None   # see tolerance()
    if kind == "quantize":
        l = _inputs(case, seed)
        _, ws = _codes(_rotate(l["W"], case["block"], l["perm"]), QMAX[case["setting"]][1])
        return None, (ws / case["block"]).reshape(-1)   # the codes' layout is opaque
    if kind == "obs":
        s = _inputs(case, seed).double().mean(0)
        N = s.shape[0]
        m = case["metric"]
        if m == "absmax":
            v = s.abs().amax(0)
        elif m == "range":
            v = s.amax(0) - s.amin(0)
        elif m == "par":
            v = s.abs().amax(0) / s.abs().mean(0)
        elif m == "topk_mean":
            v = s.abs().topk(max(1, (N + 50) // 100), 0).values.mean(0)
        else:
            o, l = s.sort(0).values, (N - 1) // 100
            v = o[N - 1 - l] - o[l]
        return v, None   # channels next to the median may swap halves
    return _exact_clps(case, seed)
