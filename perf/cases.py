"""The work that programs have this library do, as cases that can be timed and compared.

A case is one pass of the expert-choice layer through the public entry points: a forward pass (serving, prefill), the
same with one of the routing variants, the stages called one by one as an expert-parallel program calls them around
its exchanges, or a training step's forward and backward.  Sizes are the library's own workloads (workloads.py) and
generic ragged ones between them.  Inputs are drawn on the GPU with the distributions of workloads.py: unit normal
tokens and output gradients, weights scaled by 1/sqrt(fan-in), for long routing batches one per cent of the tokens
ten times larger.

Keys of a case: kind (forward, grouped, token_choice, capped, stages, train), n tokens, d width, e experts, c capacity
factor, d_ff hidden width (0: identity experts), act (relu, gelu, identity), dtype (f32, bf16, hilo = bf16 tensors
with two-part matrix-core operands); groups / m / b, lam, iters belong to the variant that has them.
"""
import math

import torch

import paper_2202_09368_amd as m

ACT = {"relu": m.EC_ACT_RELU, "gelu": m.EC_ACT_GELU, "identity": m.EC_ACT_IDENTITY}


def _case(kind, n, d, e, c, d_ff, act="gelu", dtype="bf16", **more):
    return dict(kind=kind, n=n, d=d, e=e, c=c, d_ff=d_ff, act=act, dtype=dtype, **more)


def listed():
    cases = {
        # the smallest layer in use: fp32, a handful of microseconds of work, launches and latency are what counts
        "tiny_f32": _case("forward", 256, 64, 8, 2.0, 256, act="relu", dtype="f32"),
        # one decode step of a batch of sequences routed inside their groups: few tokens, all of the weights
        "decode_grouped": _case("grouped", 256, 768, 16, 2.0, 3072, groups=4),
        # prefill of the 16-expert layer (8 x 1024 tokens)
        "prefill_16e": _case("forward", 8192, 768, 16, 2.0, 3072),
        # a batch and widths that no tile divides: odd token count, rows of 8-element multiples
        "forward_ragged": _case("forward", 3001, 520, 12, 1.25, 1368),
        # the 64-expert layer stage by stage, as expert-parallel programs run it, in the precise bf16 mode
        "stages_64e_hilo": _case("stages", 16384, 1024, 64, 2.0, 4096, dtype="hilo"),
        # the conventional top-2 baseline at the same cost as prefill_16e
        "token_choice_16e": _case("token_choice", 8192, 768, 16, 2.0, 3072, m=2),
        # at most two experts per token, the method's own 100 iterations
        "capped_16e": _case("capped", 8192, 768, 16, 2.0, 3072, b=2.0, lam=0.001, iters=100),
        # routing and data movement alone: long batch, many experts, identity experts
        "route_256e": _case("forward", 65536, 4096, 256, 1.0, 0, act="identity"),
        # training steps: the 16-expert layer, the largest single-GPU layer in the precise mode, a ragged one, fp32
        "train_16e": _case("train", 8192, 768, 16, 2.0, 3072),
        "train_128e_hilo": _case("train", 32768, 2048, 128, 2.0, 8192, dtype="hilo"),
        "train_ragged": _case("train", 5003, 704, 20, 1.5, 1856),
        "train_f32": _case("train", 2048, 512, 8, 2.0, 2048, dtype="f32"),
    }
    return [dict(case, name=name) for name, case in cases.items()]


def _bucket(case):
    """Rows of an expert's bucket."""
    groups = case.get("groups", 1)
    return groups * math.floor((case["n"] // groups) * case["c"] / case["e"])


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choices(["forward", "grouped", "token_choice", "capped", "stages", "route", "train"],
                       [24, 10, 10, 8, 10, 8, 30])[0]
    dtype = rng.choices(["bf16", "hilo", "f32"], [60, 25, 15])[0]
    n, e = _log_int(rng, 64, 32768), _log_int(rng, 4, 128)
    if rng.random() < 0.5:
        n = max(64, n // 64 * 64)
    if rng.random() < 0.5:
        e = max(8, e // 8 * 8)
    c = rng.choice([1.0, 1.25, 1.5, 2.0])
    step = 8 if dtype != "hilo" and rng.random() < 0.2 else 64  # most layers are multiples of 64 wide
    d = _log_int(rng, 64, 2048) // step * step
    d_ff = max(step, int(d * rng.choice([2.0, 2.67, 4.0])) // step * step)
    # fp32 training differentiates GeLU only: ReLU's derivative jumps at 0, where fp32 rounding decides the side
    act = "gelu" if (kind, dtype) == ("train", "f32") else rng.choice(["gelu", "gelu", "gelu", "relu"])
    if kind == "route":
        return _case("forward", _log_int(rng, 2048, 65536) // 4 * 4, _log_int(rng, 512, 4096) // 64 * 64,
                     rng.choice([32, 64, 128, 192, 256]), rng.choice([1.0, 2.0]), 0, act="identity")
    case = _case(kind, n, d, e, c, d_ff, act=act, dtype=dtype)
    if kind == "grouped":
        case["groups"] = rng.choice([2, 4, 8, 16, 32])
        case["n"] = max(64, n // (4 * case["groups"]) * (4 * case["groups"]))
    elif kind == "token_choice":
        case["m"] = rng.choice([1, 2])
    elif kind == "capped":
        case.update(b=float(rng.choice([2, 3])), lam=0.001, iters=rng.choice([20, 50, 100]))
    return case


def _affordable(case):
    """Inside the ranges above, and no dearer than the largest listed case on any path."""
    if case["n"] * case["c"] / case["e"] / case.get("groups", 1) < 4 or _bucket(case) > case["n"]:
        return False
    if case["kind"] == "capped" and case["n"] * case["e"] > 1 << 20:
        return False
    if case["dtype"] == "f32" or case["d"] % 64 or case["d_ff"] % 64:
        return _flops(case) <= 6e10
    return _flops(case) <= 6e12 and case["e"] * case["d"] * case["d_ff"] <= 1 << 30


def draw(rng):
    while True:
        case = _draw_once(rng)
        if _affordable(case):
            return case


# ------------------------------------------------------------------------------------------------------ one pass --
def prepare(case, seed):
    """Inputs, weights, workspace and the buffers that a program keeps for the results."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    n, d, e, d_ff, kind = case["n"], case["d"], case["e"], case["d_ff"], case["kind"]
    k = _bucket(case)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    code = {"f32": m.EC_F32, "bf16": m.EC_BF16, "hilo": m.EC_BF16_HILO}[case["dtype"]]
    train = kind == "train"

    def normal(*shape, std=1.0):
        out = torch.empty(shape, dtype=dt, device="cuda")
        flat = out.view(-1)
        for at in range(0, flat.numel(), 1 << 28):  # drawn in fp32, stored in the layer's type
            part = flat[at:at + (1 << 28)]
            part.copy_(torch.randn(part.numel(), generator=gen, device="cuda").mul_(std))
        return out

    def empty(*shape, dtype=dt):
        return torch.empty(shape, dtype=dtype, device="cuda")

    s = dict(case=case, k=k, act=ACT[case["act"]], hilo=case["dtype"] == "hilo")
    s["X"] = normal(n, d)
    if d_ff == 0:  # heavy competition for a few experts, near one-hot scores
        s["X"][torch.randperm(n, generator=gen, device="cuda")[:n // 100]] *= 10
    s["Wg"] = normal(d, e, std=d ** -0.5)
    s["W1"] = normal(e, d, d_ff, std=d ** -0.5) if d_ff else None
    s["W2"] = normal(e, d_ff, d, std=d_ff ** -0.5) if d_ff else None
    s["Xout"] = empty(n, d)
    ws = m.ec_moe_workspace_bytes(n, d, e, k, d_ff, code, train)
    if kind == "capped":
        ws += m.ec_moe_capped_workspace_bytes(n, e) + (4 * e * n + 255) // 256 * 256
    s["ws"] = torch.empty(ws, dtype=torch.uint8, device="cuda")
    if kind in ("stages", "train"):
        s["G"], s["I"] = empty(e, k, dtype=torch.float32), empty(e, k, dtype=torch.int32)
        s["Xin"], s["Xe"] = empty(e, k, d), empty(e, k, d)
    if kind == "stages":
        s["St"] = empty(e, n, dtype=torch.float32)
    if train:
        s["S"] = empty(n, e, dtype=torch.float32)
        s["A"], s["H"] = empty(e, k, d_ff), empty(e, k, d_ff)
        s["dY"], s["dX"] = normal(n, d), empty(n, d)
        s["dWg"] = empty(d, e, dtype=torch.float32)
        s["dW1"], s["dW2"] = empty(e, d, d_ff, dtype=torch.float32), empty(e, d_ff, d, dtype=torch.float32)
    return s


def run(s):
    case, act, hilo, ws = s["case"], s["act"], s["hilo"], s["ws"]
    kind, c = case["kind"], case["c"]
    layer = (s["X"], s["Wg"], s["W1"], s["W2"], c)
    if kind == "forward":
        m.ec_moe_forward(*layer, s["Xout"], act, ws, hilo=hilo)
    elif kind == "grouped":
        m.ec_moe_forward_grouped(*layer, case["groups"], s["Xout"], act, ws, hilo=hilo)
    elif kind == "token_choice":
        m.ec_moe_forward_token_choice(*layer, case["m"], s["Xout"], act, ws, hilo=hilo)
    elif kind == "capped":
        m.ec_moe_forward_capped(*layer, case["b"], case["lam"], case["iters"], s["Xout"], act, ws, hilo=hilo)
    elif kind == "stages":
        m.ec_moe_gate(s["X"], s["Wg"], None, s["St"], ws)
        m.ec_moe_topk_tokens(s["St"], s["k"], s["G"], s["I"], ws)
        m.ec_moe_dispatch(s["X"], s["I"], s["Xin"])
        m.ec_moe_expert_ffn(s["Xin"], s["W1"], s["W2"], s["Xe"], act, ws, hilo=hilo)
        m.ec_moe_combine(s["Xe"], s["G"], s["I"], s["Xout"], ws)
    else:
        m.ec_moe_forward(*layer, s["Xout"], act, ws, S_out=s["S"], G_out=s["G"], I_out=s["I"], Xin_out=s["Xin"],
                         A_out=s["A"], H_out=s["H"], Xe_out=s["Xe"], hilo=hilo)
        m.ec_moe_backward(s["dY"], s["X"], s["Wg"], s["W1"], s["W2"], s["S"], s["G"], s["I"], s["Xin"], s["A"], s["H"],
                          s["Xe"], s["dX"], s["dWg"], s["dW1"], s["dW2"], act, ws, hilo=hilo)
        return {key: s[key] for key in ("Xout", "dX", "dWg", "dW1", "dW2")}
    return {"Xout": s["Xout"]}


# ---------------------------------------------------------------------------------------------- what a pass needs --
def _flops(case):
    n, d, e, d_ff = case["n"], case["d"], case["e"], case["d_ff"]
    forward = 2 * n * d * e + 4 * e * _bucket(case) * d * d_ff
    return 3 * forward if case["kind"] == "train" else forward


def work(case):
    n, d, e, d_ff = case["n"], case["d"], case["e"], case["d_ff"]
    size = 4 if case["dtype"] == "f32" else 2
    weights = d * e + 2 * e * d * d_ff
    if case["kind"] == "train":  # X, dY, weights in; X_out, dX and the fp32 weight gradients out
        moved = 4 * n * d * size + weights * (size + 4)
    else:
        moved = 2 * n * d * size + weights * size
    return {"bytes": moved, "flops": _flops(case)}


def tolerance(case):
    """2-norm errors as the storage types give them.  The largest single difference is wider: scores that agree to
    fp32 rounding only may order two tokens at an expert's threshold differently, which moves those tokens' rows."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 1e-2, "max": 0.9}
