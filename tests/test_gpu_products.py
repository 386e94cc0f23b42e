"""Layer products at the edges of their tiles: whole layers, forward and backward, against the oracle, at sizes that
select each tile form and leave remainders in every dimension.  The bars are those of the fixed-shape tests: 1e-5 for
fp32 (a length-k fp32 sum is good to k * 2^-24 of its terms), 2e-2 for bf16 tensors."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_util import max_rel_err_rows, score_tolerance, sized, to_dev, to_host
from test_gpu_backward import m, ref, test_backward_reduced as check_backward  # noqa: F401 (fixtures)
from test_gpu_parity import _stagewise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(n=37, d=33, e=3, c=1.0, d_ff=31),                # scalar loads, one K stage and a remainder, 12-row buckets
    dict(n=260, d=68, e=4, c=2.0, d_ff=132),              # 16-byte loads, K-sharing tiles with remainders, k = 130
    dict(n=2048, d=96, e=4, c=2.0, d_ff=1540),            # 128 x 128 tiles, remainder columns
    dict(n=1300, d=130, e=16, c=2.0, d_ff=258),           # 64 x 64 tiles, scalar loads, short last split of tokens
])
def test_fp32_products(m, ref, kw):  # noqa: F811
    check_backward(m, ref, "cfg1", dict(kw, act=wl.ACT_GELU), 1e-5)


@pytest.mark.parametrize("kw", [
    dict(n=513, d=72, e=3, c=1.0, d_ff=8),                # K one stage and 8; K = 8 alone
    dict(n=640, d=136, e=5, c=2.0, d_ff=264),             # gathered rows, K remainders of 8
    dict(n=4100, d=520, e=12, c=2.0, d_ff=1000),          # 256-wide tiles, remainder 40
])
def test_bf16_ragged_widths(m, ref, kw):  # noqa: F811
    w = sized(wl.WORKLOADS["cfg2"], **kw)
    _stagewise(m, ref, w, wl.make_inputs(w))


@pytest.mark.parametrize("e,k,d,d_ff", [(2, 70, 8, 8), (3, 300, 136, 72), (2, 520, 520, 200), (16, 512, 520, 3080)])
def test_bf16_ragged_widths_keep_rows_apart(m, e, k, d, d_ff):  # noqa: F811
    """A row that holds infinities and NaN leaves the rows beside it what they are without it, bit for bit: the last
    stage of a contraction that 64 does not divide must not multiply the next row's elements, even by zeros."""
    gen = torch.Generator(device="cuda").manual_seed(e * k + d)
    Xin = torch.randn(e, k, d, generator=gen, device="cuda").bfloat16()
    W1 = (torch.randn(e, d, d_ff, generator=gen, device="cuda") * d ** -0.5).bfloat16()
    W2 = (torch.randn(e, d_ff, d, generator=gen, device="cuda") * d_ff ** -0.5).bfloat16()
    ws = m.alloc_workspace(e * k, d, e, k, d_ff, m.EC_BF16)
    clean, marked = torch.empty_like(Xin), torch.empty_like(Xin)
    m.ec_moe_expert_ffn(Xin, W1, W2, clean, m.EC_ACT_IDENTITY, ws)
    rows = [1, k // 2, k - 1]
    Xin[:, rows] = torch.tensor([float("inf"), float("-inf"), float("nan")], device="cuda").bfloat16()[:, None]
    m.ec_moe_expert_ffn(Xin, W1, W2, marked, m.EC_ACT_IDENTITY, ws)
    keep = torch.ones(k, dtype=torch.bool, device="cuda")
    keep[rows] = False
    assert torch.isfinite(clean).all()
    assert torch.equal(clean[:, keep], marked[:, keep])
    assert torch.isnan(marked[:, k - 1]).all()


@pytest.mark.parametrize("dtype,n,d,e", [
    ("bf16", 33, 8, 1), ("bf16", 95, 136, 7), ("bf16", 1000, 704, 20), ("bf16", 257, 200, 40), ("bf16", 100, 129, 100),
    ("bf16", 70, 320, 250), ("bf16", 64, 64, 256), ("f32", 31, 5, 3), ("f32", 1000, 260, 33), ("f32", 130, 96, 64),
    ("f32", 65, 100, 128), ("f32", 40, 67, 255),
])
def test_gate_edges(m, ref, dtype, n, d, e):  # noqa: F811
    """Every expert-tile count, vector and scalar rows, remainders in tokens, width and experts; S and S^T agree."""
    rng = np.random.default_rng(n * d + e)
    X, Wg = rng.standard_normal((n, d), dtype=np.float32), rng.standard_normal((d, e), dtype=np.float32) * d ** -0.5
    if dtype == "bf16":
        X, Wg = wl.f32_to_bf16_bits(X), wl.f32_to_bf16_bits(Wg)
    S = torch.full((n, e), float("nan"), dtype=torch.float32, device="cuda")
    St = torch.full((e, n), float("nan"), dtype=torch.float32, device="cuda")
    m.ec_moe_gate(to_dev(X), to_dev(Wg), S, St, None)
    torch.cuda.synchronize()
    S_h = to_host(S)
    assert (max_rel_err_rows(S_h, ref.gate(X, Wg)) <= score_tolerance(X, Wg)).all()
    assert (to_host(St) == S_h.T).all()
