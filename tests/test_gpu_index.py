"""The selection at the edges of its kernels and the token-major index behind it, against the oracle: rows whose length is
no multiple of four, tokens that more experts chose than a row has lanes, and static scratch too small for the dense index."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_util import max_rel_err, to_dev, to_host
from test_gpu_backward import m, ref  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 255, 257, 509, 512, 513, 1023, 4095, 4097, 8191, 16387, 32771, 65533, 65537])
@pytest.mark.parametrize("kind", ["plain", "zeros", "ties"])
def test_topk_row_lengths(m, ref, n, kind):  # noqa: F811
    e = 5
    rng = np.random.default_rng(n)
    S = rng.random((n, e), dtype=np.float32)
    if kind == "zeros":
        S[rng.random((n, e)) < 0.9] = 0.0
    elif kind == "ties":
        S = (np.round(S * 8) / 8).astype(np.float32)
    k = max(1, n // 4)
    G = torch.empty((e, k), dtype=torch.float32, device="cuda")
    I = torch.empty((e, k), dtype=torch.int32, device="cuda")
    m.ec_moe_topk_tokens(to_dev(np.ascontiguousarray(S.T)), k, G, I, None)
    torch.cuda.synchronize()
    G_o, I_o = ref.topk_tokens(S, k)
    assert (to_host(I) == I_o).all() and (to_host(G) == G_o).all()


@pytest.mark.parametrize("n,d,e,k,hot", [
    (40, 128, 100, 10, 5),       # 16 lanes per token, tokens in up to 100 lists
    (33, 8, 300, 7, 3),          # one piece per row, ten bitmap words
    (50, 2560, 1024, 9, 4),      # the most experts, several pieces per lane
    (70000, 64, 40, 3000, 0),    # too large for the static array's dense index: lists
])
@pytest.mark.parametrize("bf16", [True, False])
def test_combine_lists(m, ref, n, d, e, k, hot, bf16):  # noqa: F811
    rng = np.random.default_rng(n + d)
    rest = [rng.choice(np.arange(hot, n), size=k - hot, replace=False) for _ in range(e)]
    I = np.sort(np.stack([np.concatenate([np.arange(hot), r]) for r in rest]), axis=1).astype(np.int32)
    G = rng.random((e, k), dtype=np.float32)
    Xe = rng.standard_normal((e, k, d), dtype=np.float32)
    if bf16:
        Xe = wl.f32_to_bf16_bits(Xe)
    dt = torch.bfloat16 if bf16 else torch.float32
    out = [torch.full((n, d), float("nan"), dtype=dt, device="cuda") for _ in range(2)]
    ws = m.alloc_workspace(n, d, e, k, 0, m.EC_BF16 if bf16 else m.EC_F32)
    dXe, dG, dI = to_dev(Xe), to_dev(G), to_dev(I)
    m.ec_moe_combine(dXe, dG, dI, out[0], ws)
    m.ec_moe_combine_static(dXe, dG, dI, out[1])
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])
    # one rounding of an fp32 sum: 2^-8 of the value in bf16; e fp32 additions otherwise
    assert max_rel_err(to_host(out[0]), ref.combine(Xe, G, I, n)) <= (2.0 ** -8 if bf16 else e * 2.0 ** -24 + 1e-6)
