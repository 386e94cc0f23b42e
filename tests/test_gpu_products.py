"""Layer products at the edges of their tiles: whole layers, forward and backward, against the oracle, at sizes that
select each tile form and leave remainders in every dimension.  The bars are those of the fixed-shape tests: 1e-5 for
fp32 (a length-k fp32 sum is good to k * 2^-24 of its terms), 2e-2 for bf16 tensors."""
import pytest

import workloads as wl
from test_gpu_backward import m, ref, test_backward_reduced as check_backward  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(n=37, d=33, e=3, c=1.0, d_ff=31),                # scalar loads, one K stage and a remainder, 12-row buckets
    dict(n=260, d=68, e=4, c=2.0, d_ff=132),              # 16-byte loads, K-sharing tiles with remainders, k = 130
    dict(n=2048, d=96, e=4, c=2.0, d_ff=1540),            # 128 x 128 tiles, remainder columns
    dict(n=1300, d=130, e=16, c=2.0, d_ff=258),           # 64 x 64 tiles, scalar loads, short last split of tokens
])
def test_fp32_products(m, ref, kw):  # noqa: F811
    check_backward(m, ref, "cfg1", dict(kw, act=wl.ACT_GELU), 1e-5)
