"""3 x 3 depthwise layers of short columns, which take the batch norms around them along (dw_small_fwd_kernel, dw_small_bwd_kernel), at the
edges: images of two pixels, of one row and of one column, rows around a whole number of waves and of 512, the most rows that take
the fused kernels and one image more, few channels, every rectifier; a layer that reads the block's input, one behind a dense layer,
one behind a depthwise layer, and one whose input has another reader.  Every operation of a one-block step against the plain fp64 oracle
primitives on the tensors that the library read, at the bounds of local_parity.py."""
import pytest

import local_parity
from paper_2301_12443_amd import workloads as W

pytestmark = pytest.mark.gpu

# (batch, h, w, channels, rectifier)
SHAPES = [
    (40, 1, 2, 8, W.ACT_RELU),
    (40, 1, 5, 24, W.ACT_RELU6),
    (37, 7, 1, 40, W.ACT_NONE),
    (64, 2, 4, 64, W.ACT_RELU),           # 512 rows
    (33, 4, 4, 96, W.ACT_RELU),           # 528
    (85, 4, 4, 136, W.ACT_RELU6),         # 1360
    (128, 4, 4, 32, W.ACT_RELU),          # 2048: the most ...
    (129, 4, 4, 32, W.ACT_RELU),          # ... and one image more
]


@pytest.mark.parametrize("precision", ["bf16", "f32"])
@pytest.mark.parametrize("n,h,w,c,act", SHAPES)
def test_every_operation_of_a_small_block(n, h, w, c, act, precision):
    t, b = W.Block(), W.Block()
    t.cba(0, c, 1, act=W.ACT_NONE)
    v = b.cba(0, 16, 3, groups=16, act=act)
    v = b.cba(v, c, 1, act=act)
    v = b.cba(v, c, 3, groups=c, act=act)
    v = b.cba(v, c, 3, groups=c, act=act)
    v = b.cba(v, c, 1, act=act)
    b.add(v, b.cba(v, c, 3, groups=c, act=W.ACT_NONE))
    worst = local_parity.run_and_check(W.Workload("dw_small", n, (16, h, w), [t], [b], precision, lr=0.05), n, precision=precision)
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)
