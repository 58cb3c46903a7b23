"""The small-tile implicit GEMM with its operands in a ring of LDS stages (igemm_kernel, RING) and the tile that such a launch takes
(free_tile), at the edges: fewer and more reduction steps than stages, K steps of 64 and 32, a reduction cut in two, ragged rows and
columns, every tile shape, stride 2 both ways, images smaller than the filter, and launches that add to a gradient.  Every operation of
a one-block step against the plain fp64 oracle primitives on the tensors that the library read, at the bf16 bound of local_parity.py: one
rounding to bfloat16 separates the two sides (2^-9 of a value, up to twice that where two are added), a wrong index, mask or stage is
off by the size of the result."""
import pytest

import local_parity
from paper_2301_12443_amd import workloads as W

pytestmark = pytest.mark.gpu

# (batch, h, w, channels of the block's input, of the layer's input, of its output, k, stride)
SHAPES = [
    (1, 9, 7, 64, 64, 64, 1, 1),         # one step, 63 rows: a ragged tile of 64 x 64
    (5, 4, 4, 64, 128, 72, 1, 1),        # two steps (as many as stages), 72 of 128 columns
    (3, 5, 5, 64, 192, 512, 1, 1),       # three steps
    (85, 2, 2, 64, 512, 512, 1, 1),      # 340 rows, eight steps
    (9, 2, 2, 64, 256, 512, 3, 1),       # images smaller than the filter, 36 rows, the reduction cut in two
    (13, 7, 7, 64, 320, 1024, 1, 1),     # 64 x 128 tiles ...
    (64, 7, 7, 64, 192, 2048, 1, 1),     # ... 128 x 128 of them, ragged rows (3136)
    (20, 14, 14, 64, 64, 128, 3, 1),     # 3920 rows
    (6, 13, 13, 64, 128, 192, 3, 2),     # stride 2 on an odd image: backward-data by parity
    (6, 12, 12, 64, 96, 160, 3, 1),      # K step 32
    (33, 7, 7, 32, 160, 96, 1, 1),       # ... five steps, 96 columns
    (30, 13, 13, 64, 384, 64, 1, 1),     # 5070 rows: batch-norm sums in the store
    (40, 12, 12, 32, 96, 32, 1, 1),      # ... 32 columns
]


def _workload(n, h, w, c0, ci, co, k, s):
    t, b = W.Block(), W.Block()
    t.cba(0, co, k, s, act=W.ACT_NONE)
    v = b.cba(0, ci, 1, act=W.ACT_NONE)
    # two readers of v: the second backward-data launch adds onto the first one's result
    a = b.cba(v, co, k, s, act=W.ACT_NONE)
    c = b.cba(v, co, 1, s, act=W.ACT_NONE)
    b.add(a, c)
    return W.Workload("ring_small", n, (c0, h, w), [t], [b], "bf16", lr=0.05)


@pytest.mark.parametrize("n,h,w,c0,ci,co,k,s", SHAPES)
def test_every_operation_of_a_small_block(n, h, w, c0, ci, co, k, s):
    worst = local_parity.run_and_check(_workload(n, h, w, c0, ci, co, k, s), n, precision="bf16")
    print(", ".join(f"{key} {e:.1e}" for key, e in sorted(worst.items())), flush=True)
